"""What the library asks of the HIP runtime, without a GPU: every kernel launch that fails is reported by the call that made it, and every
launch of a profiled kernel has a pair of events of its own.

The library is loaded in a process of its own behind a stand-in for the runtime's entry points that launches nothing, counts the launches,
lets one of them fail (a status that is taken and dropped on the way shows as METIS_OK) and notes between which launches an event was
recorded."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3;
static int launches, failing, error;
static struct { dim3 g, b; size_t l; void* s; } cfg;
void fail_at(int n) { launches = 0; failing = n; error = 0; }
int launch_count(void) { return launches; }
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void* s) { cfg.g = g; cfg.b = b; cfg.l = l; cfg.s = s; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, void** s) { *g = cfg.g; *b = cfg.b; *l = cfg.l; *s = cfg.s; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t l, void* s) {
    if (++launches == failing) error = 1;
    return error;
}
int hipGetLastError(void) { int e = error; error = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
static int records, event_at[64], event_id[64];
int hipEventRecord(void* e, void* s) {
    if (records < 64) { event_at[records] = launches; event_id[records] = (int)(size_t)e; }
    ++records;
    return 0;
}
int record_count(void) { return records; }
int recorded_at(int i) { return event_at[i]; }
int recorded_event(int i) { return event_id[i]; }
"""

FAKE = 1 << 30                                   # an aligned address that is never read


def _calls(metis):
    """name -> a call of the library; the operands' sizes select its kernels"""
    L = metis.lib()
    keep = []

    def mat(rows, cols, dtype=metis.BF16):
        keep.append(metis.Mat(FAKE, rows, cols, cols, dtype))
        return C.byref(keep[-1])

    def split(M, N, k):
        f = lambda rows, cols: metis.Fp4(FAKE, FAKE, 1.0, rows, cols)
        keep.append(metis.Split(f(k, M), f(k, N), f(M, N), f(N, M), FAKE, k))
        return C.byref(keep[-1])

    def grads(N, K, k, dtype):
        return lambda: L.metis_fp4_factor_grads(None, mat(N, K, dtype), split(N, K, k), FAKE, FAKE, FAKE, FAKE, 1 << 40)

    def decompose(*jobs):
        def call():
            arr = (metis.DecomposeJob * len(jobs))()
            for a, (M, N, k, p) in zip(arr, jobs):
                keep.append(metis.Mat(FAKE, M, N, N, metis.BF16))
                a.A, a.k, a.oversample, a.sample_rate, a.sample_group = C.pointer(keep[-1]), k, p, 1.0, 1
                a.U = a.S = a.V = a.amax_out = a.workspace = a.info = FAKE
                a.workspace_bytes = 1 << 40
            return L.metis_decompose_batch(None, len(jobs), arr)
        return call

    def linear(name, a, b, out, k):
        return lambda: getattr(L, "metis_fp4_linear_" + name)(None, split(*a, k), split(*b, k), mat(*out), FAKE, 1 << 40)

    return {
        "factor gradients, bf16": grads(1024, 2048, 64, metis.BF16),
        "factor gradients, fp32": grads(1024, 2048, 8, metis.F32),
        "factor gradients, generic kernels": grads(1024, 2048, 20, metis.F32),
        "decomposition": decompose((1024, 512, 64, 16)),
        "decomposition, generic kernels": decompose((1024, 512, 61, 10)),
        "decompositions of several orders": decompose((1024, 512, 64, 16), (512, 1024, 20, 12), (256, 256, 3, 1)),
        "large decomposition, generic kernels": decompose((16384, 4096, 85, 10)),
        "forward": linear("fwd", (4096, 4096), (4096, 4096), (4096, 4096), 64),
        "forward, few rows": linear("fwd", (16, 4096), (4096, 4096), (16, 4096), 64),
        "weight gradient": linear("wgrad", (512, 1024), (512, 2048), (1024, 2048), 20),
    }


def _failed_launches(stub, metis):
    for name, call in _calls(metis).items():
        stub.fail_at(0)
        assert call() == 0, name
        n = stub.launch_count()
        assert n > 1, name
        for i in range(1, n + 1):
            stub.fail_at(i)
            status = call()
            assert status == -4, f"{name}: launch {i} of {n} failed, status {status}"
        print(name, n)


def _brackets(stub, metis):
    n = 16
    start, stop = (C.c_void_p * n)(*range(101, 101 + n)), (C.c_void_p * n)(*range(201, 201 + n))
    for name, launches in (("decomposition", 1), ("decompositions of several orders", 2)):
        assert metis.lib().metis_profile_events(metis.PROF_BROADCAST, start, stop, n) == 0
        first = stub.record_count()
        stub.fail_at(0)
        assert _calls(metis)[name]() == 0
        pairs = [(stub.recorded_event(i), stub.recorded_at(i), stub.recorded_event(i + 1), stub.recorded_at(i + 1))
                 for i in range(first, stub.record_count(), 2)]
        assert [(a, c) for a, _, c, _ in pairs] == [(101 + i, 201 + i) for i in range(launches)], (name, pairs)
        assert all(after == before + 1 for _, before, _, after in pairs), (name, pairs)


def _child(check, runtime):
    stub = C.CDLL(runtime, mode=C.RTLD_GLOBAL)
    sys.path.insert(0, ROOT)
    from paper_2509_00404_amd import metis
    {"failed_launches": _failed_launches, "brackets": _brackets}[check](stub, metis)


@pytest.mark.parametrize("check", ["failed_launches", "brackets"])
def test_behind_a_stand_in_for_the_runtime(tmp_path, check):
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH) or not shutil.which("gcc"):
        pytest.skip("library not built, or no C compiler")
    src, runtime = tmp_path / "runtime.c", tmp_path / "runtime.so"
    src.write_text(RUNTIME)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(runtime), str(src)], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), check, str(runtime)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    _child(*sys.argv[1:])
