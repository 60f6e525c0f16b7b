"""The C-ABI library loads and exports every symbol include/metis.h declares (no GPU needed)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "metis.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(metis_[a-z0-9_]+)\s*\(", text)))


def test_header_and_binding_agree():
    from paper_2509_00404_amd import metis
    assert _declared() == metis.exported_symbols()


def test_library_exports_every_declared_symbol():
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH):
        pytest.skip("library not built (run __graft_entry__.build())")
    L = ctypes.CDLL(metis.LIB_PATH)
    for name in _declared():
        assert hasattr(L, name), name
    assert metis.lib().metis_version() >= 1
    assert metis.lib().metis_status_string(-2) == b"bad shape"


def test_host_side_argument_checks_need_no_gpu():
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH):
        pytest.skip("library not built")
    L = metis.lib()
    assert L.metis_sample_count(8192, 64, 16, 1.0 / 16) == 512
    assert L.metis_sample_count(256, 8, 8, 0.25) == 64
    assert L.metis_sample_count(8192, 64, 16, 0.001) == 80
    assert L.metis_sample_count(50, 64, 16, 1.0) == 50
    assert L.metis_sample_count(100, 4, 4, 0.0) == 0
    # null pointers and bad shapes are refused before anything is enqueued
    assert L.metis_sample_rows(None, 1, 100, 10, None) == -1
    assert L.metis_gaussian_omega(None, 1, 0, 4, None) == -1
    assert L.metis_quantize(None, None, None, None) == -1
    assert L.metis_quantize_sr(None, None, 0, None, None) == -1


@pytest.mark.parametrize("L,N,K", [(8192, 4096, 4096), (16, 4096, 4096), (64, 1040, 4096), (2048, 1024, 4096), (1360, 1232, 752),
                                   (128, 256, 512), (4096, 64, 14336), (48, 48, 4096), (3056, 1520, 1040)])
def test_linear_workspace_covers_every_smaller_rank(L, N, K):
    """A workspace of linear_workspace_bytes(..., k) serves operands of any ranks up to k, equal or not: none of the three products
    finds it too small.  The workspace pointer is misaligned, so that a call whose size suffices is refused right after the size
    was looked at and nothing is enqueued (status -1), with or without a GPU."""
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH):
        pytest.skip("library not built")
    lib = metis.lib()
    fake = 1 << 20                                          # never read: the call ends before anything is enqueued

    def fp4(rows, cols):
        return metis.Fp4(fake, fake, 1.0, rows, cols)

    def split(M, N_, k):
        f = (fp4(k, M), fp4(k, N_)) if k else (metis.Fp4(None, None, 1.0, 0, 0),) * 2
        return metis.Split(*f, fp4(M, N_), fp4(N_, M), fake, k)

    for k in (1, 16, 64, 65, 80, 128):
        size = metis.linear_workspace_bytes(L, N, K, k)
        ranks = sorted({r for r in (0, 1, 8, 20, 63, 64, 65, 72, 80, 127, 128) if r <= k} | {k})
        for ka in ranks:
            for kb in ranks:
                if ka + kb == 0:
                    continue                                # two unsplit operands need no workspace
                for fn, a, b, (rows, cols) in ((lib.metis_fp4_linear_fwd, (L, K), (N, K), (L, N)),
                                               (lib.metis_fp4_linear_dgrad, (L, N), (N, K), (L, K)),
                                               (lib.metis_fp4_linear_wgrad, (L, N), (L, K), (N, K))):
                    sa, sb = split(*a, ka), split(*b, kb)
                    out = metis.Mat(fake, rows, cols, cols, metis.F32)
                    st = fn(None, ctypes.byref(sa), ctypes.byref(sb), ctypes.byref(out), fake + 8, size)
                    assert st == -1, (fn.__name__, k, ka, kb, st)


@pytest.mark.parametrize("L,N,K", [(16384, 4112, 4112), (4112, 4112, 4112), (8208, 14352, 4112), (4096, 4096, 8192), (4112, 8192, 2064)])
def test_linear_workspace_grows_with_the_rank(L, N, K):
    """Room for operands of ranks up to k is room for operands of ranks up to any smaller one: the optional regions (parts of a cut last
    round, the streaming GEMM's scale plan) included, without which a call runs on another kernel."""
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH):
        pytest.skip("library not built")
    sizes = [metis.linear_workspace_bytes(L, N, K, k) for k in range(129)]
    assert all(a <= b for a, b in zip(sizes[1:], sizes[2:]))


def test_streaming_gemm_leaves_rows_that_its_offsets_cannot_span():
    """The streaming GEMM addresses a tile's 256 rows of codes with 32-bit offsets: 255 rows of K / 2 bytes and 64 more have to fit.  Seen
    in the room for its scale plan (4 KiB per 256 rows and 128 elements), which is most of the workspace at these sizes."""
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH):
        pytest.skip("library not built")
    K = 33686016                                             # a multiple of 128
    assert 255 * (K // 2) + 64 <= 2 ** 32 < 255 * ((K + 128) // 2) + 64
    plan = 2 * 16 * (K // 128) * 4096
    assert metis.linear_workspace_bytes(4096, 4096, K, 0) > plan
    assert metis.linear_workspace_bytes(4096, 4096, K + 128, 0) < 0.6 * plan


def test_tensor_scale_helper_is_the_smallest_covering_power_of_two():
    from paper_2509_00404_amd import metis
    if not os.path.exists(metis.LIB_PATH):
        pytest.skip("library not built")
    import numpy as np
    ts = metis.tensor_scale
    assert ts(6 * 448.0) == 1.0 and ts(6 * 448.0 + 1) == 2.0 and ts(1.0) == 2.0 ** -11
    assert ts(0.0) == 1.0 and ts(-3.0) == 1.0 and ts(float("inf")) == 1.0 and ts(float("nan")) == 1.0
    rs = np.random.default_rng(0)
    for a in np.exp(rs.uniform(-40, 40, 2000)).astype(np.float32):
        g = ts(float(a))
        m, e = np.frexp(g)
        assert m == 0.5                                            # a power of two
        assert 2688.0 * g >= float(a) and 2688.0 * (g / 2) < float(a)


def test_bench_refuses_more_than_one_gpu():
    """One GPU is the whole target: `bench.py --gpus N` with N > 1 exits with a message before touching a device."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 2
    assert "ONE GPU" in r.stderr
    assert r.stdout.strip() == ""
