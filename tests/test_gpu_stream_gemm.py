"""GPU parity of the streaming GEMM kernel (256 or more tiles of 256 x 256, at least 32 units of 128 per CU; 64 without factors):
ragged edge tiles, a cut last round, an odd number of rows, extra columns for a partial last stage, outputs that cannot be stored
in vectors, many tiles of few units, and the call with too little workspace for it, on the kernel it replaced.  The three products
at full size are in tests/test_gpu_fullsize.py.  Bars of tests/test_gpu_linear.py."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_helpers import elementwise_bound, make_split, operand_parts, split_to_oracle, take_row_groups
from oracle import linear as olin
from test_gpu_linear import metis  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def plan_bytes(L, N, K):
    """Room for the block scales of both operands: 4 KiB per 256 rows and 128 elements."""
    return (-(-L // 256) + -(-N // 256)) * (K // 128) * 4096


def tail_bytes(L, N, K):
    """Room for the fp32 parts of the tiles of the last round of 256, at most four of each."""
    tail = (-(-L // 256) * -(-N // 256)) % 256
    parts = min(256 // tail, 4, K // 128) if tail else 1
    return tail * parts * 262144 if parts > 1 else 0


def mandatory_bytes(metis, xs, ws, Y, room):  # noqa: F811
    """The part of the workspace without which a product of split operands is refused.  Found on the host: with a misaligned workspace
    a call whose size suffices is refused right after the size was looked at."""
    sa, sb, out = xs.c(), ws.c(), metis._mat(Y)

    def suffices(size):
        return metis.lib().metis_fp4_linear_fwd(None, ctypes.byref(sa), ctypes.byref(sb), ctypes.byref(out),
                                                room.data_ptr() + 8, size) == -1

    low, high = 0, room.numel()
    assert suffices(high) and not suffices(low)
    while high - low > 1:
        mid = (low + high) // 2
        low, high = (low, mid) if suffices(mid) else (mid, high)
    return high


@pytest.mark.parametrize("L,N,K,kx,kw,dtype,ld_extra", [
    (4112, 4112, 2064, 24, 24, torch.bfloat16, 0),      # 289 tiles: edges of 16 rows and columns, 33 tiles cut in 4, 16 more columns
    (4099, 4096, 2048, 0, 8, torch.float32, 0),         # an odd number of rows, extra columns padded to one unit
    (4112, 4112, 4096, 0, 0, torch.bfloat16, 0),        # no extra columns at all
    (4096, 4096, 4096, 16, 48, torch.float32, 0),       # whole tiles only, one per CU, two units of extra columns
    (4099, 4112, 2048, 0, 72, torch.bfloat16, 1),       # rows of C start on odd elements; three units
    (4096, 4128, 2048, 0, 16, torch.float32, 3),
    (4112, 4112, 4112, 0, 0, torch.bfloat16, 0),        # no factors, 16 columns of a partial last stage and 16 of padding
])
def test_against_the_oracle(metis, L, N, K, kx, kw, dtype, ld_extra):  # noqa: F811
    from paper_2509_00404_amd import workloads
    assert -(-L // 256) * -(-N // 256) >= 256
    X = workloads.gaussian(L, K, 1)
    W = workloads.planted(N, K, workloads.power_law(min(N, K, 96), 1.0), 2, noise_top=0.01, rms=0.02)
    xs = make_split(metis, X, kx, 8, 0.25, 11, want_t=False)[0]
    ws = make_split(metis, W, kw, 8, 0.25, 12, want_t=False)[0]
    nbytes = metis.linear_workspace_bytes(L, N, K, max(kx, kw))
    room = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
    full = torch.full((L, N + ld_extra), float("nan"), dtype=dtype, device="cuda")
    Y = full[:, :N]
    metis.fp4_linear_fwd(xs, ws, Y, room)
    if kx + kw > 0:
        first = mandatory_bytes(metis, xs, ws, Y, room)                  # ... the tail's region, the plan's, each on 256 bytes
        plan_at = -(-(first + tail_bytes(L, N, K)) // 256) * 256
        plan_end = plan_at + plan_bytes(L, N, K)
    else:
        first = plan_at = 256                                            # (not needed at all)
        plan_end = room.numel()
    assert plan_end <= room.numel() and bool((room[plan_at:plan_end] != 0xA5).any())
    # too little for the scale plan: without any of the optional regions, and with the last round's; the plan's place stays as it is
    others = []
    for size in (first, plan_end - 1):
        if size > first and kx + kw == 0:
            continue
        room.fill_(0xA5)
        others.append(torch.empty((L, N), dtype=dtype, device="cuda"))
        metis.fp4_linear_fwd(xs, ws, others[-1], room[:size])
        assert bool((room[plan_at:] == 0xA5).all())
    room.fill_(0xA5)
    phased = torch.empty((L, N), dtype=dtype, device="cuda")
    metis.fp4_linear_phase(metis.LINEAR_FWD, metis.LINEAR_PREPARE, xs, ws, None, room)
    metis.fp4_linear_phase(metis.LINEAR_FWD, metis.LINEAR_APPLY, xs, ws, phased, room)
    torch.cuda.synchronize()
    assert torch.equal(Y, phased)
    assert bool(torch.isnan(full[:, N:]).all())                          # nothing beside the rows is written
    xo, wo = split_to_oracle(xs), split_to_oracle(ws)
    ref = olin.linear_fwd(xo, wo)
    bound = elementwise_bound(operand_parts(xo), operand_parts(wo), ref, dtype)
    for out in (Y, *others):
        assert (np.abs(out.double().cpu().numpy() - ref) <= bound).all()


@pytest.mark.parametrize("L,N,K,kx,kw,dtype", [
    (8192, 8192, 1024, 0, 8, torch.bfloat16),           # four whole tiles a workgroup, one after the other
    (8208, 4608, 1408, 16, 24, torch.float32),          # two whole tiles, then a part of one; three units of extra columns
    (16400, 16384, 256, 0, 8, torch.bfloat16),          # sixteen tiles of two units, then parts of one
    (16384, 16384, 256, 8, 8, torch.float32),
    (32784, 16384, 128, 0, 8, torch.bfloat16),          # tiles of one unit and one of extra columns
    (16400, 16384, 512, 0, 0, torch.bfloat16),          # four units, no extra columns, edge tiles among whole ones
])
def test_many_tiles_of_few_units(metis, L, N, K, kx, kw, dtype):  # noqa: F811
    """The look-ahead of three units crosses the ends of tiles, of their extra columns and of stores on their way in every combination.
    16 rows of every tile row (every second one beyond 100) against the oracle, all columns."""
    g = torch.Generator().manual_seed(K)
    xs = make_split(metis, torch.randn((L, K), generator=g).bfloat16(), kx, 8, 0.25, 11, want_t=False)[0]
    ws = make_split(metis, (0.02 * torch.randn((N, K), generator=g)).bfloat16(), kw, 8, 0.25, 12, want_t=False)[0]
    room = torch.empty((metis.linear_workspace_bytes(L, N, K, max(kx, kw)),), dtype=torch.uint8, device="cuda")
    Y = torch.full((L, N), float("nan"), dtype=dtype, device="cuda")
    metis.fp4_linear_fwd(xs, ws, Y, room)
    torch.cuda.synchronize()
    tiles = range(0, -(-L // 256), 1 if L < 25600 else 2)
    groups = sorted({min(16 * t + int(torch.randint(16, (1,), generator=g)), L // 16 - 1) for t in tiles} | {0, L // 16 - 1})
    xo, rows = take_row_groups(split_to_oracle(xs), groups)
    wo = split_to_oracle(ws)
    ref = olin.linear_fwd(xo, wo)
    got = Y[torch.from_numpy(rows).cuda()].double().cpu().numpy()
    assert (np.abs(got - ref) <= elementwise_bound(operand_parts(xo), operand_parts(wo), ref, dtype)).all()
    assert bool(torch.isfinite(Y).all())


def test_a_scale_that_is_not_a_number(metis):  # noqa: F811
    """A block scale of E4M3's NaN makes its row (of X) or column (of W) NaN and leaves every other output as it was."""
    L, N, K = 4112, 4112, 4096
    g = torch.Generator().manual_seed(3)
    xs = make_split(metis, torch.randn((L, K), generator=g).bfloat16(), 0, 8, 0.25, 11, want_t=False)[0]
    ws = make_split(metis, torch.randn((N, K), generator=g).bfloat16(), 0, 8, 0.25, 12, want_t=False)[0]
    room = torch.empty((metis.linear_workspace_bytes(L, N, K, 0),), dtype=torch.uint8, device="cuda")
    clean, got = (torch.empty((L, N), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    metis.fp4_linear_fwd(xs, ws, clean, room)
    xs.R.scales[4111, 255] = 0x7F
    ws.R.scales[17, 8] = 0xFF
    metis.fp4_linear_fwd(xs, ws, got, room)
    torch.cuda.synchronize()
    assert bool(torch.isnan(got[4111]).all()) and bool(torch.isnan(got[:, 17]).all())
    got[4111], got[:, 17] = clean[4111], clean[:, 17]
    assert torch.equal(got, clean)


@pytest.mark.parametrize("kx,kw", [(0, 8), (8, 0), (0, 0), (8, 8)])
def test_residuals_may_be_written_between_the_phases(metis, kx, kw):  # noqa: F811
    """PREPARE uses of a residual only what the other side's factors multiply: one that meets none is read by APPLY alone, codes and
    block scales alike.  Whole stages, so that no columns of the residuals are among the extra ones."""
    L, N, K = 4112, 4112, 4096
    g = torch.Generator().manual_seed(kx + 2 * kw)
    xs = make_split(metis, torch.randn((L, K), generator=g).bfloat16(), kx, 8, 0.25, 11, want_t=False)[0]
    ws = make_split(metis, (0.02 * torch.randn((N, K), generator=g)).bfloat16(), kw, 8, 0.25, 12, want_t=False)[0]
    room = torch.empty((metis.linear_workspace_bytes(L, N, K, max(kx, kw)),), dtype=torch.uint8, device="cuda")
    want, got = (torch.empty((L, N), dtype=torch.float32, device="cuda") for _ in range(2))
    metis.fp4_linear_fwd(xs, ws, want, room)
    room.fill_(0xA5)
    late = [s.R for s, other in ((xs, kw), (ws, kx)) if other == 0]
    kept = [(r.codes.clone(), r.scales.clone()) for r in late]
    for r in late:
        r.codes.fill_(0x33)
        r.scales.fill_(0x38)
    metis.fp4_linear_phase(metis.LINEAR_FWD, metis.LINEAR_PREPARE, xs, ws, None, room)
    for r, (c, s) in zip(late, kept):
        r.codes.copy_(c)
        r.scales.copy_(s)
    metis.fp4_linear_phase(metis.LINEAR_FWD, metis.LINEAR_APPLY, xs, ws, got, room)
    torch.cuda.synchronize()
    assert torch.equal(want, got)
