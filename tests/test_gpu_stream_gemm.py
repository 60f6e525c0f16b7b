"""GPU parity of the streaming GEMM kernel (256 or more tiles of 256 x 256, at least 32 units of 128 per CU; 64 without factors):
ragged edge tiles, a cut last round, an odd number of rows, extra columns for a partial last stage, outputs that cannot be stored
in vectors, and the call with too little workspace for it, on the kernel it replaced.  Bars of tests/test_gpu_linear.py."""
import numpy as np
import pytest
import torch

from gpu_helpers import elementwise_bound, make_split, operand_parts, split_to_oracle
from oracle import linear as olin
from test_gpu_linear import metis  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,K,kx,kw,dtype,ld_extra", [
    (4112, 4112, 2064, 24, 24, torch.bfloat16, 0),      # 289 tiles: edges of 16 rows and columns, 33 tiles cut in 4, 16 more columns
    (4099, 4096, 2048, 0, 8, torch.float32, 0),         # an odd number of rows, extra columns padded to one unit
    (4112, 4112, 4096, 0, 0, torch.bfloat16, 0),        # no extra columns at all
    (4096, 4096, 4096, 16, 48, torch.float32, 0),       # whole tiles only, one per CU, two units of extra columns
    (4099, 4112, 2048, 0, 72, torch.bfloat16, 1),       # rows of C start on odd elements; three units
    (4096, 4128, 2048, 0, 16, torch.float32, 3),
])
def test_against_the_oracle(metis, L, N, K, kx, kw, dtype, ld_extra):  # noqa: F811
    from paper_2509_00404_amd import workloads
    assert -(-L // 256) * -(-N // 256) >= 256
    X = workloads.gaussian(L, K, 1)
    W = workloads.planted(N, K, workloads.power_law(min(N, K, 96), 1.0), 2, noise_top=0.01, rms=0.02)
    xs = make_split(metis, X, kx, 8, 0.25, 11, want_t=False)[0]
    ws = make_split(metis, W, kw, 8, 0.25, 12, want_t=False)[0]
    nbytes = metis.linear_workspace_bytes(L, N, K, max(kx, kw))
    room = torch.empty((nbytes,), dtype=torch.uint8, device="cuda")
    full = torch.full((L, N + ld_extra), float("nan"), dtype=dtype, device="cuda")
    Y = full[:, :N]
    metis.fp4_linear_fwd(xs, ws, Y, room)
    small = torch.empty((L, N), dtype=dtype, device="cuda")
    metis.fp4_linear_fwd(xs, ws, small, room[:nbytes - 1])              # no room for the scale plan
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
    for out in (Y, small):
        assert (np.abs(out.double().cpu().numpy() - ref) <= bound).all()


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
