"""GPU parity of large products whose contraction is not a multiple of the 128-deep stage: the last elements travel
as extra bf16 columns (exact) of whichever kernel takes the output, the pipelined one or 128 x 128 tiles, or, for two unsplit
operands without a workspace, through the bounds-checked staging.  Same bars as tests/test_gpu_linear.py."""
import pytest
import torch

from gpu_helpers import make_split, operand_parts, split_to_oracle, elementwise_bound
from oracle import linear as olin
from test_gpu_linear import GEMM_RTOL, _three, metis  # noqa: F401  (metis is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,K,kx,kw,kg", [
    (1040, 1072, 1264, 16, 24, 8),      # residues 16, 48, 112 over the three contractions; 128 x 128 tiles, as the next two
    (1136, 1088, 1040, 0, 20, 0),       # one operand unsplit, 4 extra low-rank pad columns
    (1024, 1024, 144, 16, 16, 16),      # a single whole stage and one block
    (3056, 1520, 1040, 72, 80, 64),     # more than 64 low-rank columns a side; the forward product pipelined
    (2192, 2064, 2160, 16, 0, 72),      # all three pipelined: residues 112, 16, 16, one operand unsplit
])
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
def test_partial_last_stage(metis, L, N, K, kx, kw, kg, out_dtype):  # noqa: F811
    from paper_2509_00404_amd import workloads
    X = workloads.planted(L, K, workloads.power_law(min(L, K, 144), 1.2), 1, rms=1.0, outlier_cols=1)
    W = workloads.planted(N, K, workloads.power_law(min(N, K, 144), 1.0), 2, noise_top=0.01, rms=0.02)
    G = workloads.planted(L, N, workloads.power_law(min(L, N, 144), 1.0), 3, rms=1e-3)
    e, _, _ = _three(metis, X, W, G, kx, kw, kg, 8, 0.25, out_dtype)
    tol = GEMM_RTOL if out_dtype == torch.bfloat16 else 5e-3
    assert max(e) < tol, e


@pytest.mark.parametrize("M,N,K", [(1040, 1168, 400), (4112, 2064, 272)])
def test_unsplit_with_and_without_workspace(metis, M, N, K):  # noqa: F811
    from paper_2509_00404_amd import workloads
    a = make_split(metis, workloads.gaussian(M, K, 1), 0, 0, 1.0, 0, want_t=False)[0]
    b = make_split(metis, workloads.gaussian(N, K, 2), 0, 0, 1.0, 0, want_t=False)[0]
    ao, bo = split_to_oracle(a), split_to_oracle(b)
    ref = olin.linear_fwd(ao, bo)
    bound = elementwise_bound(operand_parts(ao), operand_parts(bo), ref, torch.float32)
    nbytes = metis.linear_workspace_bytes(M, N, K, 0)
    for ws in (None, torch.empty((nbytes + 8,), dtype=torch.uint8, device="cuda")[8:],      # misaligned: not used
               torch.empty((nbytes,), dtype=torch.uint8, device="cuda")):
        C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        metis.fp4_linear_fwd(a, b, C, ws)
        assert (abs(C.double().cpu().numpy() - ref) <= bound).all()
