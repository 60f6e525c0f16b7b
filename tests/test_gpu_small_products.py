"""GPU parity of products with few rows (at most 64 rows of an unsplit operand, on their own kernels or past the lines to the
general ones) and of small outputs whose contraction is cut into parts; with the bars of tests/test_gpu_linear.py, at edges of
the 32-row / 32-column tiles, the 128-deep stages and the 32-column groups of the low-rank part, and at output widths of any size."""
import pytest
import torch

from gpu_helpers import elementwise_bound, fp4_to_oracle, make_split, operand_parts, rel_fro, split_to_oracle
from oracle import linear as olin
from oracle import quant as oq
from test_gpu_linear import GEMM_RTOL, metis  # noqa: F401  (metis is a fixture)

pytestmark = pytest.mark.gpu


def _product(metis, L, N, K, kx, kw, out_dtype, seed=1):  # noqa: F811
    from paper_2509_00404_amd import workloads
    X = workloads.planted(L, K, workloads.power_law(min(L, K, 128), 1.2), seed, rms=1.0, outlier_cols=1)
    W = workloads.planted(N, K, workloads.power_law(min(N, K, 128), 1.0), seed + 1, noise_top=0.01, rms=0.02)
    xs = make_split(metis, X, kx, 4, 1.0, 11, want_t=False)[0]
    ws = make_split(metis, W, kw, 4, 1.0, 12, want_t=False)[0]
    xo, wo = split_to_oracle(xs), split_to_oracle(ws)
    ref = olin.linear_fwd(xo, wo)
    return xs, ws, ref, elementwise_bound(operand_parts(xo), operand_parts(wo), ref, out_dtype)


@pytest.mark.parametrize("L,N,K,k", [
    (1, 16, 16, 4), (1, 48, 32, 0), (3, 272, 112, 5), (16, 256, 128, 8), (16, 400, 1040, 32), (17, 528, 1184, 33),
    (31, 144, 2064, 64), (32, 1040, 1152, 65), (32, 256, 272, 88), (16, 8208, 272, 64), (5, 8224, 144, 88), (16, 4096, 4096, 64), (8, 160, 5120, 80), (33, 4096, 2064, 16), (64, 272, 4096, 20),
    (65, 304, 1232, 12), (127, 96, 2048, 88), (128, 2064, 400, 33), (100, 528, 1040, 0)])
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
def test_few_rows(metis, L, N, K, k, out_dtype):  # noqa: F811
    if k > 0 and k + 4 > min(N, K):
        k = min(N, K) - 4
    xs, ws, ref, bound = _product(metis, L, N, K, 0, k, out_dtype)
    wsb = torch.empty((max(metis.linear_workspace_bytes(L, N, K, k), 256),), dtype=torch.uint8, device="cuda")
    Y = torch.full((L, N + 8), float("nan"), dtype=out_dtype, device="cuda")
    metis.fp4_linear_fwd(xs, ws, Y[:, :N], wsb)
    got = Y[:, :N].double().cpu().numpy()
    assert torch.isnan(Y[:, N:]).all()
    assert rel_fro(got, ref) < (GEMM_RTOL if out_dtype == torch.bfloat16 else 5e-3)
    assert (abs(got - ref) <= bound).all()
    # the two-phase form is the same product
    Z = torch.full((L, N), float("nan"), dtype=out_dtype, device="cuda")
    metis.fp4_linear_phase(metis.LINEAR_FWD, metis.LINEAR_PREPARE, xs, ws, None, wsb)
    metis.fp4_linear_phase(metis.LINEAR_FWD, metis.LINEAR_APPLY, xs, ws, Z, wsb)
    assert torch.equal(Z, Y[:, :N])


@pytest.mark.parametrize("L,N,K,kx,kw", [
    (48, 4096, 2064, 8, 16),        # 64 x 128 tiles, a partial last stage
    (64, 272, 4096, 8, 20),
    (129, 1040, 4096, 0, 20),
    (16, 256, 1040, 8, 8),          # few rows of a split operand: the general path
    (144, 64, 3008, 12, 12),        # 128 x 64 tiles
    (400, 528, 1232, 20, 24),
    (1008, 1040, 2048, 16, 16),
    (65, 4096, 272, 0, 0)])         # nothing to cut
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
def test_cut_contraction(metis, L, N, K, kx, kw, out_dtype):  # noqa: F811
    xs, ws, ref, bound = _product(metis, L, N, K, kx, kw, out_dtype, seed=5)
    nbytes = max(metis.linear_workspace_bytes(L, N, K, max(kx, kw)), 256)
    Y = torch.full((L, N), float("nan"), dtype=out_dtype, device="cuda")
    metis.fp4_linear_fwd(xs, ws, Y, torch.empty((nbytes,), dtype=torch.uint8, device="cuda"))
    y = Y.double().cpu().numpy()
    assert rel_fro(y, ref) < (GEMM_RTOL if out_dtype == torch.bfloat16 else 5e-3)
    assert (abs(y - ref) <= bound).all()


@pytest.mark.parametrize("L,N,K,kx,kw", [
    (2320, 2064, 1280, 16, 24),     # pipelined kernel, its 90 tiles in two parts each, ragged edges
    (2320, 2064, 1296, 0, 24),      # the same with extra columns for the last 16 elements
    (2048, 2048, 1024, 8, 8),       # 256 small tiles, whole
    (1104, 1040, 2192, 16, 20),     # small tiles in parts, extra columns
    (1024, 3600, 1152, 0, 0)])      # 70 large tiles, 232 small ones
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
def test_large_sides_few_tiles(metis, L, N, K, kx, kw, out_dtype):  # noqa: F811
    xs, ws, ref, bound = _product(metis, L, N, K, kx, kw, out_dtype, seed=9)
    nbytes = metis.linear_workspace_bytes(L, N, K, max(kx, kw))
    for size in ((nbytes,) if kx + kw else (0, nbytes)):
        Y = torch.full((L, N + 16), float("nan"), dtype=out_dtype, device="cuda")
        metis.fp4_linear_fwd(xs, ws, Y[:, :N], torch.empty((size,), dtype=torch.uint8, device="cuda") if size else None)
        assert torch.isnan(Y[:, N:]).all()
        y = Y[:, :N].double().cpu().numpy()
        assert rel_fro(y, ref) < (GEMM_RTOL if out_dtype == torch.bfloat16 else 5e-3)
        assert (abs(y - ref) <= bound).all()


@pytest.mark.parametrize("L", [16, 100, 200])
def test_unsplit_without_workspace(metis, L):  # noqa: F811
    xs, ws, ref, bound = _product(metis, L, 528, 4096, 0, 0, torch.float32)
    nbytes = metis.linear_workspace_bytes(L, 528, 4096, 0)
    for wsb in (None, torch.empty((nbytes + 8,), dtype=torch.uint8, device="cuda")[8:],       # misaligned: not used
                torch.empty((nbytes,), dtype=torch.uint8, device="cuda")):
        Y = torch.full((L, 528), float("nan"), dtype=torch.float32, device="cuda")
        metis.fp4_linear_fwd(xs, ws, Y, wsb)
        assert (abs(Y.double().cpu().numpy() - ref) <= bound).all()


def _guarded(rows, cols, ld, dtype):
    """[rows, cols] view with row stride ld into NaN-filled storage that goes on for 64 elements behind it."""
    flat = torch.full((rows * ld + 64,), float("nan"), dtype=dtype, device="cuda")
    return flat, flat[:rows * ld].view(rows, ld)[:, :cols]


def _check_guarded(flat, view, ref, bound):
    rows, cols = view.shape
    ld = view.stride(0)
    assert torch.isnan(flat[rows * ld:]).all()                                  # nothing behind the output
    assert torch.isnan(flat[:rows * ld].view(rows, ld)[:, cols:]).all()         # nor in the caller's columns beside it
    assert (abs(view.double().cpu().numpy() - ref) <= bound).all()


# an unsplit right operand may have any number of rows: output widths that are no multiple of 4, contiguous (the next row
# begins where one ends) and padded
@pytest.mark.parametrize("L,N,K,kx", [
    (1, 1, 272, 0), (3, 50, 16, 0), (16, 257, 4096, 0), (16, 1001, 1040, 0), (64, 258, 2064, 0), (33, 1003, 128, 0),     # few rows
    (65, 50, 4096, 0), (100, 250, 4096, 0), (129, 257, 2064, 0), (256, 1001, 4096, 0), (1040, 1041, 4096, 0),     # contraction cut
    (16, 257, 2048, 8), (208, 1002, 3008, 8), (1040, 1041, 2192, 16),                                              # split left operand
    (80, 49, 96, 0), (1024, 1025, 256, 0)])                                                                        # uncut
@pytest.mark.parametrize("pad", [0, 7])
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
def test_widths_of_any_size(metis, L, N, K, kx, pad, out_dtype):  # noqa: F811
    xs, ws, ref, bound = _product(metis, L, N, K, kx, 0, out_dtype, seed=13)
    wsb = torch.empty((max(metis.linear_workspace_bytes(L, N, K, kx), 256),), dtype=torch.uint8, device="cuda")
    flat, Y = _guarded(L, N, N + pad, out_dtype)
    metis.fp4_linear_fwd(xs, ws, Y, wsb)
    _check_guarded(flat, Y, ref, bound)


@pytest.mark.parametrize("L,N,K", [(2048, 33, 250), (4096, 257, 101), (2064, 1041, 1042)])
@pytest.mark.parametrize("pad", [0, 7])
def test_weight_gradient_of_any_size(metis, L, N, K, pad):  # noqa: F811
    # dW[N, K] = G^T X of unsplit operands: only the contraction has to come in blocks of 16
    from paper_2509_00404_amd import workloads
    out_dtype = torch.float32
    t = [workloads.gaussian(L, c, s) for c, s in ((N, 31), (K, 32))]
    ops = []
    for a in t:
        sp = metis.SplitTensor(L, a.shape[1], 0, 1.0, 1.0, 2.0 ** -8, want_t=True)
        metis.quantize(a.cuda(), None, sp.Rt)
        ops.append(sp)
    g, x = (oq.dequantize(*fp4_to_oracle(sp.Rt)) for sp in ops)
    ref = g @ x.T
    bound = elementwise_bound((g, None, None, None), (x, None, None, None), ref, out_dtype)
    wsb = torch.empty((max(metis.linear_workspace_bytes(L, N, K, 0), 256),), dtype=torch.uint8, device="cuda")
    flat, dW = _guarded(N, K, K + pad, out_dtype)
    metis.fp4_linear_wgrad(ops[0], ops[1], dW, wsb)
    _check_guarded(flat, dW, ref, bound)


@pytest.mark.parametrize("L,N,K,kx,kw", [(16, 400, 1040, 0, 32), (1, 48, 272, 0, 3), (64, 1040, 2064, 0, 65), (33, 16, 128, 0, 8),      # few rows
                                         (128, 272, 1040, 0, 16), (48, 528, 1040, 16, 24), (1040, 1072, 1264, 16, 24)])   # general path
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
def test_apply_does_not_read_the_factors(metis, L, N, K, kx, kw, out_dtype):  # noqa: F811
    """What depends on the factors is in the workspace after PREPARE: a program may quantize new ones into their place before APPLY."""
    if kw + 4 > min(N, K):
        kw = min(N, K) - 4
    xs, ws, _, _ = _product(metis, L, N, K, kx, kw, out_dtype, seed=17)
    wsb = torch.full((max(metis.linear_workspace_bytes(L, N, K, max(kx, kw)), 256),), 0xA5, dtype=torch.uint8, device="cuda")
    Y = torch.empty((L, N), dtype=out_dtype, device="cuda")
    metis.fp4_linear_fwd(xs, ws, Y, wsb)
    wsb.fill_(0x5A)
    metis.fp4_linear_phase(metis.LINEAR_FWD, metis.LINEAR_PREPARE, xs, ws, None, wsb)
    for sp in (xs, ws):
        if sp.k:
            sp.S.fill_(float("nan"))
            for t in (sp.Ut.codes, sp.Vt.codes, sp.Ut.scales, sp.Vt.scales):
                t.fill_(0x33)
    Z = torch.full((L, N), float("nan"), dtype=out_dtype, device="cuda")
    metis.fp4_linear_phase(metis.LINEAR_FWD, metis.LINEAR_APPLY, xs, ws, Z, wsb)
    assert torch.equal(Z, Y)


# both sides of the lines at which few rows leave their own kernels for the general ones: 16 rows, then the output's elements, in
# steps of 2^16, by rank, contraction (6, 12, 16 stages) and rows (32); without factors 6 stages; contractions for which a lone launch
# stays whole
@pytest.mark.parametrize("L,N,K,k", [
    (16, 32784, 912, 0), (17, 30832, 912, 0), (17, 30848, 912, 0), (33, 15872, 912, 0), (33, 15888, 912, 0), (17, 30848, 2064, 0),
    (48, 272, 768, 0), (48, 272, 784, 0), (32, 24576, 144, 8), (32, 24592, 144, 8), (32, 24592, 656, 8), (64, 12288, 144, 64),
    (64, 12304, 144, 64), (64, 15360, 1424, 8), (64, 15376, 1424, 8), (64, 8192, 144, 65), (64, 8208, 144, 65), (31, 16912, 144, 72),
    (31, 16928, 144, 72), (31, 16928, 656, 72), (80, 272, 1040, 0), (64, 272, 1024, 0), (64, 272, 1280, 0)])
def test_lines_between_the_paths(metis, L, N, K, k):  # noqa: F811
    xs, ws, ref, bound = _product(metis, L, N, K, 0, k, torch.float32, seed=21)
    wsb = torch.empty((max(metis.linear_workspace_bytes(L, N, K, k), 256),), dtype=torch.uint8, device="cuda")
    flat, Y = _guarded(L, N, N, torch.float32)
    metis.fp4_linear_fwd(xs, ws, Y, wsb)
    _check_guarded(flat, Y, ref, bound)
