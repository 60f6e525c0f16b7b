"""GPU parity: gradients of the weight's low-rank factors (Sec. 3.2, backward formulas after
Eq. 3) against the oracle, both fed the SAME dW (the GPU wgrad's output) and the same
quantized factors.  The products accumulate in fp64 on both sides and the GPU rounds once to
fp32, so the bound is a few fp32 ulps of the result's scale."""
import numpy as np
import pytest
import torch

from oracle import linear as olin
from gpu_helpers import make_split, rel_fro, split_to_oracle

pytestmark = pytest.mark.gpu

FG_RTOL = 1e-6


@pytest.fixture(scope="module")
def metis():
    from paper_2509_00404_amd import metis as m
    assert torch.cuda.is_available()
    m.lib()
    return m


def _run(metis, dW, ws):
    N, K = dW.shape
    k = ws.k
    dU = torch.full((N, k), float("nan"), dtype=torch.float32, device="cuda")
    dS = torch.full((k, k), float("nan"), dtype=torch.float32, device="cuda")
    dV = torch.full((K, k), float("nan"), dtype=torch.float32, device="cuda")
    metis.fp4_factor_grads(dW, ws, dU, dS, dV)
    torch.cuda.synchronize()
    return [t.double().cpu().numpy() for t in (dU, dS, dV)]


@pytest.mark.parametrize("L,N,K,k", [(128, 256, 512, 8), (208, 144, 272, 5), (96, 80, 112, 12),
                                     (256, 1040, 1296, 64), (64, 2064, 48, 3)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_factor_grads_from_wgrad(metis, L, N, K, k, dtype):
    from paper_2509_00404_amd import workloads
    X = workloads.planted(L, K, workloads.power_law(min(L, K), 1.2), 1, rms=1.0, outlier_cols=1)
    W = workloads.planted(N, K, workloads.power_law(min(N, K), 1.0), 2, noise_top=0.01, rms=0.02)
    G = workloads.planted(L, N, workloads.power_law(min(L, N), 2.0, head=4, head_gain=100.0), 3, rms=1e-3)
    xs = make_split(metis, X, 0, 0, 1.0, 0)[0]
    gs = make_split(metis, G, 0, 0, 1.0, 0)[0]
    ws = make_split(metis, W, k, 8, 1.0, 12)[0]
    wsb = torch.empty((max(metis.linear_workspace_bytes(L, N, K, k), 256),), dtype=torch.uint8, device="cuda")
    dW = torch.empty((N, K), dtype=dtype, device="cuda")
    metis.fp4_linear_wgrad(gs, xs, dW, wsb)
    got = _run(metis, dW, ws)
    ref = olin.factor_grads(dW.double().cpu().numpy(), split_to_oracle(ws))
    for name, a, b in zip(("dU", "dS", "dV"), got, ref):
        assert a.shape == b.shape, name
        assert np.isfinite(a).all(), name
        assert rel_fro(a, b) < FG_RTOL, (name, rel_fro(a, b))
        assert np.abs(a - b).max() <= 4e-6 * np.abs(b).max(), name


def test_strided_dW_and_repeat(metis):
    """A dW that is a column slice of a wider buffer (ld > K); a second call overwrites, not accumulates."""
    from paper_2509_00404_amd import workloads
    N, K, k = 272, 320, 16
    W = workloads.planted(N, K, workloads.power_law(min(N, K), 1.0), 5, noise_top=0.01, rms=0.02)
    ws = make_split(metis, W, k, 8, 1.0, 3)[0]
    g = torch.Generator().manual_seed(7)
    wide = torch.randn((N, K + 64), generator=g, dtype=torch.float32).cuda()
    dW = wide[:, :K]
    ref = olin.factor_grads(dW.double().cpu().numpy(), split_to_oracle(ws))
    for _ in range(2):
        got = _run(metis, dW, ws)
        for a, b in zip(got, ref):
            assert rel_fro(a, b) < FG_RTOL


def test_rejects_bad_arguments(metis):
    from paper_2509_00404_amd import workloads
    N, K, k = 64, 96, 4
    W = workloads.planted(N, K, workloads.power_law(64, 1.0), 5, rms=0.02)
    ws = make_split(metis, W, k, 8, 1.0, 3)[0]
    dU = torch.empty((N, k), dtype=torch.float32, device="cuda")
    dS = torch.empty((k, k), dtype=torch.float32, device="cuda")
    dV = torch.empty((K, k), dtype=torch.float32, device="cuda")
    wrong = torch.zeros((N + 16, K), dtype=torch.float32, device="cuda")
    with pytest.raises(metis.MetisError):
        metis.fp4_factor_grads(wrong, ws, dU, dS, dV)
    small = torch.empty((16,), dtype=torch.uint8, device="cuda")
    with pytest.raises(metis.MetisError):
        metis.fp4_factor_grads(torch.zeros((N, K), dtype=torch.float32, device="cuda"), ws, dU, dS, dV, small)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_tensor_scales_that_round_in_16_bits(metis, dtype):
    """The entry point takes any positive tensor scale: one that is no power of two (the factors then need more bits than bf16
    has) gives the same precision."""
    from paper_2509_00404_amd import workloads
    N, K, k = 272, 320, 16
    W = workloads.planted(N, K, workloads.power_law(min(N, K), 1.0), 5, noise_top=0.01, rms=0.02)
    ws = make_split(metis, W, k, 8, 1.0, 3)[0]
    ws.Ut.tscale, ws.Vt.tscale = 2.0 ** -11 * 1.3125, float(np.float32(2.0 ** -11 * 1.7))
    dW = torch.randn((N, K), generator=torch.Generator().manual_seed(9)).to(dtype).cuda()
    got = _run(metis, dW, ws)
    for name, a, b in zip(("dU", "dS", "dV"), got, olin.factor_grads(dW.double().cpu().numpy(), split_to_oracle(ws))):
        assert rel_fro(a, b) < FG_RTOL, (name, rel_fro(a, b))
