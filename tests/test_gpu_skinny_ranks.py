"""The fp64 sketch and projection kernels at every width of their strips: whole tiles of 16 columns and partial ones, operands read
ahead (2 to 6 tiles) and not, contractions in one part, in several and in more than 64, through the factor gradients (2^-24 of
the sums: the bar of tests/test_gpu_factor_grads.py)."""
import pytest
import torch

from gpu_helpers import rel_fro, split_to_oracle
from oracle import linear as olin
from test_gpu_factor_grads import FG_RTOL, _run, metis  # noqa: F401  (metis is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,k", [(272, 320, 16), (1040, 368, 24), (320, 2064, 80), (336, 304, 88), (400, 528, 112), (1552, 176, 128),
                                   (528, 656, 8), (1040, 400, 32), (336, 784, 48), (656, 1040, 64), (64, 14336, 80), (8208, 96, 72)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_strip_widths(metis, N, K, k, dtype):  # noqa: F811
    g = torch.Generator().manual_seed(k)
    ws = metis.SplitTensor(N, K, k, 2.0 ** -4, 2.0 ** -4, 2.0 ** -8, want_t=False)
    for t, rows, cols in ((ws.Ut, k, N), (ws.Vt, k, K), (ws.R, N, K)):
        metis.quantize((0.05 * torch.randn((rows, cols), generator=g)).bfloat16().cuda(), t)
    ws.S.copy_(torch.rand((k,), generator=g).cuda() + 0.5)
    dW = torch.randn((N, K), generator=g).to(dtype).cuda()
    got = _run(metis, dW, ws)
    ref = olin.factor_grads(dW.double().cpu().numpy(), split_to_oracle(ws))
    for name, a, b in zip(("dU", "dS", "dV"), got, ref):
        assert rel_fro(a, b) < FG_RTOL, (name, rel_fro(a, b))
