"""The 128 x 128 two-orientation quantizer and the draw-by-draw short cut of stochastic rounding, bit-exact against the
oracle: sizes around the tile and its 256-tile threshold, and inputs (zeros, ties, saturated, huge and tiny blocks,
non-finite values) on both sides of the short cut's conditions."""
import numpy as np
import pytest
import torch

from oracle import quant as oq

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def metis():
    from paper_2509_00404_amd import metis as m
    assert torch.cuda.is_available()
    m.lib()
    return m


def _compare(got, ref):
    c, s = ref
    assert np.array_equal(got.scales.cpu().numpy(), s)
    assert np.array_equal(got.codes.cpu().numpy(), c)


# 16 x 16 tiles at (2048, 2048); one tile row or column partly filled; one row of tiles; padded rows (ld > N)
@pytest.mark.parametrize("M,N,pad", [(2048, 2048, 0), (1936, 2064, 0), (16, 32768, 0), (32768, 16, 8), (1952, 2160, 24)])
@pytest.mark.parametrize("sr", [False, True])
@pytest.mark.parametrize("rows", [False, True])
def test_both_orientations(metis, M, N, pad, sr, rows):
    g0 = torch.Generator(device="cuda").manual_seed(M + N)
    x = torch.randn((M, N + pad), device="cuda", generator=g0)
    x *= torch.exp(torch.empty((M, 1), device="cuda").uniform_(-6, 6, generator=g0))
    x = x.to(torch.bfloat16)[:, :N]
    g = oq.tensor_scale_for(float(x.abs().max()))
    out, out_t = metis.Fp4Tensor(M, N, g) if rows else None, metis.Fp4Tensor(N, M, g)
    if sr:
        metis.quantize_sr(x, 91, out, out_t)
    else:
        metis.quantize(x, out, out_t)
    torch.cuda.synchronize()
    xn = x.double().cpu().numpy()
    xt = np.ascontiguousarray(xn.T)
    _compare(out_t, oq.quantize_sr(xt, g, 91, oq.STREAM_SR_T) if sr else oq.quantize(xt, g))
    if rows:
        _compare(out, oq.quantize_sr(xn, g, 91, oq.STREAM_SR) if sr else oq.quantize(xn, g))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("scale,g", [(1.0, 2.0 ** -8), (1.0, 2.0 ** -14), (2.0 ** 104, 2.0 ** 96), (2.0 ** -100, 2.0 ** -108),
                                     (2.0 ** -60, 2.0 ** 40)])
def test_stochastic_short_cut(metis, dtype, scale, g):
    # grid values, midpoints and values a few ulp from both times every power of two of a block's range, zero blocks,
    # and random blocks: 4M draws, of which ~30 fall in the window that takes the exact path
    rs = np.random.default_rng(7)
    M, N = 2048, 2048
    x = rs.standard_normal((M, N)) * np.exp(rs.uniform(-8, 2, (M, 1)))
    grid = np.array([0, .25, .5, .75, 1, 1.25, 1.5, 1.75, 2, 2.5, 3, 3.5, 4, 5, 6, 7])
    x[:256] = rs.choice(grid, (256, N)) * rs.choice([-1.0, 1.0], (256, N)) * 2.0 ** rs.integers(-6, 3, (256, 1))
    x[256:512] = x[:256] * (1.0 + rs.integers(-3, 4, (256, N)) * 2.0 ** (-8 if dtype == torch.bfloat16 else -23))
    x[512:520] = 0.0
    t = torch.from_numpy(x * scale).to(dtype)
    out = metis.Fp4Tensor(M, N, g)
    metis.quantize_sr(t.cuda(), 5, out)
    torch.cuda.synchronize()
    _compare(out, oq.quantize_sr(t.double().numpy(), g, 5, oq.STREAM_SR))


# fp32 takes the generic tiles, bf16 the row kernel, bf16 in both orientations the 128 x 128 tiles
@pytest.mark.parametrize("special", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("dtype,M,N,both", [(torch.float32, 64, 256, False), (torch.float32, 64, 256, True),
                                            (torch.bfloat16, 64, 256, False), (torch.bfloat16, 64, 256, True),
                                            (torch.bfloat16, 2048, 2048, True)])
def test_non_finite_values_take_the_exact_path(metis, special, dtype, M, N, both):
    """A non-finite element gets a saturated code and leaves every other block alone, codes and scales, in both orientations."""
    x = torch.randn((M, N), generator=torch.Generator().manual_seed(N)).to(dtype)
    x[3, 37] = float(special)
    clean = torch.nan_to_num(x, nan=0.0, posinf=0.0, neginf=0.0)
    outs = []
    for t in (clean, x):
        o, ot = metis.Fp4Tensor(M, N, 2.0 ** -9), metis.Fp4Tensor(N, M, 2.0 ** -9) if both else None
        metis.quantize_sr(t.cuda(), 11, o, ot)
        outs.append((o, ot))
    torch.cuda.synchronize()
    for ref, got, (r, c) in zip(*outs, ((3, 37), (37, 3))):
        if got is None:
            continue
        codes, scales = got.codes.cpu().numpy(), got.scales.cpu().numpy()
        assert (codes[r, c // 2] >> (4 * (c % 2))) & 7 == 7                   # magnitude 6
        block = c // 16
        codes[r, 8 * block:8 * block + 8] = ref.codes.cpu().numpy()[r, 8 * block:8 * block + 8]
        scales[r, block] = ref.scales.cpu().numpy()[r, block]
        assert np.array_equal(codes, ref.codes.cpu().numpy())
        assert np.array_equal(scales, ref.scales.cpu().numpy())


# thin matrices on both sides of the lines between the two tile kernels: 48 and 80 rows, 32 columns
@pytest.mark.parametrize("M,N", [(32, 32768), (48, 32768), (64, 32768), (80, 32768), (32768, 16), (32768, 32)])
@pytest.mark.parametrize("sr", [False, True])
@pytest.mark.parametrize("rows", [False, True])
def test_thin_matrices(metis, M, N, sr, rows):
    x = torch.randn((M, N), generator=torch.Generator().manual_seed(M + 3 * N)).to(torch.bfloat16)
    g = oq.tensor_scale_for(float(x.abs().max()))
    out, out_t = metis.Fp4Tensor(M, N, g) if rows else None, metis.Fp4Tensor(N, M, g)
    if sr:
        metis.quantize_sr(x.cuda(), 17, out, out_t)
    else:
        metis.quantize(x.cuda(), out, out_t)
    torch.cuda.synchronize()
    xn = x.double().numpy()
    xt = np.ascontiguousarray(xn.T)
    _compare(out_t, oq.quantize_sr(xt, g, 17, oq.STREAM_SR_T) if sr else oq.quantize(xt, g))
    if rows:
        _compare(out, oq.quantize_sr(xn, g, 17, oq.STREAM_SR) if sr else oq.quantize(xn, g))
