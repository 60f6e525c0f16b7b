"""GPU parity of the MXFP4 variant: quantizer codes and scales bit-exact against the oracle, and the
block-scaled matrix-instruction GEMM against the oracle's fp64 product of the same quantized operands
(every product is exact and only the fp32 accumulation rounds: 1e-5 relative Frobenius)."""
import numpy as np
import pytest
import torch

from oracle import mx as omx
from gpu_helpers import rel_fro

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def metis():
    from paper_2509_00404_amd import metis as m
    assert torch.cuda.is_available()
    m.lib()
    return m


def _data(M, K, seed, dtype):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((M, K), generator=g) * torch.exp(1.5 * torch.randn((M, 1), generator=g))
    x[0, :8] = torch.tensor([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0, 7.0])      # grid midpoints and a saturating value
    x[0, 8:32] = 0.0
    x[0, 9] = 7.5
    if M > 2:
        x[1, 32:64] = 0.0                                                      # an all-zero block with a negative zero
        x[1, 40] = -0.0
        x[2, :32] = 2.0 ** -130                                               # below the fp32 normal range
    return x.to(dtype)


@pytest.mark.parametrize("M,K", [(128, 256), (77, 96), (1, 32), (513, 4096)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_quantize_mx_bit_exact(metis, M, K, dtype):
    x = _data(M, K, M + K, dtype)
    out = metis.MxTensor(M, K)
    metis.quantize_mx(x.cuda(), out)
    torch.cuda.synchronize()
    c, s = omx.quantize_mx(x.double().numpy())
    assert np.array_equal(out.scales.cpu().numpy(), s)
    assert np.array_equal(out.codes.cpu().numpy(), c)


@pytest.mark.parametrize("M,N,K", [(256, 256, 256), (300, 200, 768), (1040, 528, 1024), (64, 1100, 512),
                                   # K not a multiple of the 256-deep stage: the tail variant (whole blocks of 32 only)
                                   (256, 256, 128), (300, 200, 384), (130, 70, 96), (520, 264, 1248)])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_mxfp4_gemm_against_oracle(metis, M, N, K, out_dtype):
    a, b = _data(M, K, 1, torch.bfloat16), _data(N, K, 2, torch.bfloat16)
    qa, qb = metis.MxTensor(M, K), metis.MxTensor(N, K)
    metis.quantize_mx(a.cuda(), qa)
    metis.quantize_mx(b.cuda(), qb)
    Cm = torch.full((M, N), float("nan"), dtype=out_dtype, device="cuda")
    metis.mxfp4_gemm_nt(qa, qb, Cm)
    torch.cuda.synchronize()
    ref = omx.mx_gemm_nt((qa.codes.cpu().numpy(), qa.scales.cpu().numpy()), (qb.codes.cpu().numpy(), qb.scales.cpu().numpy()))
    got = Cm.double().cpu().numpy()
    assert np.isfinite(got).all()
    assert rel_fro(got, ref) < (1e-5 if out_dtype == torch.float32 else 4e-3)
    # and the quantized product approximates the unquantized one as FP4 does (~10 %)
    assert rel_fro(ref, a.double().numpy() @ b.double().numpy().T) < 0.25


def test_rejects_bad_arguments(metis):
    Cm = torch.empty((64, 64), dtype=torch.float32, device="cuda")
    qc = metis.MxTensor(64, 256)
    with pytest.raises(metis.MetisError):
        metis.mxfp4_gemm_nt(qc, metis.MxTensor(32, 512), Cm)
    with pytest.raises(metis.MetisError):
        metis.quantize_mx(torch.zeros((64, 64), dtype=torch.float32, device="cuda"), qc)


@pytest.mark.parametrize("M,N,K,ld_extra", [(257, 255, 256, 0), (255, 261, 288, 3), (33, 67, 96, 8), (512, 1283, 512, 1), (2305, 1288, 256, 0)])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_mxfp4_gemm_rows_that_do_not_store_in_vectors(metis, M, N, K, ld_extra, out_dtype):
    """Odd widths, rows of C that start off 16 bytes, last bands of 1 and 2 tile columns; nothing beside the rows is written.  The bars of
    test_mxfp4_gemm_against_oracle."""
    a, b = _data(M, K, 3, torch.bfloat16), _data(N, K, 4, torch.bfloat16)
    qa, qb = metis.MxTensor(M, K), metis.MxTensor(N, K)
    metis.quantize_mx(a.cuda(), qa)
    metis.quantize_mx(b.cuda(), qb)
    full = torch.full((M, N + ld_extra), float("nan"), dtype=out_dtype, device="cuda")
    metis.mxfp4_gemm_nt(qa, qb, full[:, :N])
    torch.cuda.synchronize()
    ref = omx.mx_gemm_nt((qa.codes.cpu().numpy(), qa.scales.cpu().numpy()), (qb.codes.cpu().numpy(), qb.scales.cpu().numpy()))
    got = full[:, :N].double().cpu().numpy()
    assert np.isfinite(got).all()
    assert rel_fro(got, ref) < (1e-5 if out_dtype == torch.float32 else 4e-3)
    assert bool(torch.isnan(full[:, N:]).all())


@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (3, 2, 64), (1, 7, 224), (1, 1, 288), (2, 257, 480), (3, 5, 544), (257, 3, 1024 + 32)])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_mxfp4_gemm_partial_last_stage(metis, M, N, K, out_dtype):
    """One partial stage and a partial stage after whole ones, 1 to 7 blocks of 32 in it, operands of a few rows: the scale bytes of the last
    row are fetched from before where they start.  The bars of test_mxfp4_gemm_against_oracle."""
    a, b = _data(M, K, 5, torch.bfloat16), _data(N, K, 6, torch.bfloat16)
    qa, qb = metis.MxTensor(M, K), metis.MxTensor(N, K)
    metis.quantize_mx(a.cuda(), qa)
    metis.quantize_mx(b.cuda(), qb)
    Cm = torch.full((M, N), float("nan"), dtype=out_dtype, device="cuda")
    metis.mxfp4_gemm_nt(qa, qb, Cm)
    torch.cuda.synchronize()
    ref = omx.mx_gemm_nt((qa.codes.cpu().numpy(), qa.scales.cpu().numpy()), (qb.codes.cpu().numpy(), qb.scales.cpu().numpy()))
    got = Cm.double().cpu().numpy()
    assert np.isfinite(got).all()
    # elementwise, for outputs of few elements: 2^-22 sqrt(K) of the sum of magnitudes (fp32 sums), and half a bf16 unit of the result
    mag = omx.mx_gemm_nt((qa.codes.cpu().numpy() & 0x77, qa.scales.cpu().numpy()), (qb.codes.cpu().numpy() & 0x77, qb.scales.cpu().numpy()))
    bound = (2.0 ** -22 * np.sqrt(K)) * mag + (2.0 ** -8 * np.abs(ref) if out_dtype == torch.bfloat16 else 0.0)
    assert (np.abs(got - ref) <= bound).all()


# 448 tiles of 128 x 128, 476 and more; a grid of 256 x 256 tiles that splits into near-square regions and ones that do not
@pytest.mark.parametrize("M,N", [(2048, 3584), (2176, 3584), (2049, 4090), (4100, 2433), (4090, 2048)])
@pytest.mark.parametrize("K", [256, 288, 96])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_mxfp4_gemm_on_both_sides_of_the_tile_rule(metis, M, N, K, out_dtype):
    """Outputs of up to 448 tiles of 128 x 128 and larger ones, each with whole, partial and short contractions.  The bars of
    test_mxfp4_gemm_against_oracle, for every 256 x 256 block of the output."""
    a, b = _data(M, K, 7, torch.bfloat16), _data(N, K, 8, torch.bfloat16)
    qa, qb = metis.MxTensor(M, K), metis.MxTensor(N, K)
    metis.quantize_mx(a.cuda(), qa)
    metis.quantize_mx(b.cuda(), qb)
    Cm = torch.full((M, N), float("nan"), dtype=out_dtype, device="cuda")
    metis.mxfp4_gemm_nt(qa, qb, Cm)
    torch.cuda.synchronize()
    ref = omx.mx_gemm_nt((qa.codes.cpu().numpy(), qa.scales.cpu().numpy()), (qb.codes.cpu().numpy(), qb.scales.cpu().numpy()))
    got = Cm.double().cpu().numpy()
    assert np.isfinite(got).all()
    for i in range(0, M, 256):
        for j in range(0, N, 256):
            assert rel_fro(got[i:i + 256, j:j + 256], ref[i:i + 256, j:j + 256]) < (1e-5 if out_dtype == torch.float32 else 4e-3), (i, j)


# 256 x 256 tiles of whole units of 256: two units, three, more; fewer tiles than CUs, more than one a CU, ragged last rows and columns
@pytest.mark.parametrize("M,N,K", [(3000, 3000, 2304), (2817, 6399, 768), (4200, 4399, 512), (4352, 4100, 768), (2600, 2900, 2048)])
@pytest.mark.parametrize("ld_extra", [0, 1])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_mxfp4_gemm_streamed(metis, M, N, K, ld_extra, out_dtype):
    """The bars of test_mxfp4_gemm_against_oracle for every 256 x 256 block; rows of C that start off 16 bytes, nothing written beside them."""
    a, b = _data(M, K, 9, torch.bfloat16), _data(N, K, 10, torch.bfloat16)
    qa, qb = metis.MxTensor(M, K), metis.MxTensor(N, K)
    metis.quantize_mx(a.cuda(), qa)
    metis.quantize_mx(b.cuda(), qb)
    full = torch.full((M, N + ld_extra), float("nan"), dtype=out_dtype, device="cuda")
    for _ in range(2):                     # the second launch finds other data in LDS
        metis.mxfp4_gemm_nt(qa, qb, full[:, :N])
    torch.cuda.synchronize()
    ref = omx.mx_gemm_nt((qa.codes.cpu().numpy(), qa.scales.cpu().numpy()), (qb.codes.cpu().numpy(), qb.scales.cpu().numpy()))
    got = full[:, :N].double().cpu().numpy()
    assert np.isfinite(got).all()
    for i in range(0, M, 256):
        for j in range(0, N, 256):
            assert rel_fro(got[i:i + 256, j:j + 256], ref[i:i + 256, j:j + 256]) < (1e-5 if out_dtype == torch.float32 else 4e-3), (i, j)
    assert bool(torch.isnan(full[:, N:]).all())


# three and more tiles a workgroup (256 of them), two units a tile, three and five: the staging buffers change hands several times, an odd
# number of units swaps them from tile to tile; the last one walks its tiles in bands (1536 tiles and more, a contraction beyond 1024)
@pytest.mark.parametrize("M,N,K", [(5900, 6100, 512), (5900, 6100, 768), (10200, 9800, 1280)])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_mxfp4_gemm_streamed_over_many_tiles(metis, M, N, K, out_dtype):
    """The bars of test_mxfp4_gemm_against_oracle for every 256 x 256 block, against the fp64 product of the oracle's dequantized operands."""
    a, b = _data(M, K, 11, torch.bfloat16), _data(N, K, 12, torch.bfloat16)
    qa, qb = metis.MxTensor(M, K), metis.MxTensor(N, K)
    metis.quantize_mx(a.cuda(), qa)
    metis.quantize_mx(b.cuda(), qb)
    C = torch.full((M, N), float("nan"), dtype=out_dtype, device="cuda")
    metis.mxfp4_gemm_nt(qa, qb, C)
    fa, fb = (torch.from_numpy(omx.dequantize_mx(q.codes.cpu().numpy(), q.scales.cpu().numpy())).cuda() for q in (qa, qb))
    ref = fa @ fb.T
    err = C.double() - ref
    tiles = lambda x: torch.nn.functional.pad(x, (0, -N % 256, 0, -M % 256)).unflatten(1, (-1, 256)).unflatten(0, (-1, 256)).pow(2).sum((1, 3))
    worst = (tiles(err) / tiles(ref)).sqrt().max()
    assert float(worst) < (1e-5 if out_dtype == torch.float32 else 4e-3)
