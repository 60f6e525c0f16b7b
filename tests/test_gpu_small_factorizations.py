"""The small factorizations at the orders where their tiles end: Cholesky panels of 16 columns (one below, at, and one
above a multiple), the eigenvector preconditioner's range of 72 to 84, its neighbours, and the largest orders; repeated and
vanishing singular values (the preconditioner's fallback).  Bars of tests/test_gpu_decompose.py."""
import numpy as np
import pytest
import torch

from oracle import decompose as odec
from test_gpu_decompose import _compare, _planted_bf16, _run, metis  # noqa: F401  (metis is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,p", [(1, 1), (8, 7), (16, 1), (17, 14), (31, 2), (48, 16), (49, 16), (63, 8), (64, 8), (65, 8),
                                 (64, 15), (65, 15), (65, 16), (76, 8), (77, 8), (72, 15), (80, 8), (81, 8), (90, 5), (95, 1)])
def test_orders_at_the_edges_of_tiles(metis, k, p):  # noqa: F811
    M, N = 512, 256
    s = 50.0 * np.arange(1, N + 1) ** -1.1 + 0.02
    A = _planted_bf16(M, N, s, seed=k + 7 * p)
    got = _run(metis, A, k, p, 0.5, seed=5)
    _compare(A, got, odec.decompose(A.double().numpy(), k, p, 0.5, seed=5), k)


@pytest.mark.parametrize("k,p", [(63, 8), (64, 8), (40, 33), (66, 13), (66, 14), (67, 14), (82, 2), (84, 1)])
@pytest.mark.parametrize("alpha", [1.1, 1.5])
def test_orders_of_the_eigenvector_preconditioner(metis, k, p, alpha):  # noqa: F811
    # its least and largest order (72, 84) and their neighbours, whole and ragged tiles, the spectra of the tests above
    s = 50.0 * np.arange(1, 257) ** -alpha + 0.02
    A = _planted_bf16(512, 256, s, seed=k + 5 * p)
    got = _run(metis, A, k, p, 1.0, seed=9)
    _compare(A, got, odec.decompose(A.double().numpy(), k, p, 1.0, seed=9), k)


@pytest.mark.parametrize("k,p", [(20, 12), (60, 20), (72, 16)])
def test_repeated_singular_values(metis, k, p):  # noqa: F811
    # pairs of equal singular values down to the last kept one: the subspaces are determined up to the pair, so compare
    # the singular values and the projector
    M, N = 512, 256
    s = 20.0 * 0.9 ** (np.arange(N) // 2)
    s[k + p - 2:] *= 0.01
    A = _planted_bf16(M, N, s, seed=3)
    U, S, V, _ = _run(metis, A, k, p, 1.0, seed=8)
    Ur, Sr, Vr = odec.decompose(A.double().numpy(), k, p, 1.0, seed=8)
    assert np.max(np.abs(S - Sr) / Sr) < 1e-3
    assert np.abs(V.T @ V - np.eye(k)).max() < 1e-4
    An = A.double().numpy()
    assert np.linalg.norm((U * S) @ V.T - (Ur * Sr) @ Vr.T) / np.linalg.norm(An) < 1e-3


@pytest.mark.parametrize("k,p", [(1, 1), (2, 2), (5, 4), (8, 8), (24, 8), (33, 8), (40, 24), (61, 10), (64, 8), (64, 16), (65, 16),
                                 (66, 18), (72, 16), (80, 16)])
def test_ill_conditioned_sketch(metis, k, p):  # noqa: F811
    # the kept directions within a factor of 16, the others 2^-18 of them: the first orthogonalisation leaves its basis orthonormal to
    # ~2^-52 2^36 only, and the second pass repairs it; orders that are multiples of 8, and the generic kernels' that are not
    g = torch.Generator().manual_seed(100 * k + p)
    A = torch.randn((512, 256), generator=g)
    A[:, :k] *= 2.0 ** -torch.div(4 * torch.arange(k), k, rounding_mode="floor")
    A[:, k:] *= 2.0 ** -18
    A = A.to(torch.bfloat16)
    got = _run(metis, A, k, p, 1.0, seed=9)
    _compare(A, got, odec.decompose(A.double().numpy(), k, p, 1.0, seed=9), k)


@pytest.mark.parametrize("k,p", [(1, 1), (1, 2), (2, 2), (3, 2)])
def test_orders_up_to_four(metis, k, p):  # noqa: F811
    # factored on one lane up to order 4
    A = _planted_bf16(512, 256, 50.0 * np.arange(1, 257) ** -1.5 + 0.02, seed=40 + k + p)
    got = _run(metis, A, k, p, 1.0, seed=5)
    _compare(A, got, odec.decompose(A.double().numpy(), k, p, 1.0, seed=5), k)
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    metis.decompose(torch.zeros((64, 64), dtype=torch.bfloat16, device="cuda"), k, p, 1.0, 1, info=info)
    assert int(info.item()) != 0
