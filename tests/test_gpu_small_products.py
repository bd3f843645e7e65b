"""Products whose output is too small for the 64 x 64 tiles (the split of K over
the wavefronts of a workgroup), against NumPy in FP64: edges of the 16-wide
tiles, of the 8-long K steps and of their split over 8 or 16 wavefronts, the
last tile count that takes this path and the first that does not, leading
dimensions above the row length, and in-place products."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")
U = 2.0 ** -53


def crand(rng, *shape):
    return rng.normal(size=shape) + 1j * rng.normal(size=shape)


def abs1(x):
    return np.abs(x.real) + np.abs(x.imag)


def bound(opA, B, alpha, beta, C):
    """Each real part of a K-term complex sum takes 2 K products and sums, whatever
    their order; alpha, beta and the final sum add four roundings more."""
    K = B.shape[-2]
    return (2 * K + 8) * U * (abs1(np.asarray(alpha)) * (abs1(opA) @ abs1(B)) +
                              abs1(np.asarray(beta)) * abs1(C)) + 1e-300


@pytest.mark.parametrize("M,N,K", [(1, 16, 1), (16, 1, 7), (15, 17, 8), (17, 15, 9), (31, 33, 63),
                                   (16, 16, 127), (33, 16, 129), (16, 48, 4001), (160, 157, 1025),
                                   (700, 250, 1030), (1024, 1024, 9), (1025, 1024, 9)])
@pytest.mark.parametrize("transA", [0, 2])
@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (-1.0, 1.0), (0.7 - 0.2j, -0.3 + 1.1j)])
def test_small_products_match_numpy(M, N, K, transA, alpha, beta):
    rng = np.random.default_rng(M * 131 + N * 17 + K)
    batch = 2 if M * N <= 160 * 160 else 1
    pad = 3  # leading dimension = row length + 3, filled with NaN
    rows, cols = (M, K) if transA == 0 else (K, M)
    hA, hB, hC = (np.full((batch, r, c + pad), np.nan + 0j) for r, c in ((rows, cols), (K, N), (M, N)))
    hA[:, :, :cols], hB[:, :, :N], hC[:, :, :N] = (crand(rng, batch, r, c) for r, c in
                                                   ((rows, cols), (K, N), (M, N)))
    tA, tB, tC = (torch.from_numpy(x).to(DEV) for x in (hA, hB, hC))
    fm.zgemm_batched(tA[:, :, :cols], tB[:, :, :N], tC[:, :, :N], alpha, beta, transA)
    out = tC.cpu().numpy()
    A, B, C = hA[:, :, :cols], hB[:, :, :N], hC[:, :, :N]
    opA = A if transA == 0 else np.conj(np.transpose(A, (0, 2, 1)))
    ref = alpha * (opA @ B) + beta * C
    # twice: NumPy's own product rounds as well
    assert np.all(np.abs(out[:, :, :N] - ref) <= 2 * bound(opA, B, alpha, beta, C))
    assert np.all(np.isnan(out[:, :, N:].real))  # nothing written past a row


@pytest.mark.parametrize("M", [5, 64])
def test_in_place_products_keep_one_workgroup_per_column_block(M):
    rng = np.random.default_rng(M)
    A, X = crand(rng, 2, M, M), crand(rng, 2, M, 200)
    tX = torch.from_numpy(X).to(DEV)
    fm.zgemm_batched(torch.from_numpy(A).to(DEV), tX, tX)
    assert np.all(np.abs(tX.cpu().numpy() - A @ X) <= 2 * bound(A, X, 1.0, 0.0, X))
