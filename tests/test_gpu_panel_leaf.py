"""The panel leaves of the LU at the edges of their row classes and with awkward
pivots: ties, columns of zeros, magnitudes whose squares over- or underflow."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")


def factor(M):
    tM = torch.from_numpy(M.copy()).to(DEV)
    piv, info = fm.zgetrf_batched(tM)
    return tM.cpu().numpy(), piv.cpu().numpy(), info.cpu().numpy()


def backward_error(M, F, piv):
    n = M.shape[0]
    P = M.copy()
    for i, p in enumerate(piv):
        P[[i, p]] = P[[p, i]]
    return np.linalg.norm(P - (np.tril(F, -1) + np.eye(n)) @ np.triu(F)) / np.linalg.norm(M)


@pytest.mark.parametrize("n", [8, 9, 255, 256, 257, 512, 513, 1024, 1025, 2049])
@pytest.mark.parametrize("scale", [1.0, 1e200, 1e-200])
def test_factors_at_the_row_class_edges(n, scale):
    rng = np.random.default_rng(n)
    M = (rng.normal(size=(1, n, n)) + 1j * rng.normal(size=(1, n, n))) * scale
    F, piv, info = factor(M)
    assert info[0] == 0
    assert backward_error(M[0] / scale, np.where(np.tri(n, k=-1) > 0, F[0], F[0] / scale),
                          piv[0]) < 1e-14 * n


@pytest.mark.parametrize("n", [70, 600, 1500])
def test_equal_pivots_take_the_lowest_row(n):
    # |re| + |im| = 4 in several rows of column 0, in one wavefront, in several,
    # and in several rows of one thread; the lowest of them is the pivot
    rng = np.random.default_rng(n)
    M = 0.1 * (rng.normal(size=(3, n, n)) + 1j * rng.normal(size=(3, n, n)))
    rows = [[5, 9, 63], [64, 1, n - 1], [n // 2, n - 2, n - 1, 40]]
    vals = [3 - 1j, -2 + 2j, 4j, -4]
    for b, rr in enumerate(rows):
        for r, v in zip(rr, vals):
            M[b, r, 0] = v
    F, piv, info = factor(M)
    assert np.all(info == 0)
    assert [int(p[0]) for p in piv] == [min(rr) for rr in rows]
    assert all(backward_error(M[b], F[b], piv[b]) < 1e-14 * n for b in range(3))


def test_zero_columns_are_reported_and_leave_the_rest_finite():
    n = 300
    rng = np.random.default_rng(3)
    M = rng.normal(size=(2, n, n)) + 1j * rng.normal(size=(2, n, n))
    M[0, :, 0] = 0.0
    M[1, :, 130] = 0.0
    F, piv, info = factor(M)
    assert list(info) == [1, 131]
    assert np.all(np.isfinite(F)) and int(piv[0, 0]) == 0


@pytest.mark.parametrize("n,nb", [(40, 0), (129, 0), (300, 64), (700, 0)])
@pytest.mark.parametrize("kind", ["none", "reverse", "cycle", "pairs"])
def test_exchanges_follow_a_planted_permutation(n, nb, kind):
    # rows of a diagonally dominant matrix in a known order: the pivots restore
    # it, whether a panel has no exchange, one chain through all rows, or many
    rng = np.random.default_rng(n)
    D = 0.01 * (rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))) / np.sqrt(n) + np.eye(n)
    order = {"none": np.arange(n), "reverse": np.arange(n)[::-1],
             "cycle": np.roll(np.arange(n), 1), "pairs": np.arange(n) ^ 1}[kind].copy()
    if kind == "pairs" and n % 2:
        order[-1] = n - 1
    M = D[order]
    tM = torch.from_numpy(M[None].copy()).to(DEV)
    piv, info = fm.zgetrf_batched(tM, nb=nb)
    F, piv = tM.cpu().numpy()[0], piv.cpu().numpy()[0]
    rows = order.copy()
    for i, p in enumerate(piv):
        rows[[i, p]] = rows[[p, i]]
    assert int(info[0]) == 0 and np.array_equal(rows, np.arange(n))
    assert backward_error(M, F, piv) < 1e-14 * n
