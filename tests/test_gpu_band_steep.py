"""Band pencils with one side's window much wider than the other's (the two sides have
windows and shares of the rows of their own): known eigenpairs at the orders where the
split begins and beyond."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")


def banded(rng, n, lo, up, c):
    M = np.zeros((n, n), complex)
    for k in range(-lo, up + 1):
        d = n - abs(k)
        M += np.diag(c * (rng.normal(size=d) + 1j * rng.normal(size=d)) / np.sqrt(lo + up + 1), k)
    return M + np.eye(n)


def csr(M, keep):
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    i, j = np.nonzero(keep)
    return [torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
            for x in (rp, j.astype(np.int32), M[i, j].astype(np.complex128))]


def pencil(seed, n, kl, ku, s=6):
    rng = np.random.default_rng(seed)
    P, Q = banded(rng, n, kl, 0, 0.3), banded(rng, n, 0, ku, 0.3)
    r = np.concatenate([np.sqrt(rng.random(s)) * 0.8, np.sqrt(1.69 + rng.random(n - s) * 8)])
    d = (r * np.exp(2j * np.pi * rng.random(n)))[rng.permutation(n)]
    i, j = np.indices((n, n))
    keep = (i - j <= kl) & (j - i <= ku)
    V = rng.normal(size=(n, 12)) + 1j * rng.normal(size=(n, 12))
    return (P * d) @ Q, P @ Q, Q, d, keep, V


@pytest.mark.parametrize("kl,ku", [(0, 48), (15, 48), (0, 63), (1, 60), (48, 0), (48, 15),
                                   (63, 0), (60, 1), (0, 47), (47, 16)])
@pytest.mark.parametrize("more", [-1, 0, 1, 33, 190])
def test_pairs(kl, ku, more):
    n = 4 * (kl + ku) + 64 + more
    A, B, Q, d, keep, V = pencil(100 * kl + ku, n, kl, ku)
    with fm.Plan(n, V.shape[1], 0.0, 1.0, 16, max_iter=10) as plan:
        r = plan.solve_csr(csr(A, keep), csr(B, keep), torch.from_numpy(V).to(DEV))
    assert r.band == (kl, ku) and r.flag == 1
    inside = np.flatnonzero(np.abs(d) < 1.0)
    assert len(r.lam) == len(inside)
    X = r.X.cpu().numpy()
    Qi = np.linalg.inv(Q)
    for i in inside:
        k = int(np.argmin(np.abs(r.lam - d[i])))
        assert abs(r.lam[k] - d[i]) < 1e-10
        x = Qi[:, i] / np.linalg.norm(Qi[:, i])
        assert abs(abs(np.vdot(x, X[:, k])) - 1.0) < 1e-8
        assert np.linalg.norm(A @ X[:, k] - r.lam[k] * (B @ X[:, k])) < 1e-8
