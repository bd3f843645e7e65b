"""Band factorisation from both ends: pencils A = P D Q, B = P Q with banded P, Q
(known eigenvalues and eigenvectors) at the orders where the split begins, with
unequal, one-sided and no bandwidths, and singular pencils whose zero row lies in
either side or between them."""
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
    d = r * np.exp(2j * np.pi * rng.random(n))
    d = d[rng.permutation(n)]
    i, j = np.indices((n, n))
    keep = (i - j <= kl) & (j - i <= ku)
    V = rng.normal(size=(n, 12)) + 1j * rng.normal(size=(n, 12))
    return (P * d) @ Q, P @ Q, Q, d, keep, V


def edges(kl, ku):
    s = 4 * (kl + ku) + 64
    return [s - 1, s, s + 1, s + 34, s + 131]


@pytest.mark.parametrize("kl,ku", [(0, 0), (1, 0), (0, 3), (2, 5), (16, 7), (11, 24), (31, 32)])
@pytest.mark.parametrize("which", range(5))
def test_pairs_of_a_banded_pencil(kl, ku, which):
    n = edges(kl, ku)[which]
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
        res = A @ X[:, k] - r.lam[k] * (B @ X[:, k])
        assert np.linalg.norm(res) < 1e-8


@pytest.mark.parametrize("where", [2, 0.5, -3])
def test_a_zero_row_is_reported_wherever_it_lies(where):
    n, kl, ku = 200, 2, 3
    A, B, Q, d, keep, V = pencil(5, n, kl, ku)
    r = where if isinstance(where, int) else int(n * where)
    A[r], B[r] = 0.0, 0.0
    with fm.Plan(n, V.shape[1], 0.0, 1.0, 8) as plan:
        with pytest.raises(fm.FeastError) as e:
            plan.solve_csr(csr(A, keep), csr(B, keep), torch.from_numpy(V).to(DEV))
        assert e.value.code == fm.FEAST_SINGULAR
