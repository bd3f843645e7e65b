"""Inverted triangular blocks by substitution: columns whose sizes span the range of the
type come through the solves as they do through a substitution, and a product with an
inverted block leaves the residual of a column-by-column substitution (NumPy, the same
precision), not the larger one of an inverse that is put together from halves."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")
U = 2.0 ** -53


def crand(rng, *shape):
    return rng.normal(size=shape) + 1j * rng.normal(size=shape)


def lu_solve(F, piv, R, trans=0):
    X = torch.from_numpy(np.ascontiguousarray(R)).to(DEV)
    fm.zgetrs_batched(F, piv, X, trans=trans)
    return X.cpu().numpy()


@pytest.mark.parametrize("n", [9, 17, 33, 64, 130, 200])
@pytest.mark.parametrize("decades", [(160, -160), (-155, 155)])
@pytest.mark.parametrize("trans", [0, 2])
def test_columns_of_very_different_size(n, decades, trans):
    """Partial pivoting does not see the columns' scale D (powers of two): the solution of
    (A D) x = r is D^-1 times that of A x = r, with the error 8 n u cond(A) of the latter;
    the adjoint system (A D)^* x = D r has the solution of A^* x = r."""
    rng = np.random.default_rng(n)
    A, R = crand(rng, 2, n, n), crand(rng, 2, n, 5)
    d = 2.0 ** np.round(np.linspace(*decades, n) / np.log10(2.0))
    F = torch.from_numpy(A * d).to(DEV)
    piv, info = fm.zgetrf_batched(F)
    assert int(info.abs().sum()) == 0
    X = lu_solve(F, piv, R if trans == 0 else R * d[:, None], trans)
    if trans == 0:
        X = X * d[:, None]
    for a, x, r in zip(A, X, R):
        want = np.linalg.solve(a if trans == 0 else a.conj().T, r)
        err = np.linalg.norm(x - want) / np.linalg.norm(want)
        assert err < 8 * n * U * np.linalg.cond(a), err


def triangle(seed, which):
    """64 rows of a factor that partial pivoting leaves: the first ones of L, and of U
    those of the second panel."""
    rng = np.random.default_rng(seed)
    a = crand(rng, 200, 200)
    for k in range(128):
        p = k + np.argmax(np.abs(a[k:, k].real) + np.abs(a[k:, k].imag))
        a[[k, p]] = a[[p, k]]
        a[k + 1:, k] /= a[k, k]
        a[k + 1:, k + 1:] -= np.outer(a[k + 1:, k], a[k, k + 1:])
    if which == "L":
        return np.tril(a[:64, :64], -1) + np.eye(64)
    return np.triu(a[64:128, 64:128])


def substitution_inverse(T, which):
    X = np.eye(64, dtype=T.dtype)
    order = range(64) if which == "L" else range(63, -1, -1)
    for i in order:
        X[i] /= T[i, i]
        rest = slice(i + 1, 64) if which == "L" else slice(0, i)
        X[rest] -= np.outer(T[rest, i], X[i])
    return X


@pytest.mark.parametrize("which", ["L", "U"])
def test_residual_of_a_product_with_an_inverted_block(which):
    """Geometric mean of ||T x - b|| over 24 factors, as a multiple of what a substitution
    inverse leaves.  In a NumPy model the inverse by halves leaves 2.3 (L) and 2.0 (U)
    times as much: the line is drawn at the square root of 2."""
    ratio = []
    for seed in range(24):
        T = triangle(seed, which)
        b = crand(np.random.default_rng(1000 + seed), 64, 40)
        F = T if which == "U" else np.tril(T, -1) + np.eye(64)  # (the other factor is I)
        x = lu_solve(torch.from_numpy(F[None].astype(complex)).to(DEV),
                     torch.arange(64, dtype=torch.int32, device=DEV)[None].contiguous(), b[None])[0]
        y = substitution_inverse(T, which) @ b
        res = [np.linalg.norm((T.astype(np.clongdouble) @ v - b).astype(complex)) for v in (x, y)]
        ratio.append(res[0] / res[1])
    assert np.exp(np.mean(np.log(ratio))) < np.sqrt(2.0), np.exp(np.mean(np.log(ratio)))


def panel_join_ratio(seed, n=128):
    """||L11 U12 - (P A)12|| of a factorisation's join of its first two 64-column halves,
    over what a substitution in NumPy leaves for the same L11 and right-hand sides."""
    A = crand(np.random.default_rng(seed), 1, n, n)
    F = torch.from_numpy(A.copy()).to(DEV)
    piv, _ = fm.zgetrf_batched(F)
    f, p, r = F.cpu().numpy()[0], piv.cpu().numpy()[0], np.arange(n)
    for k in range(n):
        r[[k, p[k]]] = r[[p[k], k]]
    L, b, x = np.tril(f[:64, :64], -1) + np.eye(64), A[0][r][:64, 64:], f[:64, 64:]
    y = b.copy()
    for i in range(64):
        y[i + 1:] -= np.outer(L[i + 1:, i], y[i])
    res = [np.linalg.norm((L.astype(np.clongdouble) @ v - b).astype(complex)) for v in (x, y)]
    return res[0] / res[1]


def test_residual_of_the_panel_join():
    """In a NumPy model products with inverted 16-row diagonal blocks leave 1.67 times the
    residual of a substitution: the line is drawn at the square root of that."""
    r = np.exp(np.mean([np.log(panel_join_ratio(s)) for s in range(24)]))
    assert r < np.sqrt(1.67), r
