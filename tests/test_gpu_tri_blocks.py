"""The 64 x 64 triangular blocks (inverses by halves, Cholesky 16 columns at a
time) at the orders where their 8-, 16-, 32- and 64-row pieces begin and end."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")
U = 2.0 ** -53


def crand(rng, *shape):
    return rng.normal(size=shape) + 1j * rng.normal(size=shape)


@pytest.mark.parametrize("n", [2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 48, 49, 63, 65, 127, 128, 129])
@pytest.mark.parametrize("trans", [0, 2])
def test_solves_through_the_inverted_blocks(n, trans):
    rng = np.random.default_rng(n)
    M, R = crand(rng, 2, n, n), crand(rng, 2, n, 5)
    tM, tX = torch.from_numpy(M.copy()).to(DEV), torch.from_numpy(R.copy()).to(DEV)
    piv, info = fm.zgetrf_batched(tM)
    fm.zgetrs_batched(tM, piv, tX, trans=trans)
    X = tX.cpu().numpy()
    for b in range(2):
        Mb = M[b] if trans == 0 else M[b].conj().T
        be = np.linalg.norm(Mb @ X[b] - R[b]) / (np.linalg.norm(Mb) * np.linalg.norm(X[b]) +
                                                 np.linalg.norm(R[b]))
        assert be < 1e-15 * n + 1e-15, be


@pytest.mark.parametrize("m", [1, 2, 8, 15, 16, 17, 31, 33, 48, 49, 63, 64, 65, 81, 128, 129])
def test_orthonormalisation_at_the_block_edges(m):
    rng = np.random.default_rng(m)
    n = 300
    A, B = crand(rng, n, n), np.eye(n) + 0.05 * crand(rng, n, n) / np.sqrt(n)
    V = (crand(rng, n, m) * np.logspace(0, -4, m)) @ crand(rng, m, m)
    tA, tB, tV = (torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in (A, B, V))
    with fm.Plan(n, m, 0.0, 1.0, 1) as plan:
        Q, AQ, BQ, At, Bt = plan.project(tA, tB, tV.clone())
    Q, BQ = Q.cpu().numpy(), BQ.cpu().numpy()
    # Cholesky QR leaves ||Q^* Q - I|| of the order of the Gram product's rounding
    assert np.linalg.norm(Q.conj().T @ Q - np.eye(m)) < 5 * np.sqrt(n) * m * U
    assert np.linalg.norm(V - Q @ (Q.conj().T @ V)) < 5 * np.sqrt(n) * m * U * np.linalg.norm(V)
    # B~ = R_2 of B U_1 = U_2 R_2: upper triangular with a positive diagonal
    low = np.tril(Bt, -1)
    assert np.linalg.norm(low) < 5 * np.sqrt(n) * m * U * np.linalg.norm(Bt)
    assert np.all(np.diag(Bt).real > 0)
    assert np.allclose(Bt.conj().T @ Bt, BQ.conj().T @ BQ, rtol=0, atol=1e-12 * m)


@pytest.mark.parametrize("n,nrhs", [(64, 3), (65, 17), (300, 20), (520, 130)])
@pytest.mark.parametrize("trans", [0, 2])
@pytest.mark.parametrize("noalloc", [False, True])
def test_solves_between_padded_blocks(n, nrhs, trans, noalloc):
    # the right-hand sides' own rows serve as the solves' second block: nothing
    # beside them (columns past nrhs, rows past n) may be read or written
    rng = np.random.default_rng(n + nrhs)
    M, R = crand(rng, 2, n, n), crand(rng, 2, n, nrhs)
    tM = torch.from_numpy(M.copy()).to(DEV)
    piv, info = fm.zgetrf_batched(tM)
    box = torch.full((2, n + 2, nrhs + 3), complex(np.nan, np.nan), dtype=torch.complex128, device=DEV)
    tX = box[:, :n, :nrhs]
    tX.copy_(torch.from_numpy(R).to(DEV))
    (fm.zgetrs_batched_noalloc if noalloc else fm.zgetrs_batched)(tM, piv, tX, trans=trans)
    out = box.cpu().numpy()
    assert np.all(np.isnan(out[:, n:].real)) and np.all(np.isnan(out[:, :, nrhs:].real))
    for b in range(2):
        X = out[b, :n, :nrhs]
        Mb = M[b] if trans == 0 else M[b].conj().T
        be = np.linalg.norm(Mb @ X - R[b]) / (np.linalg.norm(Mb) * np.linalg.norm(X) +
                                              np.linalg.norm(R[b]))
        assert be < 1e-15 * n + 1e-15, be
