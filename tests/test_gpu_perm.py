"""Solves with given factors: row exchanges composed 64 at a time (positions met by
several exchanges of a group, exchanges across groups and across the 1024 that one round
takes, the last partial group), both triangles' inverted blocks from one launch, whole
and partial, and copies of all matrices at once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 200, 1023, 1024, 1025, 2100])
@pytest.mark.parametrize("kind", ["any", "near", "last", "none"])
def test_row_exchanges(n, kind):
    # with L = U = 1 a solve is the exchanges alone: exact
    rng = np.random.default_rng(n)
    i = np.arange(n)
    piv = {"any": rng.integers(i, n), "near": np.minimum(i + rng.integers(0, 4, n), n - 1),
           "last": np.full(n, n - 1), "none": i}[kind].astype(np.int32)
    perm = i.copy()
    for k in range(n):
        perm[[k, piv[k]]] = perm[[piv[k], k]]
    LU = torch.eye(n, dtype=torch.complex128, device=DEV)[None].contiguous()
    dp = torch.from_numpy(piv[None]).to(DEV)
    X = (rng.normal(size=(n, 3)) + 1j * rng.normal(size=(n, 3)))[None]
    for trans, want in ((0, X[0][perm]), (2, X[0][np.argsort(perm)])):
        t = torch.from_numpy(X).to(DEV)
        fm.zgetrs_batched(LU, dp, t, trans=trans)
        assert np.array_equal(t.cpu().numpy()[0], want)


@pytest.mark.parametrize("n,nrhs,batch", [(17, 1, 5), (64, 16, 2), (65, 15, 2), (128, 5, 3),
                                          (129, 33, 2), (193, 17, 2), (256, 16, 2), (257, 8, 2),
                                          (320, 40, 3), (513, 7, 2)])
@pytest.mark.parametrize("trans", [0, 2])
def test_solves(n, nrhs, batch, trans):
    rng = np.random.default_rng(n)
    M = (rng.normal(size=(batch, n, n)) + 1j * rng.normal(size=(batch, n, n))) / np.sqrt(n)
    M += 2.0 * np.eye(n)[None]
    R = rng.normal(size=(batch, n, nrhs)) + 1j * rng.normal(size=(batch, n, nrhs))
    LU, ld = torch.from_numpy(M).to(DEV), nrhs + 2
    piv, _ = fm.zgetrf_batched(LU)
    out = []
    for solve in (fm.zgetrs_batched, fm.zgetrs_batched_noalloc):
        X = torch.zeros((batch, n, ld), dtype=torch.complex128, device=DEV)
        X[:, :, :nrhs] = torch.from_numpy(R).to(DEV)
        solve(LU, piv, X[:, :, :nrhs], trans=trans)
        torch.cuda.synchronize()
        out.append(X.cpu().numpy())
    assert np.array_equal(out[0], out[1])
    assert not out[0][:, :, nrhs:].any()
    op = M if trans == 0 else np.conj(np.transpose(M, (0, 2, 1)))
    for a, x, r in zip(op, out[0][:, :, :nrhs], R):
        assert np.linalg.norm(a @ x - r) <= 8 * n * 2.0 ** -53 * (np.linalg.norm(a) *
                                                                  np.linalg.norm(x))
