"""The paths of the complex products by the sizes that select them now, against NumPy in
FP64.  Output tiles are 64 x 32; below a line (op = 1: 400 tiles, 512 for sums of 512 and
more, 832 from 1024 on; op = ^*: 512 tiles, 1024 for sums past 128) a product splits its sum
over a workgroup's wavefronts, from there on it takes the tiles."""
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


def product(M, N, K, batch, transA, alpha, beta):
    """Each real part of a K-term complex sum takes 2 K products and sums, whatever their
    order; alpha, beta and the final sum add four roundings more.  Twice that: NumPy's own
    product rounds as well."""
    rng = np.random.default_rng(M * 131 + N * 17 + K + batch)
    rows, cols = (M, K) if transA == 0 else (K, M)
    hA, hB, hC = (np.full((batch, r, c + 3), np.nan + 0j) for r, c in ((rows, cols), (K, N), (M, N)))
    A, B, C = hA[:, :, :cols], hB[:, :, :N], hC[:, :, :N]
    A[:], B[:], C[:] = crand(rng, *A.shape), crand(rng, *B.shape), crand(rng, *C.shape)
    tA, tB, tC = (torch.from_numpy(x).to(DEV) for x in (hA, hB, hC))
    fm.zgemm_batched(tA[:, :, :cols], tB[:, :, :N], tC[:, :, :N], alpha, beta, transA)
    out = tC.cpu().numpy()
    opA = A if transA == 0 else np.conj(np.transpose(A, (0, 2, 1)))
    lim = (2 * K + 8) * U * (abs1(np.asarray(alpha)) * (abs1(opA) @ abs1(B)) +
                             abs1(np.asarray(beta)) * abs1(C)) + 1e-300
    assert np.all(np.abs(out[:, :, :N] - (alpha * (opA @ B) + beta * C)) <= 2 * lim)
    assert np.all(np.isnan(out[:, :, N:].real))  # nothing written past a row


AB = [(1.0 + 0j, 0j), (-1.0 + 0j, 1.0 + 0j), (0.7 - 0.2j, -0.3 + 1.1j)]


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (63, 31, 7), (64, 32, 8), (65, 33, 3), (17, 5, 12)])
@pytest.mark.parametrize("transA", [0, 2])
@pytest.mark.parametrize("alpha,beta", AB)
def test_tiles_with_one_or_two_steps(M, N, K, transA, alpha, beta):
    product(M, N, K, 1030, transA, alpha, beta)  # past every line


@pytest.mark.parametrize("transA,K,line", [(0, 9, 400), (0, 511, 400), (0, 512, 512), (0, 1023, 512),
                                           (0, 1024, 832), (2, 128, 512), (2, 129, 1024)])
@pytest.mark.parametrize("below", [1, 0])
def test_both_sides_of_each_line(transA, K, line, below):
    product(3, 2, K, line - below, transA, 0.7 - 0.2j, -0.3 + 1.1j)


@pytest.mark.parametrize("M,N,K", [(1000, 300, 1030), (1000, 300, 1024), (1009, 289, 1500),
                                   (1000, 300, 100), (1000, 300, 64), (300, 300, 65)])
@pytest.mark.parametrize("transA", [0, 2])
@pytest.mark.parametrize("alpha,beta", AB)
def test_many_16_wide_tiles(M, N, K, transA, alpha, beta):
    # more than 1024 of them: two rows of tiles a workgroup, eight wavefronts for sums
    # of 1024 and more and four for shorter ones
    product(M, N, K, 1, transA, alpha, beta)


@pytest.mark.parametrize("n,m", [(2049, 150), (1031, 150), (2600, 40), (1024, 17), (4001, 64),
                                 (1535, 16), (1537, 16)])
def test_sums_of_a_plan_in_ranges(n, m):
    """Gram and projection products of a plan split their sums over workgroups (at most 128
    tiles of 16 x 16, n >= 1024), the last range being shorter and no multiple of 8 long.
    B U_1 = U_2 Bt and At = U_2^* A U_1, so Bt^* [At Bt] = (B U_1)^* [A U_1, B U_1]: n-term
    sums on either side, 4 n u in the Frobenius norm with room for U_2's own error."""
    rng = np.random.default_rng(n)
    A, B, X = crand(rng, n, n), crand(rng, n, n), crand(rng, n, m)
    with fm.Plan(n, m, 0.0, 1.0, 1) as plan:
        U1, AU, BU, At, Bt = plan.project(*(torch.from_numpy(x).to(DEV) for x in (A, B, X)))
    U1, AU, BU = (t.cpu().numpy() for t in (U1, AU, BU))
    norm = np.linalg.norm
    assert norm(U1.conj().T @ U1 - np.eye(m)) < 5 * np.sqrt(n) * m * U
    for t, P in ((At, AU), (Bt, BU)):
        assert norm(Bt.conj().T @ t - BU.conj().T @ P) < 4 * n * U * norm(BU) * norm(P)
