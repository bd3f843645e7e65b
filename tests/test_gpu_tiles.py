"""Products on the 64 x 32 output tiles (outputs too large for the split of K over
wavefronts), against NumPy in FP64: edges of the tile's rows, columns and 8-long K
steps, with one, two and more steps of its double buffer; leading dimensions past the
reach of a 32-bit offset within a tile (the launch then takes 64-bit addresses), in
single, shifted and grouped products; and C on top of A or B."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402
import pencilgen as pg  # noqa: E402

DEV = torch.device("cuda:0")
U = 2.0 ** -53
FAR = 2 ** 21 + 3      # 64 rows of this many complex128 numbers: past 2^31 bytes
FAR8 = 2 ** 24 + 3     # 8 rows


def crand(rng, *shape):
    return rng.normal(size=shape) + 1j * rng.normal(size=shape)


def abs1(x):
    return np.abs(x.real) + np.abs(x.imag)


def check(out, opA, B, C, alpha, beta):
    """Each real part of a K-term complex sum takes 2 K products and sums, whatever
    their order; alpha, beta and the final sum add four roundings more.  Twice that:
    NumPy's own product rounds as well."""
    ref = alpha * (opA @ B) + beta * C
    lim = (2 * B.shape[-2] + 8) * U * (abs(alpha.real) + abs(alpha.imag)) * (abs1(opA) @ abs1(B))
    lim = lim + (2 * B.shape[-2] + 8) * U * (abs(beta.real) + abs(beta.imag)) * abs1(C) + 1e-300
    assert np.all(np.abs(out - ref) <= 2 * lim)


def conj_t(A):
    return np.conj(np.transpose(A, (0, 2, 1)))


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (63, 31, 7), (64, 32, 8), (65, 33, 9), (33, 65, 16),
                                   (128, 64, 17), (129, 16, 24), (17, 97, 131)])
@pytest.mark.parametrize("transA", [0, 2])
@pytest.mark.parametrize("alpha,beta", [(1.0 + 0j, 0j), (-1.0 + 0j, 1.0 + 0j),
                                        (0.7 - 0.2j, -0.3 + 1.1j)])
def test_tiles_match_numpy(M, N, K, transA, alpha, beta):
    rng = np.random.default_rng(M * 131 + N * 17 + K)
    batch = 260  # past the outputs that the split of K takes
    rows, cols = (M, K) if transA == 0 else (K, M)
    hA, hB, hC = (np.full((batch, r, c + 3), np.nan + 0j) for r, c in ((rows, cols), (K, N), (M, N)))
    hA[:, :, :cols], hB[:, :, :N], hC[:, :, :N] = (crand(rng, batch, r, c) for r, c in
                                                   ((rows, cols), (K, N), (M, N)))
    tA, tB, tC = (torch.from_numpy(x).to(DEV) for x in (hA, hB, hC))
    fm.zgemm_batched(tA[:, :, :cols], tB[:, :, :N], tC[:, :, :N], alpha, beta, transA)
    out = tC.cpu().numpy()
    A, B, C = hA[:, :, :cols], hB[:, :, :N], hC[:, :, :N]
    check(out[:, :, :N], A if transA == 0 else conj_t(A), B, C, alpha, beta)
    assert np.all(np.isnan(out[:, :, N:].real))  # nothing written past a row


def far(x, ld):
    """x (batch, r, c) with rows ld apart and the matrices of the batch side by side."""
    b, r, c = x.shape
    buf = torch.empty(r * ld, dtype=torch.complex128, device=DEV)
    t = buf.as_strided((b, r, c), (c + 3, ld, 1))
    t.copy_(torch.from_numpy(x))
    return t


@pytest.mark.parametrize("which,transA", [("A", 0), ("A", 2), ("B", 0), ("C", 0)])
@pytest.mark.parametrize("alpha,beta", [(-1.0 + 0j, 1.0 + 0j), (0.7 - 0.2j, -0.3 + 1.1j)])
def test_far_rows_match_numpy(which, transA, alpha, beta):
    rng = np.random.default_rng(5)
    batch, M, N, K = 150, 66, 35, 9
    A = crand(rng, batch, *((M, K) if transA == 0 else (K, M)))
    B, C = crand(rng, batch, K, N), crand(rng, batch, M, N)
    ld = FAR8 if which == "B" or transA == 2 else FAR
    put = lambda name, x: far(x, ld) if which == name else torch.from_numpy(x).to(DEV)
    tA, tB, tC = put("A", A), put("B", B), put("C", C)
    fm.zgemm_batched(tA, tB, tC, alpha, beta, transA)
    check(tC.cpu().numpy(), A if transA == 0 else conj_t(A), B, C, alpha, beta)


@pytest.mark.parametrize("on", ["A", "B"])
def test_in_place(on):
    rng = np.random.default_rng(6)
    X, Y = crand(rng, 3, 300, 50), crand(rng, 3, 50, 50)
    if on == "B":
        X = conj_t(X).copy()
    tX, tY = torch.from_numpy(X).to(DEV), torch.from_numpy(Y).to(DEV)
    fm.zgemm_batched(*((tX, tY) if on == "A" else (tY, tX)), tX)
    check(tX.cpu().numpy(), *((X, Y) if on == "A" else (Y, X)), X, 1.0 + 0j, 0j)


@pytest.mark.parametrize("batched", [False, True])
def test_filter_of_matrices_with_far_rows(batched):
    # The residuals of the refinement sweeps (shifted products, the grouped B V of the
    # batched form) read A and B in place: the same results as from contiguous ones, to
    # the accuracy at which the sweeps stop
    p = pg.make_pencil(70, m=8, inside=4, inside_radius=0.8, outside_r=(1.3, 10.0), center=0.2,
                       radius=1.0, nodes=4, c=0.05, seed=3, name="far")
    near = [torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in (p.A, p.B, p.V)]
    away = [far(np.ascontiguousarray(x)[None], FAR)[0] for x in (p.A, p.B, p.V)]
    out = []
    for A, B, V in (near, away):
        if batched:
            with fm.Batch([p.n], [p.m], [p.center], [p.radius], p.nodes, prec=fm.MIXED) as b:
                out.append(b.filter([A], [B], [V], 3)[0].cpu().numpy())
        else:
            plan = fm.Plan(p.n, p.m, p.center, p.radius, p.nodes, prec=fm.MIXED)
            out.append(plan.filter(A, B, V).cpu().numpy())
    assert np.max(np.abs(out[0] - out[1])) <= 1e-12 * np.max(np.abs(out[0]))


@pytest.mark.parametrize("n,m", [(2049, 150), (2600, 97)])
def test_projection_products_over_ranges_of_k(n, m):
    # A U_1 and B U_1 of a plan (which has room for partial sums): four ranges of K
    rng = np.random.default_rng(n)
    A, B, X = crand(rng, n, n), crand(rng, n, n), crand(rng, n, m)
    plan = fm.Plan(n, m, 0.0, 1.0, 1)
    U1, AU, BU, _, _ = plan.project(*(torch.from_numpy(x).to(DEV) for x in (A, B, X)))
    U1 = U1.cpu().numpy()
    zero = np.zeros((n, m))
    check(AU.cpu().numpy(), A, U1, zero, 1.0 + 0j, 0j)
    check(BU.cpu().numpy(), B, U1, zero, 1.0 + 0j, 0j)
