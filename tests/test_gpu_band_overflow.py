"""Band pencils whose node solutions grow exponentially from one end to the other (random
entries, many more subdiagonals than superdiagonals): the elimination from both ends
overflows where partial pivoting from the top does not, and the solve must come back as
that of the latter, here with Ritz pairs that have not converged."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")


def csr(n, offsets, diagonals):
    rows, cols, vals = [], [], []
    for o, d in zip(offsets, diagonals):
        i = np.arange(max(0, -o), min(n, n - o))
        rows.append(i)
        cols.append(i + o)
        vals.append(d)
    rows, cols, vals = map(np.concatenate, (rows, cols, vals))
    order = np.lexsort((cols, rows))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    return [torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
            for x in (rp, cols[order].astype(np.int32), vals[order].astype(np.complex128))]


@pytest.mark.parametrize("kl,ku", [(60, 1), (40, 1)])
@pytest.mark.parametrize("seed", [0, 1])
def test_comes_back_from_the_top(kl, ku, seed):
    n, m = 3000, 20
    rng = np.random.default_rng(seed)
    offsets = list(range(-kl, ku + 1))
    A = csr(n, offsets, [rng.normal(size=n - abs(o)) for o in offsets])
    B = csr(n, [0], [np.ones(n)])
    V = rng.normal(size=(n, m)) + 1j * rng.normal(size=(n, m))
    with fm.Plan(n, m, 0.3, 0.05, 16, max_iter=6) as plan:
        r = plan.solve_csr(A, B, torch.from_numpy(V).to(DEV))
        assert r.band == (kl, ku) and r.flag in (0, -1)  # (which of the two rounding decides)
        assert np.all(np.isfinite(r.lam)) and bool(torch.isfinite(r.X.abs()).all())
