"""A sparse solve whose band factors do not fit from both ends but do from the top (no
subdiagonals, 63 superdiagonals: from the top there are no multipliers to keep)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")


def free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def test_less_memory_from_the_top():
    n, m, ku, nodes = 16000, 12, 63, 64
    rng = np.random.default_rng(3)
    # A = D Q, B = Q with Q = I + an upper band: eigenvalues D
    cols = np.arange(n)[:, None] + np.arange(ku + 1)
    keep = cols < n
    q = 0.3 * (rng.normal(size=cols.shape) + 1j * rng.normal(size=cols.shape)) / np.sqrt(ku + 1)
    q[:, 0] += 1.0
    r = np.concatenate([np.sqrt(rng.random(6)) * 0.8, np.sqrt(1.69 + rng.random(n - 6) * 8)])
    d = (r * np.exp(2j * np.pi * rng.random(n)))[rng.permutation(n)]
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    put = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)  # noqa: E731
    ci = put(cols[keep].astype(np.int32))
    A, B = (put(rp), ci, put((q * d[:, None])[keep])), (put(rp), ci, put(q[keep]))
    V = put(rng.normal(size=(n, m)) + 1j * rng.normal(size=(n, m)))

    def solve(plan):
        res = plan.solve_csr(A, B, V)
        assert res.band == (0, ku) and res.flag == 1
        return np.sort_complex(res.lam)

    with fm.Plan(n, m, 0.0, 1.0, nodes, max_iter=10) as plan:
        at = free()
        lam = solve(plan)
        need = at - free()
    multipliers = 16 * nodes * 63 * (n - 63) * 7 // 20  # the bottom side's
    with fm.Plan(n, m, 0.0, 1.0, nodes, max_iter=10) as plan:
        hog, quiet = [], 0
        while quiet < 3:  # (HIP takes back freed memory a little later)
            more = free() - (need - multipliers // 2)
            if more > (16 << 20):
                hog.append(torch.empty(more, dtype=torch.uint8, device=DEV))
                quiet = 0
            else:
                quiet += 1
                time.sleep(0.2)
        again = solve(plan)
        del hog
    free()
    want = np.sort_complex(d[np.abs(d) < 1.0])
    assert len(lam) == len(again) == len(want)
    assert np.max(np.abs(lam - want)) < 1e-10 and np.max(np.abs(again - want)) < 1e-10
