"""Orthonormalisation of a column whose squared norm lies near the ends of the type's
range (the pivot of its Gram matrix is then subnormal, or nearly overflows)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("scale", [1e-157, 4e-156, 1e-155, 1e-100, 1.0, 1e100, 5e152])
def test_a_single_column_at_the_ends_of_the_range(scale):
    n = 300
    rng = np.random.default_rng(7)
    g = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)  # noqa: E731
    A, B, v = g(n, n), np.eye(n) + 0.05 * g(n, n) / np.sqrt(n), g(n, 1)
    with fm.Plan(n, 1, 0.0, 1.0, 1) as plan:
        Q = plan.project(*(torch.from_numpy(x).to(DEV) for x in (A, B, v * scale)))[0].cpu().numpy()
    # a norm of n terms, a division: (n + 4) u in the worst case
    assert np.linalg.norm(Q - v / np.linalg.norm(v)) < (n + 4) * 2.0 ** -53
