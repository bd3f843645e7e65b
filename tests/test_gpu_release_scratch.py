"""Idle scratch goes back to the device on request: that of the batched factorisations and
solves, and a plan's; the calls then take it again."""
import time

import numpy as np
import pytest

import paper_1404_1768_amd as fm


def test_nothing_to_release():
    fm.release_scratch()  # (also where there is no GPU)


def free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def comes_back(want):
    """Free memory reaches `want` (HIP takes back freed memory a little later)."""
    for _ in range(50):
        if free() >= want - (32 << 20):
            return True
        time.sleep(0.1)
    return False


@pytest.mark.gpu
def test_scratch_of_the_batched_calls():
    import torch
    M = torch.eye(64, dtype=torch.complex128, device="cuda").repeat(2000, 1, 1)  # 262 MB scratch
    X = torch.ones(2000, 64, 1, dtype=torch.complex128, device="cuda")
    fm.release_scratch()
    before = free()
    for _ in range(2):
        piv, info = fm.zgetrf_batched(M)
        fm.zgetrs_batched(M, piv, X)
        fm.release_scratch()
        assert comes_back(before)
    assert torch.equal(X, torch.ones_like(X)) and int(info.abs().sum()) == 0


@pytest.mark.gpu
def test_scratch_of_a_plan():
    import torch
    n, m, nodes = 256, 256, 128  # 134 MB scratch
    rng = np.random.default_rng(2)
    g = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)  # noqa: E731
    A, B, V = (torch.from_numpy(x).to("cuda")
               for x in (g(n, n) / np.sqrt(n), np.eye(n, dtype=complex), g(n, m)))
    U = torch.empty_like(V)
    with fm.Plan(n, m, 0.0, 3.0, nodes) as plan:
        first = plan.filter(A, B, V, U).clone()
        torch.cuda.synchronize()
        time.sleep(1.0)
        held = free()
        fm.release_scratch()
        assert comes_back(held + 16 * n * m * nodes)
        assert torch.equal(plan.filter(A, B, V, U), first)
