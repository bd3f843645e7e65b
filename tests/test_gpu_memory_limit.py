"""The scratch of the node solves where device memory is short: a filter (and the making of
a mixed plan) that fits without it runs, with the same result; and a plan's idle scratch
goes to another plan that needs the memory.  The memory is taken up by a tensor; how much
a call needs is read off the same call with memory to spare."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")
N_, M_, NODES = 512, 256, 128
PIECE = {fm.FP64: 16 * N_ * M_ * NODES, fm.MIXED: 8 * N_ * M_ * NODES}  # 268, 134 MB


def free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def leave(nbytes):
    """Tensors that leave about nbytes of device memory free (HIP takes back freed
    memory a little later: until that is seen no more)."""
    hog, quiet = [], 0
    while quiet < 3:
        more = free() - nbytes
        if more > (16 << 20):
            hog.append(torch.empty(more, dtype=torch.uint8, device=DEV))
            quiet = 0
        else:
            quiet += 1
            time.sleep(0.2)
    return hog


@pytest.fixture(scope="module")
def pencil():
    rng = np.random.default_rng(1)
    g = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)  # noqa: E731
    A = g(N_, N_) / np.sqrt(N_)
    return [torch.from_numpy(x).to(DEV) for x in (A, np.eye(N_, dtype=complex), g(N_, M_))]


def plan(prec):
    return fm.Plan(N_, M_, 0.0, 3.0, NODES, prec=prec)  # (the spectrum lies in |z| < 2)


@pytest.mark.parametrize("prec", [fm.FP64, fm.MIXED])
def test_filter_without_room_for_the_solves_scratch(pencil, prec):
    A, B, V = pencil
    U, U2 = torch.empty_like(V), torch.empty_like(V)
    with plan(prec) as p:
        at = free()
        p.filter(A, B, V, U)
        need = at - free()
    with plan(prec) as p:
        hog = leave(need - PIECE[prec] // 2)
        p.filter(A, B, V, U2)
        torch.cuda.synchronize()
        del hog
        p.filter(A, B, V, U2)  # (with memory to spare again)
    free()
    # u cond(z B - A) of each node, cond < 10 for |z| = 3
    assert float((U - U2).norm() / U.norm()) < 1e-12


def test_making_a_mixed_plan_needs_no_scratch(pencil):
    at = free()
    with plan(fm.MIXED):
        need = at - free()
    n2 = 8 * N_ * M_ * NODES
    # Y, T1, T2 (complex128) and Yc (complex64), the n x m and m x m blocks beside them
    assert need < 7 * n2 + 40 * 16 * N_ * M_ + (64 << 20)


def test_idle_scratch_goes_to_the_next_plan(pencil):
    A, B, V = pencil
    at = free()
    with plan(fm.FP64):
        need = at - free()
    with plan(fm.FP64) as p:
        U = p.filter(A, B, V)
        hog = leave(need - PIECE[fm.FP64] // 2)
        with plan(fm.FP64):
            del hog
            free()
        U2 = p.filter(A, B, V)
    free()
    assert float((U - U2).norm() / U.norm()) < 1e-12
