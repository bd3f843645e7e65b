"""The orthonormalisation's number of passes: blocks whose second Gram matrix is
near the identity stop at two, ill-conditioned ones take three; either way U_1 is
orthonormal to rounding and spans the block."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")
U = 2.0 ** -53


@pytest.mark.parametrize("n,m", [(64, 5), (257, 40), (900, 130)])
@pytest.mark.parametrize("decades", [0, 3, 5, 7, 10])
@pytest.mark.parametrize("ldpad", [0, 7])
def test_orthonormal_for_every_condition_number(n, m, decades, ldpad):
    rng = np.random.default_rng(n + decades)
    g = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)  # noqa: E731
    Ql, _ = np.linalg.qr(g(n, m))
    Qr, _ = np.linalg.qr(g(m, m))
    V = (Ql * np.logspace(0, -decades, m)) @ Qr
    A, B = g(n, n), np.eye(n) + 0.05 * g(n, n) / np.sqrt(n)
    tA, tB = torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV)
    box = torch.full((n, m + ldpad), complex(np.nan, np.nan), dtype=torch.complex128, device=DEV)
    tV = box[:, :m]
    tV.copy_(torch.from_numpy(V).to(DEV))
    with fm.Plan(n, m, 0.0, 1.0, 1) as plan:
        for _ in range(2):  # the second time on an orthonormal block
            Q, AQ, BQ, At, Bt = plan.project(tA, tB, tV)
            Qh = Q.cpu().numpy()
            assert np.linalg.norm(Qh.conj().T @ Qh - np.eye(m)) < 5 * np.sqrt(n) * m * U
            assert np.linalg.norm(V - Qh @ (Qh.conj().T @ V)) < 5 * np.sqrt(n) * m * U * np.linalg.norm(V)
            assert np.all(np.isnan(box.cpu().numpy()[:, m:].real))
