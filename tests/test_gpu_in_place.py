"""Products written over an operand whose rows have another length than the output's:
outputs of up to 64 x 64 come from one workgroup, which has read both operands by then."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402

import paper_1404_1768_amd as fm  # noqa: E402

DEV = torch.device("cuda:0")
U = 2.0 ** -53


def crand(rng, *shape):
    return rng.normal(size=shape) + 1j * rng.normal(size=shape)


@pytest.mark.parametrize("on", ["A", "B"])
@pytest.mark.parametrize("transA", [0, 2])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (40, 33, 57), (64, 32, 20), (17, 64, 33)])
def test_over_rows_of_another_length(on, transA, M, N, K):
    rng = np.random.default_rng(M + N + K)
    batch = 300
    A = crand(rng, batch, *((M, K) if transA == 0 else (K, M)))
    B = crand(rng, batch, K, N)
    X = A if on == "A" else B
    ld, room = X.shape[2] + 5, 64 * 80
    box = torch.zeros(batch * room, dtype=torch.complex128, device=DEV)
    tX = box.as_strided(X.shape, (room, ld, 1))
    tX.copy_(torch.from_numpy(X))
    tC = box.as_strided((batch, M, N), (room, N + 1, 1))
    other = torch.from_numpy(B if on == "A" else A).to(DEV)
    fm.zgemm_batched(*((tX, other) if on == "A" else (other, tX)), tC, 1.0, 0.0, transA)
    opA = A if transA == 0 else np.conj(np.transpose(A, (0, 2, 1)))
    # 2 K products and sums for each part, NumPy's as many
    lim = 2 * (2 * K + 8) * U * np.sqrt(2.0) * (np.abs(opA) @ np.abs(B))
    assert np.all(np.abs(tC.cpu().numpy() - opA @ B) <= lim)
