"""The eigensolver at the tile edges of the register-resident tridiagonalisation
(32-row tiles, up to 192 rows; the next size takes the blocked form), against
LAPACK's eigh, with the tolerances of the kernel-level test: the backward
error of a Householder reduction, about m roundings of ||G||."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api
from tests.test_gpu_heig import _gram

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("m,batch", [(3, 2), (31, 3), (32, 2), (33, 2), (64, 2), (65, 2), (96, 2), (97, 2), (128, 2),
                                     (129, 2), (160, 2), (161, 3), (191, 2), (192, 300), (193, 2)])
def test_tile_edges_vs_lapack(m, batch):
    print(f"[tridiag] m={m} batch={batch}", flush=True)
    k = max(1, m // 3)
    G = _gram(min(batch, 3), m, seed=m, decay=1.5)
    G = G[np.arange(batch) % len(G)]
    lam, W, info = api.diag_heig(torch.tensor(G, device="cuda"), k)
    assert info["eig_noconv"] == 0 and info["nonfinite"] == 0
    lam, W = host(lam), host(W)
    assert all(np.array_equal(lam[f], lam[f % 3]) and np.array_equal(W[f], W[f % 3]) for f in range(3, batch))
    for f in range(min(batch, 3)):
        ref = np.linalg.eigvalsh(G[f])[::-1][:k]
        assert np.max(np.abs(lam[f] - ref)) <= 1e-13 * m * ref[0]
        R = G[f] @ W[f] - W[f] * lam[f]
        assert np.max(np.linalg.norm(R, axis=0)) <= 1e-12 * m * ref[0]
        assert np.max(np.abs(W[f].conj().T @ W[f] - np.eye(k))) <= 1e-10


def test_identity_and_diagonal_reflectors():
    """Columns whose reflector is the identity: a diagonal matrix, a matrix
    with a zero trailing block, and the zero matrix."""
    m, k = 40, 6
    G = np.zeros((3, m, m), dtype=np.complex128)
    G[0] = np.diag(np.arange(m, 0, -1.0))
    G[1, :20, :20] = _gram(1, 20, seed=1, decay=1.0)[0]
    lam, W, info = api.diag_heig(torch.tensor(G, device="cuda"), k)
    assert info["nonfinite"] == 0
    lam, W = host(lam), host(W)
    for f in range(3):
        ref = np.linalg.eigvalsh(G[f])[::-1][:k]
        assert np.max(np.abs(lam[f] - ref)) <= 1e-13 * m * max(ref[0], 1e-300)
        assert np.max(np.abs(G[f] @ W[f] - W[f] * lam[f])) <= 1e-12 * m * max(ref[0], 1e-300)
