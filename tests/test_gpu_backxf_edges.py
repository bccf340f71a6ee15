"""The eigensolver at the sizes where its back-transformation changes form (448 /
449 and 640 / 641 rows; the smaller ones change every 32 to 64 rows), a number of
columns that does not fill its last workgroup, and between the register-resident
and the cooperative tridiagonalisations, with the kernel-level test's bounds."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api
from tests.test_gpu_heig import _gram

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("m,k", [(32, 9), (33, 9), (64, 9), (65, 9), (128, 17), (129, 17), (192, 17), (193, 17), (230, 23),
                                 (256, 17), (257, 17), (448, 17), (449, 17), (640, 17), (641, 17)])
def test_back_transformation_edges(m, k):
    print(f"[backxf] m={m} k={k}", flush=True)
    G = _gram(2, m, seed=m, decay=1.5)
    lam, W, info = api.diag_heig(torch.tensor(G, device="cuda"), k)
    lam, W = host(lam), host(W)
    assert info["eig_noconv"] == 0 and info["nonfinite"] == 0
    for f in range(2):
        ref = np.linalg.eigvalsh(G[f])[::-1][:k]
        assert np.max(np.abs(lam[f] - ref)) <= 1e-13 * m * ref[0]
        assert np.max(np.linalg.norm(G[f] @ W[f] - W[f] * lam[f], axis=0)) <= 1e-12 * m * ref[0]
        assert np.max(np.abs(W[f].conj().T @ W[f] - np.eye(k))) <= 1e-10
