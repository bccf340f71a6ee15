"""The eigensolver on large clusters of equal eigenvalues, of sizes that its
cluster pass holds in LDS and beyond (60 KB of members), against the precision of
well-separated eigenvalues.

Tolerances, relative to ||G||: the cluster pass leaves a residual of 16 eps, the
Householder reduction and its back-transformation m roundings u of either kind:
16 eps + 2 m u for the residual, and twice that for the orthonormality (the
other eigenvalues are at least half of ||G|| away, and the back-transformation
adds its own).  Past 192 rows the reduction adds its products in fixed point with
a step scaled to m ||G||_F, which is coarser; its residual there is held to the
kernel-level test's 1e-12 m, the orthonormality to the same as below."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("m,k,equal", [(16, 16, 15), (64, 40, 30), (192, 150, 120), (192, 192, 190), (193, 193, 190),
                                       (600, 60, 40), (600, 350, 300)])
def test_equal_eigenvalues(m, k, equal):
    print(f"[clusters] m={m} k={k}, {equal} equal", flush=True)
    rng = np.random.default_rng(m + equal)
    lam = np.concatenate([np.full(equal, 2.0), np.linspace(1.0, 0.9, m)[: m - equal]])
    G = np.empty((3, m, m), complex)
    for f in range(3):
        U, _ = np.linalg.qr(rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m)))
        G[f] = (U * lam) @ U.conj().T
        G[f] = (G[f] + G[f].conj().T) / 2
    got, W, info = api.diag_heig(torch.tensor(G, device="cuda"), k)
    got, W = host(got), host(W)
    assert info["eig_noconv"] == 0 and info["nonfinite"] == 0
    tol = 16 * 2.0 ** -52 + 2 * m * 2.0 ** -53
    for f in range(3):
        res = np.max(np.linalg.norm(G[f] @ W[f] - W[f] * got[f], axis=0)) / 2.0
        orth = np.max(np.abs(W[f].conj().T @ W[f] - np.eye(k)))
        print(f"[clusters]   slice {f}: residual {res:.1e}, W^H W {orth:.1e} (tolerance {tol:.1e})", flush=True)
        assert res <= (tol if m <= 192 else 1e-12 * m) and orth <= 2 * tol
