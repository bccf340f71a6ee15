"""The eigensolver up to its largest matrices, m = 1024, where the panel of the
blocked tridiagonalisation is cut to what LDS holds (the panel's width changes
at 480 / 481 and 928 / 929 rows), with the kernel-level test's bounds; and a call
whose basis has 1000 columns, against the same method with numpy's QR and SVD.
The columns are Gaussian, so X_hat keeps the parity bound of 1e-10."""
import numpy as np
import pytest
import torch

from tests.gpu_util import dev, host, load_api
from tests.test_gpu_heig import _gram

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("m,batch", [(480, 200), (481, 200), (864, 1), (865, 1), (896, 2), (928, 2), (929, 2), (1000, 130), (1024, 3)])
def test_largest(m, batch):
    k = 12
    print(f"[heig] m={m} batch={batch}", flush=True)
    G = _gram(1, m, seed=m, decay=1.5)[0]
    lam, W, info = api.diag_heig(torch.tensor(G, device="cuda").expand(batch, m, m).contiguous(), k)
    lam, W = host(lam), host(W)
    assert info["eig_noconv"] == 0 and info["nonfinite"] == 0
    assert np.array_equal(lam, np.broadcast_to(lam[0], lam.shape)) and np.array_equal(W, np.broadcast_to(W[0], W.shape))
    ref = np.linalg.eigvalsh(G)[::-1][:k]
    assert np.max(np.abs(lam[0] - ref)) <= 1e-13 * m * ref[0]
    assert np.max(np.linalg.norm(G @ W[0] - W[0] * lam[0], axis=0)) <= 1e-12 * m * ref[0]
    assert np.max(np.abs(W[0].conj().T @ W[0] - np.eye(k))) <= 1e-10


def test_basis_of_1000_columns():
    n1, n2, n3, k, b, q = 1010, 1020, 1, 20, 500, 1
    print(f"[heig] rbk m={b * (q + 1)}", flush=True)
    rng = np.random.default_rng(4)
    A, W = rng.standard_normal((n1, n2, n3)), rng.standard_normal((n2, b, n3))
    X = host(api.tsvd_rbk_approx(dev(A), dev(W), k, b, q, "f64")[3])
    a, w = A[:, :, 0], W[:, :, 0]
    x0 = np.linalg.qr(a @ w)[0]
    y = a @ (a.T @ x0)
    for _ in range(2):
        y = y - x0 @ (x0.T @ y)
    Q = np.linalg.qr(np.concatenate([x0, y], axis=1))[0]
    u, s, v = np.linalg.svd(Q.T @ a, full_matrices=False)
    ref = (Q @ u[:, :k] * s[:k]) @ v[:k]
    assert np.linalg.norm(X[:, :, 0] - ref) <= 1e-10 * np.linalg.norm(ref)
