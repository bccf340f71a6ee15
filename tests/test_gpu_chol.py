"""CholeskyQR at the edges of the register-resident elimination's 16-column
blocks, through the T-QR (whose panels are at most 128 columns wide): Q and R
against numpy's QR per Fourier slice with the diagonal of R positive, FP64.
Tolerance: a few hundred roundings of the column norms for well-conditioned
Gaussian slices (condition below 10)."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("r", [1, 2, 15, 16, 17, 32, 33, 48, 64, 65, 96, 112, 127, 128])
def test_tqr_block_edges(r):
    print(f"[chol] r={r}", flush=True)
    n1, n3 = 4 * r + 3, 3
    A = np.random.default_rng(r).standard_normal((n1, r, n3))
    Q, R = (host(x) for x in api.tsvd_tqr(torch.tensor(A, device="cuda"), prec="f64"))
    Af, Qf, Rf = (np.fft.fft(x, axis=2) for x in (A, Q, R))
    for f in range(n3):
        q, t = np.linalg.qr(Af[:, :, f])
        ph = np.diag(t) / np.abs(np.diag(t))
        assert np.max(np.abs(Qf[:, :, f] - q * ph)) <= 1e-13
        assert np.max(np.abs(Rf[:, :, f] - ph.conj()[:, None] * t)) <= 1e-13 * np.linalg.norm(t)
