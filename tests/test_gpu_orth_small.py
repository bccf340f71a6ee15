"""Small blocks, orthonormalised whole by one workgroup per slice, at the edges
of its tiles (16 columns, 16 rows), of its size limits and past them, through
the projection P = Q Q^H A (Alg. 2) and Alg. 1's factors: per Fourier slice
against the same recursion with numpy's QR.  The slices are Gaussian, n x n/2
(condition below 10), so the subspaces' condition stays below about 100:
tolerance 100 x 1000 roundings of the working precision, relative to ||A||."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()

# (n1, n2, b, q)
CASES = [(2, 1, 1, 0), (16, 9, 1, 1), (17, 33, 4, 3), (63, 40, 15, 1), (64, 32, 16, 1), (65, 40, 17, 1), (130, 70, 10, 3),
         (159, 80, 32, 1), (160, 96, 31, 2), (161, 80, 32, 1), (300, 150, 16, 3), (431, 100, 16, 2), (600, 60, 9, 2)]


def krylov(a, w, q, power):
    x = np.linalg.qr(a @ w)[0]
    basis = [x]
    for _ in range(q):
        y = a.conj().T @ basis[-1]
        if power:
            y = np.linalg.qr(y)[0]
        y = a @ y
        if not power:
            prev = np.concatenate(basis, axis=1)
            for _ in range(2):
                y = y - prev @ (prev.conj().T @ y)
        basis.append(np.linalg.qr(y)[0])
    return basis[-1] if power else np.linalg.qr(np.concatenate(basis, axis=1))[0]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n1,n2,b,q", CASES)
def test_small_blocks(n1, n2, b, q, prec):
    n3 = 4
    print(f"[orth] {n1} x {n2}, b={b}, q={q}, {prec}", flush=True)
    rng = np.random.default_rng(n1 + b)
    dt = np.float64 if prec == "f64" else np.float32
    A = rng.standard_normal((n1, n2, n3)).astype(dt)
    W = rng.standard_normal((n2, b, n3)).astype(dt)
    Ad, Wd = torch.tensor(A, device="cuda"), torch.tensor(W, device="cuda")
    tol = 1e5 * (2.0 ** -53 if prec == "f64" else 2.0 ** -24)
    P = np.fft.fft(host(api.tsvd_proj(Ad, Wd, b, q, prec)).astype(np.float64), axis=2)
    U, S, V = (np.fft.fft(host(x).astype(np.float64), axis=-1) for x in api.tsvd_power(Ad, Wd, b, b, q, prec))
    Af, Wf = (np.fft.fft(x.astype(np.float64), axis=2) for x in (A, W))
    for f in range(n3):
        a, w = Af[:, :, f], Wf[:, :, f]
        x = krylov(a, w, q, False)
        assert np.linalg.norm(P[:, :, f] - x @ (x.conj().T @ a)) <= tol * np.linalg.norm(a)
        x = krylov(a, w, q, True)
        got = (U[:, :, f] * S[:, f]) @ V[:, :, f].conj().T
        assert np.linalg.norm(got - x @ (x.conj().T @ a)) <= tol * np.linalg.norm(a)
