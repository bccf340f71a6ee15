"""Upper-triangle products of FP32 blocks at the edges of their 128-column
chunks, row groups and K splits, through the T-QR (block Grams up to 128
columns, R up to the trapezoid of a wide tensor) and the T-pseudoinverse (one
Gram).  Per Fourier slice: Q R = A, Q^H Q = I and A X A = A, X A = I.
Tolerances: FP32 storage of Q, R and X (2^-24 per entry of values of the norm
of the factor's row or column, sums over up to n entries taken as n roundings
of random sign, four of them), condition numbers below 20."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()

EPS = 2.0 ** -24


def slices(x):
    return np.moveaxis(np.fft.fft(x, axis=2), 2, 0)


@pytest.mark.parametrize("n1,n2", [(300, 65), (260, 119), (700, 120), (700, 121), (515, 127), (1100, 128), (600, 129),
                                   (600, 193), (700, 255), (1300, 256), (100, 300), (130, 384), (64, 130)])
def test_tqr_chunks(n1, n2):
    print(f"[gram] tqr {n1} x {n2}", flush=True)
    rng = np.random.default_rng(n1 + n2)
    A = rng.standard_normal((n1, n2, 5)).astype(np.float32)
    Q, R = (host(x) for x in api.tsvd_tqr(torch.tensor(A, device="cuda"), prec="f32"))
    for a, q, r in zip(slices(A.astype(np.float64)), slices(Q.astype(np.float64)), slices(R.astype(np.float64))):
        m = min(n1, n2)
        assert np.max(np.abs(np.tril(r, -1))) <= 16 * EPS * np.linalg.norm(r)
        assert np.linalg.norm(q @ r - a) <= 64 * EPS * np.linalg.norm(a)
        assert np.linalg.norm(q.conj().T @ q - np.eye(m)) <= 64 * EPS * m


@pytest.mark.parametrize("n2", [65, 121, 128, 129, 240, 241, 250, 256, 270])
def test_tpinv_chunks(n2):
    print(f"[gram] tpinv {n2}", flush=True)
    rng = np.random.default_rng(n2)
    A = rng.standard_normal((3 * n2 + 1, n2, 5)).astype(np.float32)
    X = host(api.tsvd_tpinv(torch.tensor(A, device="cuda"), prec="f32"))
    for a, x in zip(slices(A.astype(np.float64)), slices(X.astype(np.float64))):
        assert np.linalg.norm(x @ a - np.eye(n2)) <= 64 * EPS * 20 * n2 ** 0.5
