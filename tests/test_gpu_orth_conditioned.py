"""Orthonormalisation of ill-conditioned blocks, through the T-QR of one panel: the
small blocks that one workgroup takes whole, at the edges of its tiles and limits,
and their neighbours that take the separate launches.  Columns of a slice fall
geometrically down to 1 / kappa in random directions.

Tolerances.  FP64, CholeskyQR2 after the shifted passes: 6 (n r + r (r + 1)) u for
Q^H Q - I (Yamamoto et al., 2015) and the same, of ||A||, for Q R - A.  FP32
storage adds one rounding 2^-24 of the entries of Q and R: twice that times
sqrt(r) for Q^H Q - I in the Frobenius norm, and of ||A|| for Q R - A; both through
the inverse DFT and its FP32 store and back, hence twice as much again."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()

SIZES = [(2, 1), (16, 15), (17, 16), (18, 17), (160, 16), (160, 17), (160, 32), (161, 32), (164, 33), (431, 16), (600, 9)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kappa", [1e4, 1e8, 1e14])
@pytest.mark.parametrize("n,r", SIZES)
def test_ill_conditioned_panel(n, r, kappa, prec):
    n3 = 3
    rng = np.random.default_rng(n + r)
    s = kappa ** (-np.arange(r) / max(r - 1, 1))
    X = np.empty((2, n, r), complex)
    for f in range(2):
        u, v = (np.linalg.qr(rng.standard_normal((d, r)) + f * 1j * rng.standard_normal((d, r)))[0] for d in (n, r))
        X[f] = (u * s) @ v.conj().T
    A = np.fft.irfft(X, n3, axis=0).transpose(1, 2, 0).astype(np.float64 if prec == "f64" else np.float32)
    A = np.ascontiguousarray(A)
    ws = api.workspace(n, r, n3, 0, 0, 0, prec, "tqr", "cuda")
    Q, R = api.tsvd_tqr(torch.tensor(A, device="cuda"), prec, ws=ws)
    info = api.read_info(ws)
    assert info["chol_breakdown"] == 0 and info["nonfinite"] == 0
    Qf, Rf, Af = (np.fft.fft(np.asarray(x, np.float64), axis=2) for x in (host(Q), host(R), A))
    t64 = 6 * (n * r + r * (r + 1)) * 2.0 ** -53
    t32 = 0.0 if prec == "f64" else 4 * 2.0 ** -24
    for f in range(n3):
        q = Qf[:, :, f]
        orth = np.linalg.norm(q.conj().T @ q - np.eye(r))
        res = np.linalg.norm(q @ Rf[:, :, f] - Af[:, :, f]) / np.linalg.norm(Af[:, :, f])
        print(f"[orth] {n} x {r} kappa {kappa:.0e} {prec} slice {f}: {orth:.1e} {res:.1e}", flush=True)
        assert orth <= t64 + t32 * r ** 0.5
        assert res <= t64 + t32
