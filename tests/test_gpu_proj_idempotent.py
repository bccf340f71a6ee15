"""P(A) = Q Q^H A of square, well-conditioned slices gives back the projector Q Q^H
= P_f A_f^{-1}: Hermitian, idempotent and of trace m, at the edges of the blocks
that one workgroup orthonormalises whole and beyond them.

Tolerance: n-term sums in the working precision u behind P, multiplied by the
slice's condition number (about 3) and by two for the products of the check,
in the 2-norm; with the trace, n times that."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,b,q", [(3, 1, 1), (16, 4, 2), (63, 15, 1), (64, 16, 2), (65, 17, 1), (130, 10, 3), (159, 32, 1),
                                   (160, 31, 2), (161, 32, 1), (300, 16, 3), (431, 16, 2), (600, 9, 2)])
def test_projector(n, b, q, prec):
    n3, m = 4, b * (q + 1)
    print(f"[idempotent] n={n} b={b} q={q} {prec}", flush=True)
    rng = np.random.default_rng(n + b)
    dt, u = (np.float64, 2.0 ** -53) if prec == "f64" else (np.float32, 2.0 ** -24)
    A = rng.standard_normal((n, n, n3))
    A[:, :, 0] += 4 * n ** 0.5 * np.eye(n)
    A = A.astype(dt)
    W = rng.standard_normal((n, b, n3)).astype(dt)
    P = host(api.tsvd_proj(torch.tensor(A, device="cuda"), torch.tensor(W, device="cuda"), b, q, prec))
    Pf, Af = (np.fft.fft(x.astype(np.float64), axis=2) for x in (P, A))
    for f in range(n3):
        pi = Pf[:, :, f] @ np.linalg.inv(Af[:, :, f])
        tol = 2 * n * u * np.linalg.cond(Af[:, :, f])
        e = [np.linalg.norm(x, 2) for x in (pi @ pi - pi, pi - pi.conj().T)]
        print(f"[idempotent]   slice {f}: {e[0]:.1e} {e[1]:.1e} (tolerance {tol:.1e})", flush=True)
        assert max(e) <= tol and abs(np.trace(pi) - m) <= n * tol
