"""The orthonormal basis of slices of a lower rank than it has columns: blocks that
are part rounding noise, or nothing else.

Tolerances, u the storage precision's rounding unit.  U^H U - I, Q^H Q - I: CholeskyQR2's
6 (n b + b (b + 1)) 2^-53 (Yamamoto et al., 2015) with b the number of columns compared,
and for FP32 storage 2^-24 on every entry of two unit vectors and of the result, both
through the inverse DFT and its store and back, (4 + sqrt(b)) 2^-24 in all.  P(A) - A and
Q R - A, of ||A||: n2-term sums in the working precision behind the products, n2 u, and
twice the noise that was added (more than the range finder's error for a basis far wider
than the rank)."""
import numpy as np
import pytest
import torch

from paper_2504_04989_amd import inputs
from tests.gpu_util import load_api

pytestmark = pytest.mark.gpu
api = load_api()
UNIT = {"f64": 2.0 ** -53, "f32": 2.0 ** -24}
N3 = 3


def tensor(n1, n2, rank, noise, prec):
    A = inputs.lowrank_tensor(n1, n2, N3, rank, ("geom", 0.8), noise, seed=n1 + rank)
    return torch.tensor(A, device="cuda", dtype=torch.float64 if prec == "f64" else torch.float32)


def orth_error(Q):
    Qf = torch.fft.fft(Q.double(), dim=2)
    eye = torch.eye(Q.shape[1], device="cuda")
    return max(float((Qf[:, :, f].conj().T @ Qf[:, :, f] - eye).abs().max()) for f in range(N3))


def orth_tol(n, b, prec):
    return 6 * (n * b + b * (b + 1)) * 2.0 ** -53 + (0.0 if prec == "f64" else (4 + b ** 0.5) * 2.0 ** -24)


# one workgroup per slice (b <= 16, b <= 32), separate launches, and blocks that
# change from the one to the other; bases that fill the space; ranks within a block
SMALL = [(8, 8, 2, 3, 3), (24, 24, 6, 3, 7), (64, 64, 16, 3, 20), (60, 200, 20, 2, 1), (120, 100, 32, 2, 60),
         (161, 120, 17, 3, 30), (300, 200, 33, 2, 50), (431, 150, 16, 2, 20), (200, 150, 9, 5, 20)]


@pytest.mark.parametrize("noise", [0.0, 1e-13])
@pytest.mark.parametrize("n1,n2,b,q,rank", SMALL)
def test_blocks_of_signal_and_noise(n1, n2, b, q, rank, noise):
    A = tensor(n1, n2, rank, noise, "f64")
    W = torch.tensor(inputs.omega(n2, b, N3, 1), device="cuda")
    P = api.tsvd_proj(A, W, b, q, "f64")
    U = api.tsvd_rbk(A, W, b, b, q, "f64")[0]
    e, r = orth_error(U), float(torch.linalg.norm(P - A) / torch.linalg.norm(A))
    tol = n2 * UNIT["f64"] + 2 * noise * (n1 * n2 * N3) ** 0.5 / float(torch.linalg.norm(A))
    print(f"[lowrank] {n1}x{n2} b={b} q={q} rank {rank} noise {noise}: U^H U {e:.1e} P {r:.1e} ({tol:.1e})", flush=True)
    assert e <= orth_tol(n1, b * (q + 1), "f64") and r <= tol


# many blocks, m = b (q + 1) up to 800: P alone (an FP32 call's U comes from the same basis)
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n1,n2,b,q,rank", [(900, 900, 16, 12, 5), (300, 280, 16, 7, 3), (150, 140, 32, 3, 40), (150, 719, 16, 8, 1),
                                            (641, 870, 52, 6, 16), (1000, 900, 100, 7, 10), (90, 259, 16, 4, 5)])
def test_many_blocks(n1, n2, b, q, rank, prec):
    A = tensor(n1, n2, rank, 0.0, prec)
    W = torch.tensor(inputs.omega(n2, b, N3, 1), device="cuda", dtype=A.dtype)
    P = api.tsvd_proj(A, W, b, q, prec)
    r = float(torch.linalg.norm((P - A).double()) / torch.linalg.norm(A.double()))
    print(f"[lowrank] {n1}x{n2} b={b} q={q} rank {rank} {prec}: P {r:.1e} ({n2 * UNIT[prec]:.1e})", flush=True)
    assert r <= n2 * UNIT[prec]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n1,n2,rank", [(300, 200, 10), (600, 400, 150), (512, 384, 1), (1000, 1000, 10), (400, 900, 130)])
def test_tqr(n1, n2, rank, prec):
    A = tensor(n1, n2, rank, 0.0, prec)
    Q, R = api.tsvd_tqr(A, prec)
    Qf, Rf, Af = (torch.fft.fft(x.double(), dim=2) for x in (Q, R, A))
    e = orth_error(Q)
    r = max(float(torch.linalg.norm(Qf[:, :, f] @ Rf[:, :, f] - Af[:, :, f]) / torch.linalg.norm(Af[:, :, f])) for f in range(N3))
    print(f"[lowrank] T-QR {n1}x{n2} rank {rank} {prec}: Q^H Q {e:.1e} Q R {r:.1e}", flush=True)
    assert e <= orth_tol(n1, Q.shape[1], prec) and r <= n2 * UNIT[prec]
