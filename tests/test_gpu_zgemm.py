"""The batched complex product at the edges of its two tiles and of its K step,
against NumPy in complex128."""
import numpy as np
import pytest
import torch

from paper_2504_04989_amd import api

pytestmark = pytest.mark.gpu

# (batch, M, N, K): many workgroups and little column padding take the wide
# tile (64 x 64 FP32, 64 x 32 FP64), the others 32 x 32
CASES = [
    (512, 65, 127, 1), (512, 127, 128, 17), (700, 64, 121, 33), (513, 128, 64, 16), (1024, 63, 64, 7),
    (1, 31, 33, 15), (2, 32, 32, 8), (3, 1, 65, 9), (600, 33, 50, 24), (511, 64, 65, 31),
]


def draw(shape, rng, dt):
    x = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    x = x.astype(np.complex64 if dt == torch.complex64 else np.complex128)
    return x.astype(np.complex128), torch.tensor(x, device="cuda")


@pytest.mark.parametrize("batch,M,N,K", CASES)
@pytest.mark.parametrize("mode", ["NN", "HN", "NH"])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("beta", [0.0, 1.0])
def test_zgemm_tiles(batch, M, N, K, mode, prec, beta):
    dt = torch.complex128 if prec == "f64" else torch.complex64
    rng = np.random.default_rng(K)
    ac, bc = mode[0] == "H", mode[1] == "H"
    A, Ad = draw((batch, K, M) if ac else (batch, M, K), rng, dt)
    B, Bd = draw((batch, N, K) if bc else (batch, K, N), rng, dt)
    C, Cd = draw((batch, M, N), rng, dt)
    # a row and a column that are not finite stay in their own row and column
    if ac:
        Ad[-1, :, -1] = float("nan")
    else:
        Ad[-1, -1, :] = float("nan")
    if bc:
        Bd[-1, -1, :] = float("inf")
    else:
        Bd[-1, :, -1] = float("inf")
    got = api.diag_zgemm(Ad, Bd, ac, bc, Cd, 1.0, beta).cpu().numpy()
    a = np.conj(A.transpose(0, 2, 1)) if ac else A
    b = np.conj(B.transpose(0, 2, 1)) if bc else B
    ref = a @ b + beta * C
    assert not np.isfinite(got[-1, -1, :]).any() and not np.isfinite(got[-1, :, -1]).any()
    got[-1, -1, :] = ref[-1, -1, :]
    got[-1, :, -1] = ref[-1, :, -1]
    # 4 K + 4 rounded operations per part, each at most u times the sum of the products' sizes
    u = 2.0 ** -53 if prec == "f64" else 2.0 ** -24
    bound = (4 * K + 4) * u * (2 * (abs(a) @ abs(b)) + abs(beta * C))
    assert np.all(abs(got - ref) <= bound)
