"""The mode-3 DFT over lengths of every kind of factorisation: the radices 2 to
13, one or several larger primes (general passes), their products, the last
length that fits LDS and lengths beyond it, against numpy.  Tolerance: 8 N
roundings of 2^-53 of the tube's absolute sum (N-term sums with twiddles of one
rounding each), plus one FP32 rounding of the result for FP32 storage."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()

LENGTHS = [1, 2, 3, 5, 6, 7, 9, 11, 13, 15, 17, 19, 34, 37, 39, 51, 100, 121, 169, 191, 200, 221, 243, 251, 255, 289, 323,
           510, 1021, 1300, 1361, 1367, 1500]


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ntubes", [1, 67])
def test_lengths(n, prec, ntubes):
    print(f"[fft] n3={n} {prec} {ntubes} tubes", flush=True)
    rng = np.random.default_rng(n)
    dt, ulp = (np.float64, 0.0) if prec == "f64" else (np.float32, 2.0 ** -24)
    X = rng.standard_normal((ntubes, n)).astype(dt)
    ref = np.fft.rfft(X.astype(np.float64), axis=1).T
    bound = 8 * n * 2.0 ** -53 * np.abs(X).sum(axis=1).max()
    got = api.diag_fft_r2c(torch.tensor(X, device="cuda"))
    assert np.all(np.abs(host(got).astype(np.complex128) - ref) <= bound + 2 * ulp * np.abs(ref))
    # the inverse of a spectrum whose real bins are made real on the way in
    S = (rng.standard_normal(ref.shape) + 1j * rng.standard_normal(ref.shape)).astype(np.complex64 if ulp else np.complex128)
    T = S.astype(np.complex128)
    T[0].imag = 0
    if n % 2 == 0:
        T[n // 2].imag = 0
    back = np.fft.irfft(T, n, axis=0).T
    bound = 8 * n * 2.0 ** -53 * 2 * np.abs(T).sum(axis=0).max() / n
    got = host(api.diag_fft_c2r(torch.tensor(S, device="cuda"), n)).astype(np.float64)
    assert np.all(np.abs(got - back) <= bound + 2 * ulp * np.abs(back))
