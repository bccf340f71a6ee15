"""The mode-3 DFT of lengths with a prime factor above 13, at numbers of tubes on
both sides of the rule that gives few of them to the direct form and many to the
general passes in LDS, against numpy.  Tolerance as for the other lengths: 8 N
roundings of 2^-53 of the tube's absolute sum, plus two FP32 roundings of the
result for FP32 storage."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,ntubes", [(17, 5), (17, 40001), (34, 100), (34, 9001), (59, 2000), (59, 9000), (51, 1), (51, 3000),
                                      (191, 300), (191, 5003), (218, 65), (218, 3001), (289, 3), (509, 130), (509, 1025),
                                      (838, 700), (1361, 9), (1361, 515)])
def test_few_and_many_tubes(n, ntubes, prec):
    print(f"[fft] n3={n} {ntubes} tubes {prec}", flush=True)
    rng = np.random.default_rng(n + ntubes)
    dt, ulp = (np.float64, 0.0) if prec == "f64" else (np.float32, 2.0 ** -24)
    X = rng.standard_normal((ntubes, n)).astype(dt)
    ref = np.fft.rfft(X.astype(np.float64), axis=1).T
    bound = 8 * n * 2.0 ** -53 * np.abs(X).sum(axis=1).max()
    got = host(api.diag_fft_r2c(torch.tensor(X, device="cuda"))).astype(np.complex128)
    assert np.all(np.abs(got - ref) <= bound + 2 * ulp * np.abs(ref))
    S = (rng.standard_normal(ref.shape) + 1j * rng.standard_normal(ref.shape)).astype(np.complex64 if ulp else np.complex128)
    T = S.astype(np.complex128)
    T[0].imag = 0
    if n % 2 == 0:
        T[n // 2].imag = 0
    back = np.fft.irfft(T, n, axis=0).T
    bound = 8 * n * 2.0 ** -53 * 2 * np.abs(T).sum(axis=0).max() / n
    got = host(api.diag_fft_c2r(torch.tensor(S, device="cuda"), n)).astype(np.float64)
    assert np.all(np.abs(got - back) <= bound + 2 * ulp * np.abs(back))
