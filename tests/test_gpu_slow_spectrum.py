"""FP64 calls on Fourier slices whose singular values fall slowly and far: no
two neighbours are a factor of sqrt(1.5) apart, so the small SVD has no gap to
split at, and sigma_k lies below the 3e-5 sigma_0 at which its second pass would
begin.  Every one of the k components comes back.

Tolerances, with u = 2^-53 and m columns of the basis.  The eigenvalues of the
m x m Gram carry at most about m u sigma_0^2, so sigma_j^2 (against the same
method with numpy's QR and SVD) is held to 4 m u sigma_0^2, and the squared error
of X_hat to that of the best rank-k tensor (times 1.01 for the random basis)
plus k times that.  Eigenvectors of eigenvalues 1e-9 sigma_0^2 apart may carry
2e-7 of each other: U^H U = I to 1e-6."""
import numpy as np
import pytest
import torch

from tests.gpu_util import dev, host, load_api

pytestmark = pytest.mark.gpu
api = load_api()

N1, N2, N3 = 240, 250, 3
# (spectrum, k, b, q): 1e-6 and 1e-8 at index k, and the ratio 0.85
CASES = [(lambda j: 1e-6 ** (j / 80), 80, 90, 1), (lambda j: 1e-8 ** (j / 100), 100, 110, 1), (lambda j: 0.85 ** j, 80, 84, 1)]


def tensor(s, seed):
    rng = np.random.default_rng(seed)
    X = np.empty((N3 // 2 + 1, N1, N2), complex)
    for f in range(len(X)):
        u, v = (np.linalg.qr(rng.standard_normal((n, len(s))) + (f > 0) * 1j * rng.standard_normal((n, len(s))))[0]
                for n in (N1, N2))
        X[f] = (u * s) @ v.conj().T
    return np.fft.irfft(X, N3, axis=0).transpose(1, 2, 0).copy()


def basis(a, w, q, power):
    x = [np.linalg.qr(a @ w)[0]]
    for _ in range(q):
        y = a.conj().T @ x[-1]
        y = a @ (np.linalg.qr(y)[0] if power else y)
        if not power:
            p = np.concatenate(x, axis=1)
            for _ in range(2):
                y = y - p @ (p.conj().T @ y)
        x.append(np.linalg.qr(y)[0])
    return x[-1] if power else np.linalg.qr(np.concatenate(x, axis=1))[0]


def check(A, s, k, m, U, S, V, ref, label):
    Uf, Sf, Vf = (np.fft.fft(host(x), axis=a)[..., :2] for x, a in ((U, 2), (S, 1), (V, 2)))
    level = 4 * m * 2.0 ** -53 * s[0] ** 2
    Af = np.fft.fft(A, axis=2)
    for f in range(2):
        u, sv, v = Uf[:, :, f], Sf[:, f].real, Vf[:, :, f]
        err = np.linalg.norm((u * sv) @ v.conj().T - Af[:, :, f])
        best = np.linalg.norm(s[k:])
        print(f"[slow] {label} slice {f}: sigma_k {sv[-1]:.2e} ({s[k - 1]:.2e}) error {err:.2e} best {best:.2e} "
              f"U^H U {np.max(np.abs(u.conj().T @ u - np.eye(k))):.1e}", flush=True)
        assert np.all(sv > 0)
        assert np.max(np.abs(sv ** 2 - ref[f][:k] ** 2)) <= level
        assert err ** 2 <= (1.01 * best) ** 2 + k * level
        assert np.max(np.abs(u.conj().T @ u - np.eye(k))) <= 1e-6
        assert np.max(np.abs(np.linalg.norm(v, axis=0) - 1)) <= 1e-6


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("method", ["rbk", "power", "ritz"])
def test_every_component_comes_back(case, method):
    law, k, b, q = CASES[case]
    s = law(np.arange(N1, dtype=float))
    A = tensor(s, 3 + case)
    w = np.random.default_rng(7).standard_normal((N2, b, N3))
    Af, wf = np.fft.fft(A, axis=2), np.fft.fft(w, axis=2)
    ref = []
    for f in range(2):
        x = basis(Af[:, :, f], wf[:, :, f], q, method == "power")
        ref.append(np.linalg.svd(x.conj().T @ Af[:, :, f], compute_uv=False))
    m = b if method == "power" else b * (q + 1)
    if method == "ritz":
        Q, U, S, V = api.tsvd_rbk_ritz(dev(A), dev(w), k, b, q, "f64")
        Qf = np.fft.fft(host(Q), axis=2)
        for f in range(2):
            assert np.max(np.abs(Qf[:, :, f].conj().T @ Qf[:, :, f] - np.eye(b))) <= 1e-6
    else:
        ws = api.workspace(N1, N2, N3, k, b, q, "f64", "approx" if method == "rbk" else "power_approx", "cuda")
        U, S, V, _ = (api.tsvd_rbk_approx if method == "rbk" else api.tsvd_power_approx)(
            dev(A), dev(w), k, b, q, "f64", ws=ws)
        info = api.read_info(ws)
        assert info["eig_noconv"] == 0 and info["nonfinite"] == 0
    check(A, s, k, m, U, S, V, ref, f"case {case} {method}")
