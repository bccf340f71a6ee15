"""Eigenvalues of graded diagonal matrices, 1 down to 1e-57, in no order, and
exact zeros: each eigenvalue relative to itself, for every number of lanes that
the multisection gives an eigenvalue (64, 16 and 8, by the number of
eigenvalues).  The reduction leaves a diagonal matrix as it is, so the only errors
are the final interval, 2 eps of the eigenvalue, and its midpoint's rounding:
tolerance 4 eps.  A zero is found to 1e-100 of the largest eigenvalue."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("batch", [2, 40, 120])
def test_graded(batch):
    m, k = 62, 60
    print(f"[graded] {batch} slices, {batch * k} eigenvalues", flush=True)
    lam = np.concatenate([3.0 * 10.0 ** -np.arange(58.0), np.zeros(4)])
    G = np.zeros((batch, m, m), complex)
    for f in range(batch):
        G[f] = np.diag(np.random.default_rng(f).permutation(lam))
    got, _, info = api.diag_heig(torch.tensor(G, device="cuda"), k)
    got = host(got)
    assert info["nonfinite"] == 0
    assert np.max(np.abs(got[:, :58] / lam[:58] - 1)) <= 4 * 2.0 ** -52
    assert np.max(np.abs(got[:, 58:])) <= 3e-100
