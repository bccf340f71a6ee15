"""The FP32 adjoint of the projection at sizes where its slice products are cut
along K (also into the block that they are added to) and its gradient is one
product over one, two or three pairs of factors, against the FP64 adjoint of
the same inputs (checked against the oracle elsewhere).  The slices are
Gaussian; the FP32 gradient carries the rounding of products over up to 1100
terms through subspaces of condition below 100: tolerance 100 x 1000 roundings
of 2^-24, relative to the gradient's norm."""
import numpy as np
import pytest
import torch

from tests.gpu_util import host, load_api

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("n1,n2", [(400, 300), (300, 520), (130, 1100), (1100, 97), (257, 272)])
@pytest.mark.parametrize("b,q", [(7, 0), (16, 1), (9, 2), (40, 1)])
def test_adjoint_split(n1, n2, b, q):
    print(f"[adjoint] {n1} x {n2}, b={b}, q={q}", flush=True)
    rng = np.random.default_rng(n1 + b)
    A, G, W = (rng.standard_normal(s).astype(np.float32) for s in ((n1, n2, 3), (n1, n2, 3), (n2, b, 3)))
    out = []
    for dt, prec in ((torch.float64, "f64"), (torch.float32, "f32")):
        a, g, w = (torch.tensor(x, dtype=dt, device="cuda") for x in (A, G, W))
        out.append(host(api.tsvd_proj_backward(a, w, g, b, q, prec)).astype(np.float64))
    assert np.linalg.norm(out[1] - out[0]) <= 1e5 * 2.0 ** -24 * np.linalg.norm(out[0])
