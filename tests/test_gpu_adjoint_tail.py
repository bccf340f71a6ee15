"""The FP32 adjoint of the projection and of the truncation at the gradient's
parity bound (1e-4 of its norm) against the FP64 adjoint of the same inputs: at
sizes with many K splits, at slices narrower than a tile, and with so many
slices (200 and 257 of three tiles) that the last round of tiles is split along K
and added to the block that is already there."""
import pytest
import torch

from tests.gpu_util import load_api

pytestmark = pytest.mark.gpu
api = load_api()


@pytest.mark.parametrize("n1,n2,n3,b,q", [(400, 300, 3, 16, 1), (300, 520, 3, 9, 2), (130, 1100, 3, 7, 0), (1100, 97, 3, 40, 1),
                                          (260, 270, 398, 16, 1), (300, 260, 512, 7, 2), (33, 300, 40, 5, 1)])
def test_adjoint_fp32(n1, n2, n3, b, q):
    print(f"[adjoint] {n1} x {n2} x {n3}, b={b}, q={q}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n1 + b)
    A, G, W = (torch.randn(s, dtype=torch.float32, device="cuda", generator=g)
               for s in ((n1, n2, n3), (n1, n2, n3), (n2, b, n3)))
    for op in ("proj", "approx"):
        out = []
        for dt, prec in ((torch.float64, "f64"), (torch.float32, "f32")):
            a, o, c = A.to(dt), W.to(dt), G.to(dt)
            d = (api.tsvd_proj_backward(a, o, c, b, q, prec) if op == "proj" else
                 api.tsvd_rbk_approx_backward(a, o, c, max(b // 2, 1), b, q, prec))
            out.append(d.double())
        e = float((out[1] - out[0]).norm() / out[0].norm())
        print(f"[adjoint]   {op} {e:.1e}", flush=True)
        assert e <= 1e-4
