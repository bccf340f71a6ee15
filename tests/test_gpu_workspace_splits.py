"""FP32 calls with few slices, whose Krylov products take more K splits, and more
scratch for them, where the workspace allows.

A workspace of the size that served the call with the narrow splits is accepted
and gives the same result to FP32 (X_hat to 2 x 1e-5, the gradient of a Gaussian
tensor to 2 x 1e-4: the bounds of the parity tests for two FP32 results).  P(A) of
these tensors depends on directions that FP32 holds to a few digits; its error
against the FP64 call is at most twice that with the full workspace.
Calls that run the same launches give the same bits: tsvd_rbk, tsvd_rbk_approx, Alg.
1 with q = 0 and the entry point that allocates nothing, also where that one's
static scratch holds the narrow splits only (285 x 223 x 30)."""
import numpy as np
import pytest
import torch

from paper_2504_04989_amd import inputs
from tests.gpu_util import dev, host, load_api, rel_f

pytestmark = pytest.mark.gpu
api = load_api()

# (n1, n2, n3, k, b, q) and bytes by operation, with the narrow splits
SIZES = {
    (300, 2000, 4, 20, 30, 2): dict(rbk=31084544, approx=31228672, power=24174592, power_approx=24318720, proj=29328640,
                                    proj_bwd=65617152, literal=31228672, ritz=32686592, complete2=51165184,
                                    complete1=44255232, approx_bwd=76676096),
    (512, 768, 3, 50, 60, 2): dict(rbk=22823936, approx=23233536, power=13949440, power_approx=14359040, proj=20061952,
                                   proj_bwd=39526144, literal=23233536, ritz=23699968, complete2=33439488,
                                   complete1=24564992, approx_bwd=50284288),
}


def call(op, A, G, shape, seed, ws):
    k, b, q = shape[3:]
    if op in ("rbk", "power"):
        U, S, V = (api.tsvd_rbk if op == "rbk" else api.tsvd_power)(A, seed, k, b, q, "f32", ws=ws)
        Uf, Sf, Vf = (np.fft.fft(host(x).astype(np.float64), axis=-1) for x in (U, S, V))
        return np.einsum("ijf,jf,kjf->ikf", Uf, Sf, Vf.conj())
    if op == "proj":
        return host(api.tsvd_proj(A, seed, b, q, "f32", ws=ws)).astype(np.float64)
    if op == "proj_bwd":
        return host(api.tsvd_proj_backward(A, seed, G, b, q, "f32", ws=ws)).astype(np.float64)
    if op == "approx_bwd":
        return host(api.tsvd_rbk_approx_backward(A, seed, G, k, b, q, "f32", ws=ws)).astype(np.float64)
    if op in ("complete2", "complete1"):
        mask = torch.ones_like(A, dtype=torch.bool)
        mask[::3, ::2] = False
        return host(api.tsvd_complete(A, mask, seed, k, b, q, 2, int(op[-1]), "f32", ws=ws)).astype(np.float64)
    if op == "ritz":
        return host(api.tsvd_rbk_ritz(A, seed, k, b, q, "f32", ws=ws)[2]).astype(np.float64)
    fn = {"approx": api.tsvd_rbk_approx, "power_approx": api.tsvd_power_approx, "literal": api.tsvd_rbk_literal}[op]
    return host(fn(A, seed, k, b, q, "f32", ws=ws)[3]).astype(np.float64)


@pytest.mark.parametrize("shape", list(SIZES))
@pytest.mark.parametrize("op", list(SIZES[(300, 2000, 4, 20, 30, 2)]))
def test_workspace_of_the_narrow_splits(shape, op):
    n1, n2, n3, k, b, q = shape
    size = SIZES[shape][op]
    print(f"[splits] {op} {shape}: {size} bytes of {api.workspace_bytes(*shape, 'f32', op)}", flush=True)
    if op in ("proj_bwd", "approx_bwd"):
        A = dev(inputs.random_tensor((n1, n2, n3), 3), torch.float32)
    elif op == "literal":  # (raw Krylov blocks want a flat spectrum)
        A = dev(inputs.lowrank_tensor(n1, n2, n3, k, ("geom", 0.999), 1e-4, seed=3), torch.float32)
    else:
        A = dev(inputs.lowrank_tensor(n1, n2, n3, k + 20, ("geom", 0.9), 1e-3, seed=3), torch.float32)
    G = dev(inputs.random_tensor((n1, n2, n3), 4), torch.float32)
    full = call(op, A, G, shape, 9, None)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    less = call(op, A, G, shape, 9, ws)
    torch.cuda.synchronize()
    if op == "proj":
        Om = dev(inputs.omega(n2, b, n3, 9))
        ref = host(api.tsvd_proj(A.double(), Om, b, q, "f64"))
        e, bound = rel_f(less, ref), 2 * rel_f(full, ref)
    else:
        e, bound = rel_f(less, full), 2 * (1e-4 if op.endswith("_bwd") else 1e-5)
    print(f"[splits]   {e:.1e} (bound {bound:.1e})", flush=True)
    assert e <= bound
    with pytest.raises(api.TsvdError) as err:
        call(op, A, G, shape, 9, ws[: size // 2])
    assert err.value.code == api.TSVD_ENOMEM


@pytest.mark.parametrize("n1,n2,n3,k,b", [(512, 768, 3, 50, 60), (300, 2000, 4, 20, 30), (285, 223, 30, 24, 108)])
def test_same_launches_same_bits(n1, n2, n3, k, b):
    print(f"[splits] bits {n1} x {n2} x {n3}, b={b}", flush=True)
    A = dev(inputs.lowrank_tensor(n1, n2, n3, k + 20, ("geom", 0.9), 1e-3, seed=5), torch.float32)
    assert api.workspace_bytes(n1, n2, n3, k, b, 0, "f32", "rbk") <= api.NOALLOC_SCRATCH_BYTES
    ref = api.tsvd_rbk(A, 11, k, b, 0, "f32")
    for other in (api.tsvd_rbk_approx(A, 11, k, b, 0, "f32"), api.tsvd_power(A, 11, k, b, 0, "f32"),
                  api.tsvd_power_approx(A, 11, k, b, 0, "f32"), api.tsvd_rbk_noalloc(A, 11, k, b, 0, "f32")):
        torch.cuda.synchronize()
        for x, y in zip(ref, other):
            assert torch.equal(x, y)
