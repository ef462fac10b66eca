"""Mode products in FP64 and FP32 at the edges of their tiles, slices and vectors.

Mode sizes one below, at and above the tile edges (32, 64, 96, 128), the k slices (16 in FP64, 32 in
FP32) and the 16-byte vectors (2 and 4 elements), down to inputs of fewer elements than one vector.
The reference is the float64 oracle; the bound is the forward error of nested dot products,
sum_k (n_k + J + 3) eps |K1| (x) .. |x| entry by entry (each mode product of n_k terms, the sum over
J terms, the diagonal term), with eps the rounding unit of the working precision plus that of the
factors' conversion.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import kron

pytestmark = pytest.mark.gpu

SHAPES = [(1,), (3,), (1, 1), (1, 2), (2, 1), (3, 1), (5, 1, 3), (15, 17), (16, 31, 2), (33, 95), (96, 32), (97, 129),
          (128, 64, 3), (127, 65), (2, 257), (257, 2), (31, 63, 33), (95, 70, 17)]


@pytest.mark.parametrize("prec,eps", [("fp64", 2.0 ** -53), ("fp32", 2.0 ** -24)])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_products_at_tile_edges(shape, prec, eps):
    import torch
    from gpu_util import make_op, pack, unpack
    rng = np.random.default_rng(sum(shape) + 7 * len(shape))
    J, nrhs = (2, 3) if np.prod(shape) > 4 else (1, 1)
    s = wl.random_system(rng, shape, nterms=J, diag=True, sigma2=0.3)
    s.factors = [[f + 0.05 * rng.standard_normal(f.shape) for f in row] for row in s.factors]    # not symmetric
    B = rng.standard_normal((nrhs, s.n))
    op = make_op([s], prec=prec)
    for name in ("slab", "gemm64", "gemm3"):
        op.set_engine(name, False)
    x = pack([B])
    if prec == "fp32":
        x = x.to(torch.float32)
        B = x.cpu().numpy().astype(np.float64).reshape(B.shape)
    y = unpack(op.matvec(x, nrhs), [s], nrhs)[0]
    ref = kron.mvm(s.factors, B, s.sigma2, s.diag)
    size = kron.mvm([[np.abs(k) for k in row] for row in s.factors], np.abs(B), s.sigma2, s.diag)
    bound = (sum(shape) + len(shape) * (J + 3)) * eps * size
    assert np.all(np.abs(y - ref) <= bound), float(np.max(np.abs(y - ref) / bound))
    op.close()


@pytest.mark.parametrize("shape", [(97, 33), (33, 65, 17), (1, 70)], ids=str)
def test_solve_on_odd_modes(shape):
    """The direction, CG and residual epilogues on partial tiles: the FP64 residual at the end of an
    FP64 solve to 1e-11 (recursion and true residual agree to rounding at this condition)."""
    from gpu_util import infos, make_op, pack, unpack
    rng = np.random.default_rng(3)
    s = wl.random_system(rng, shape, nterms=2, diag=True, sigma2=0.5)
    B = rng.standard_normal((3, s.n))
    op = make_op([s], prec="fp64")
    op.set_engine("slab", False)
    X, info = op.solve(pack([B]), 3, tol=1e-11, max_iters=2000)
    rr = kron.relres(s.factors, unpack(X, [s], 3)[0], B, s.sigma2, s.diag)
    assert all(r["status"] == 0 for r in infos(info, 3)) and np.all(rr <= 2e-11), rr
    op.close()
