"""The persistent fused CG at mode sizes below 64: edges of its 16-wide tiles, vectors cut at the end of
a row, strips cut at the end of a slab, idle quads, one and two slabs per quad.

Solutions are certified by the oracle's FP64 residual at 1e-9; stopped after 40 iterations, the iterate
agrees with the separate kernels up to FP32 rounding of the two reduction orders (1e-4, as for 64-wide
modes).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import kron

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,nrhs,diag", [
    ((16, 16, 16), 1, True), ((17, 15, 33), 6, False), ((64, 63, 64), 6, True), ((16, 64, 1), 5, False),
    ((1, 64, 16), 6, True), ((2, 47, 43), 5, True), ((4, 4, 4), 3, False), ((3, 31, 33), 20, False),
    ((32, 2, 40), 5, True), ((33, 41, 32), 16, False), ((48, 40, 56), 17, True), ((32, 31, 64), 40, False)], ids=str)
def test_modes_below_64(dims, nrhs, diag):
    from gpu_util import infos, make_op, pack, unpack
    rng = np.random.default_rng(sum(dims) + nrhs)
    facs = [wl.wishart_factor(rng, m, shift=0.3) for m in dims]
    s = wl.System(factors=[facs], sigma2=0.2, diag=rng.uniform(0.05, 0.5, size=int(np.prod(dims))) if diag else None)
    B = rng.standard_normal((nrhs, s.n))
    op = make_op([s], prec="fp32")
    op.profile_enable(True)
    X, info = op.solve(pack([B]), nrhs, tol=1e-9, max_iters=3000, inner_tol=0.1)
    assert op.profile_read("cg_fused")[1] > 0 and op.profile_read("slab23")[1] == 0
    op.profile_enable(False)
    rr = kron.relres(s.factors, unpack(X, [s], nrhs)[0], B, s.sigma2, s.diag)
    assert all(i["status"] == 0 for i in infos(info, nrhs)) and np.all(rr <= 1e-9), rr
    kw = dict(tol=1e-14, max_iters=40, inner_tol=0.1)
    Xf, inf_f = op.solve(pack([B]), nrhs, **kw)
    op.set_engine("fused_cg", False)
    Xu, inf_u = op.solve(pack([B]), nrhs, **kw)
    a, b = unpack(Xf, [s], nrhs)[0], unpack(Xu, [s], nrhs)[0]
    assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b)
    op.close()


def test_small_batches_of_large_groups_take_the_separate_kernels():
    from gpu_util import make_op, pack
    rng = np.random.default_rng(2)
    s = wl.random_system(rng, (50, 50, 50), sigma2=0.5)
    op = make_op([s], prec="fp32")
    op.profile_enable(True)
    op.solve(pack([rng.standard_normal((2, s.n))]), 2, tol=1e-5)
    assert op.profile_read("cg_fused")[1] == 0 and op.profile_read("contract_last")[1] > 0
    op.close()
