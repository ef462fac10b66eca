"""Routes of FP32 three-mode solves below 64-wide modes: the persistent CG with and without host checks alike
(the same result bit for bit), and the separate kernels once a group barrier has timed out.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import kron

pytestmark = pytest.mark.gpu


def test_one_route_with_and_without_host_checks():
    from gpu_util import infos, make_op, pack, unpack
    rng = np.random.default_rng(7)
    dims, nrhs = (48, 40, 56), 8
    s = wl.System(factors=[[wl.wishart_factor(rng, m, shift=0.3) for m in dims]], sigma2=0.2, diag=None)
    B = rng.standard_normal((nrhs, s.n))
    op = make_op([s], prec="fp32")
    out = []
    for every in (0, 32):
        op.profile_enable(True)
        X, info = op.solve(pack([B]), nrhs, tol=1e-8, max_iters=320, inner_tol=0.1, check_every=every)
        assert op.profile_read("cg_fused")[1] > 0 and op.profile_read("contract_last")[1] == 0
        out.append((unpack(X, [s], nrhs)[0], [(i["status"], i["iters"]) for i in infos(info, nrhs)]))
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]
    op.close()


@pytest.mark.parametrize("refine", ["reliable", "restart"])
@pytest.mark.parametrize("warm", [False, True])
def test_time_out_falls_back(refine, warm):
    """A group barrier that gives up (its polls limited to one; every block still leaves the launch) hands
    the solve to the separate kernels, and so do the solves that follow."""
    import ctypes
    import torch
    from gpu_util import infos, make_op, pack, unpack
    rng = np.random.default_rng(11)
    dims, nrhs = (48, 40, 56), 8
    s = wl.System(factors=[[wl.wishart_factor(rng, m, shift=0.3) for m in dims]], sigma2=0.2, diag=None)
    B = rng.standard_normal((nrhs, s.n))
    op = make_op([s], prec="fp32")
    op.lib.cola_internal_fused_spin_limit.argtypes = [ctypes.c_void_p, ctypes.c_uint32]
    assert op.lib.cola_internal_fused_spin_limit(op.handle, 1) == 0
    op.profile_enable(True)
    kw = dict(tol=1e-9, max_iters=2000, inner_tol=0.1, refine=refine)
    if warm:
        kw["x0"] = pack([0.1 * B])
    launches = []
    for _ in range(2):
        X, info = op.solve(pack([B]), nrhs, **kw)
        torch.cuda.synchronize()
        launches.append(op.profile_read("cg_fused")[1])
        assert op.profile_read("contract_last")[1] > 0
        rr = kron.relres(s.factors, unpack(X, [s], nrhs)[0], B, s.sigma2)
        assert all(i["status"] == 0 for i in infos(info, nrhs)) and np.all(rr <= 1e-9), rr
    # a chunk or two before the host knew, and the second solve does not try the engine again
    assert 1 <= launches[0] <= 2 and launches[1] == launches[0], launches
    op.close()
