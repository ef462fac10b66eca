"""Kernels that ordinary small calls no longer reach, each run on a call that does, with the route checked
by the launch classes: the mode products of the smallest operators (the one-launch product takes them up to
512 right-hand sides), their element-wise variant, and the 64 x 64 slab kernel on the static scratch and
in FP64.

Products are held to the float64 oracle by the forward error of nested dot products,
sum_k (n_k + J + 3) eps |K1| (x) .. |x| entry by entry; solves by the oracle's residual.
"""
import ctypes

import numpy as np
import pytest

import workloads as wl
from oracle import kron

pytestmark = pytest.mark.gpu

EPS = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24}
CONTRACT = ("contract_rows", "contract_mid", "contract_last")


def _launches(op, names):
    return sum(op.profile_read(n + suffix)[1] for n in names for suffix in ("", "_fp64"))


def _bound(s, B, shape, J, prec):
    size = kron.mvm([[np.abs(k) for k in row] for row in s.factors], np.abs(B), s.sigma2, s.diag)
    return (sum(shape) + len(shape) * (J + 3)) * EPS[prec] * size


def _input(B, prec):
    import torch
    from gpu_util import pack
    x = pack([B])
    if prec == "fp64":
        return x, B
    x = x.to(torch.float32)
    return x, x.cpu().numpy().astype(np.float64).reshape(B.shape)


# the smallest operators, then column passes with few trailing indices after their last full slice
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(1,), (3,), (1, 1), (1, 2), (2, 1), (3, 1), (5, 1, 3), (15, 17), (16, 31, 2), (33, 1),
                                   (33, 2), (34, 1), (33, 8), (17, 8), (65, 1), (4, 33, 2), (100, 2), (129, 15)], ids=str)
def test_mode_products_of_small_operators(shape, prec):
    from gpu_util import make_op, unpack
    rng = np.random.default_rng(sum(shape) + 11 * len(shape))
    J, nrhs = 2, 513
    s = wl.random_system(rng, shape, nterms=J, diag=True, sigma2=0.3)
    s.factors = [[f + 0.05 * rng.standard_normal(f.shape) for f in row] for row in s.factors]    # not symmetric
    x, B = _input(rng.standard_normal((nrhs, s.n)), prec)
    op = make_op([s], prec=prec)
    op.profile_enable(True)
    y = unpack(op.matvec(x, nrhs), [s], nrhs)[0]
    assert _launches(op, CONTRACT) >= 2 and _launches(op, ("tiny_mvm",)) == 0
    err, bound = np.abs(y - kron.mvm(s.factors, B, s.sigma2, s.diag)), _bound(s, B, shape, J, prec)
    assert np.all(err <= bound), float(np.max(err / bound))
    op.profile_enable(True)                                  # up to 512 right-hand sides: one launch
    x1 = x[:s.n].contiguous()
    y1 = unpack(op.matvec(x1, 1), [s], 1)[0]
    if max(shape) <= 5:
        assert _launches(op, ("tiny_mvm",)) == 1 and _launches(op, CONTRACT) == 0
    err = np.abs(y1 - kron.mvm(s.factors, B[:1], s.sigma2, s.diag))
    assert np.all(err <= bound[:1]), float(np.max(err / bound[:1]))
    op.close()


@pytest.mark.parametrize("shape,prec", [((1,), "fp64"), ((1, 1), "fp64"), ((1, 1, 1), "fp64"), ((1,), "fp32"), ((3,), "fp32"),
                                        ((1, 2), "fp32"), ((2, 1), "fp32"), ((3, 1), "fp32"), ((1, 1, 3), "fp32")], ids=str)
def test_solves_with_fewer_unknowns_than_a_vector(shape, prec):
    """One right-hand side and fewer unknowns than the 16 bytes of one vector, on the separate kernels."""
    from gpu_util import infos, make_op, pack, unpack
    rng = np.random.default_rng(sum(shape))
    s = wl.random_system(rng, shape, nterms=2, diag=True, sigma2=0.5)
    B = rng.standard_normal((1, s.n))
    op = make_op([s], prec=prec)
    for name in ("small64", "resident"):
        op.set_engine(name, False)
    op.profile_enable(True)
    X, info = op.solve(pack([B]), 1, tol=1e-12, max_iters=100, inner_tol=0.1)
    assert _launches(op, CONTRACT) > 0
    rr = kron.relres(s.factors, unpack(X, [s], 1)[0], B, s.sigma2, s.diag)
    assert infos(info, 1)[0]["status"] == 0 and np.all(rr <= 1e-12), rr
    op.close()


def test_slab_kernel_on_the_static_scratch():
    """Two terms of 48 x 64 x 64, three right-hand sides: 144 slabs, the terms' intermediates side by side."""
    import torch
    from paper_2309_03060_amd import _lib as L
    from paper_2309_03060_amd.ops import _stream_ptr
    from gpu_util import make_op, unpack
    rng = np.random.default_rng(5)
    shape, J, nrhs = (48, 64, 64), 2, 3
    s = wl.random_system(rng, shape, nterms=J, diag=True, sigma2=0.2)
    x, B = _input(rng.standard_normal((nrhs, s.n)), "fp32")
    op = make_op([s], prec="fp32")
    y = torch.full_like(x, float("nan"))
    assert op.lib.cola_kron_matvec_noalloc(op.handle, ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(y.data_ptr()), nrhs,
                                           L.COLA_F32, L.COLA_PREC_FP32, ctypes.c_void_p(_stream_ptr())) == 0
    op.profile_enable(True)
    z = op.matvec(x, nrhs)
    assert _launches(op, ("slab23",)) == 1 and torch.equal(y, z)
    err, bound = np.abs(unpack(y, [s], nrhs)[0] - kron.mvm(s.factors, B, s.sigma2, s.diag)), _bound(s, B, shape, J, "fp32")
    assert np.all(err <= bound), float(np.max(err / bound))
    op.close()


@pytest.mark.parametrize("prec,shape,nrhs", [("fp64", (128, 64, 64), 16), ("fp32", (48, 64, 64), 3)], ids=str)
def test_slab_kernel_product_and_solve(prec, shape, nrhs):
    """As many slabs as the rule asks for: the product, and a solve (whose slabs form the direction)."""
    from gpu_util import infos, make_op, pack, unpack
    rng = np.random.default_rng(6)
    s = wl.System(factors=[[wl.wishart_factor(rng, m, shift=0.3) for m in shape] for _ in range(2)], sigma2=0.5, diag=None)
    x, B = _input(rng.standard_normal((nrhs, s.n)), prec)
    op = make_op([s], prec=prec)
    op.set_engine("fused_cg", False)
    op.profile_enable(True)
    y = unpack(op.matvec(x, nrhs), [s], nrhs)[0]
    assert _launches(op, ("slab23",)) == 1 and _launches(op, ("contract_rows", "contract_mid")) == 0
    err, bound = np.abs(y[:3] - kron.mvm(s.factors, B[:3], s.sigma2)), _bound(s, B[:3], shape, 2, prec)
    assert np.all(err <= bound), float(np.max(err / bound))
    op.profile_enable(True)
    X, info = op.solve(pack([B]), nrhs, tol=1e-8, max_iters=400, inner_tol=0.1)
    assert op.profile_read("slab23_fp64" if prec == "fp64" else "slab23")[1] > 0
    rr = kron.relres(s.factors, unpack(X, [s], nrhs)[0][:3], B[:3], s.sigma2)
    assert all(i["status"] == 0 for i in infos(info, nrhs)) and np.all(rr <= 1.01e-8), rr
    op.close()
