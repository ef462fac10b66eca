"""Matrix-vector products of the smallest operators (one launch): one below, at and above groups of four
rows, one to three modes, several terms, right-hand sides on both sides of the rule's edges, in place.

The reference is the float64 oracle; the bound is the forward error of nested dot products,
sum_k (n_k + J + 3) eps |K1| (x) .. |x| entry by entry, as for the mode products.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import kron

pytestmark = pytest.mark.gpu

CASES = [((1,), 1, 1), ((5,), 2, 512), ((1, 1), 1, 2), ((3, 4), 3, 513), ((7, 9), 1, 5), ((50, 8), 1, 3), ((40, 40), 1, 2),
         ((41, 40), 1, 2), ((30, 40), 1, 2), ((2, 3, 5), 4, 7), ((12, 10, 14), 1, 1), ((8, 8, 8), 4, 3), ((1, 17, 3), 2, 2),
         ((16, 16, 16), 1, 63), ((16, 16, 16), 1, 64), ((20, 20, 6), 2, 64), ((4, 1, 60), 1, 2)]


@pytest.mark.parametrize("prec,eps", [("fp64", 2.0 ** -53), ("fp32", 2.0 ** -24)])
@pytest.mark.parametrize("dims,J,nrhs", CASES, ids=str)
def test_products(dims, J, nrhs, prec, eps):
    import torch
    from gpu_util import make_op, pack, unpack
    rng = np.random.default_rng(sum(dims) + 5 * J + nrhs)
    s = wl.random_system(rng, dims, nterms=J, diag=J != 2, sigma2=0.3)
    s.factors = [[f + 0.05 * rng.standard_normal(f.shape) for f in row] for row in s.factors]    # not symmetric
    B = rng.standard_normal((nrhs, s.n))
    op = make_op([s], prec=prec)
    x = pack([B])
    if prec == "fp32":
        x = x.to(torch.float32)
        B = x.cpu().numpy().astype(np.float64).reshape(B.shape)
    y = unpack(op.matvec(x, nrhs), [s], nrhs)[0]
    ref = kron.mvm(s.factors, B, s.sigma2, s.diag)
    size = kron.mvm([[np.abs(k) for k in row] for row in s.factors], np.abs(B), s.sigma2, s.diag)
    bound = (sum(dims) + len(dims) * (J + 3)) * eps * size
    assert np.all(np.abs(y - ref) <= bound), float(np.max(np.abs(y - ref) / bound))
    z = op.matvec_noalloc(x, x, nrhs)                        # in place
    assert np.array_equal(unpack(z, [s], nrhs)[0], y)
    op.close()
