"""Factor gradients at the edges of the gradient product's tiles (32, 64, 128), slices (16) and chunks.

The gradient of the library's own lambda against the oracle's closed forms of the same lambda and x;
the bound is the forward error of nested sums entry by entry: (inner terms + mode sizes + 8) eps times
the same contraction of absolute values.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import grad

pytestmark = pytest.mark.gpu

SHAPES = [((1,), 1), ((5,), 2), ((1, 3), 1), ((31, 16), 2), ((33, 15), 3), ((63, 17), 1), ((64, 2), 4), ((65, 130), 2),
          ((3, 31, 33), 2), ((17, 1, 64), 3), ((129, 5, 2), 2), ((40, 260), 5), ((255, 33), 9), ((260, 1030), 17),
          ((1030, 260), 17)]


@pytest.mark.parametrize("dims,nrhs", SHAPES, ids=str)
def test_factor_gradients(dims, nrhs):
    from gpu_util import make_op, pack, unpack
    rng = np.random.default_rng(sum(dims) + nrhs)
    s = wl.random_system(rng, dims, sigma2=1.0, diag=True)
    X = rng.standard_normal((nrhs, s.n))
    W = rng.standard_normal((nrhs, s.n))
    op = make_op([s], prec="fp64")
    Lam, dfac, ddiag, ds2, _ = op.solve_backward(pack([X]), pack([W]), nrhs, tol=1e-2, max_iters=50, prec="fp64")
    Lam = unpack(Lam, [s], nrhs)[0]
    ref = grad.grad_kron(s.factors, X, Lam, True)
    size = grad.grad_kron([[np.abs(k) for k in row] for row in s.factors], np.abs(X), np.abs(Lam), True)
    eps = 2.0 ** -53

    def close(got, want, mag, terms):
        bound = (terms + sum(dims) + 8) * eps * np.abs(mag)
        assert np.all(np.abs(got - want) <= bound), float(np.max(np.abs(got - want) / bound))
    for k, m in enumerate(dims):
        close(dfac[0][0][k].cpu().numpy(), ref[0][0][k], size[0][0][k], nrhs * s.n // m)
    close(ddiag[0].cpu().numpy(), ref[1], size[1], nrhs)
    close(float(ds2[0]), ref[2], size[2], nrhs * s.n)
    op.close()
