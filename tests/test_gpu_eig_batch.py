"""Batched Jacobi decomposition of factors that fit a workgroup's LDS (up to 140 points): sixteen-row
edges, odd sizes (an idle player), both sides of the size limit, mixed batches and extreme scales.

Reference: the oracle's Cholesky solve; bounds: 50 kappa eps forward (the decomposition and the two
transforms are backward stable), 1e-12 in the residual (kappa is at most 1e4 here).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import direct, kron

pytestmark = pytest.mark.gpu


def _check(systems, nrhs=2):
    from gpu_util import make_op, pack, unpack
    rng = np.random.default_rng(9)
    Bs = [rng.standard_normal((nrhs, s.n)) for s in systems]
    op = make_op(systems, prec="fp64")
    for s, B, X in zip(systems, Bs, unpack(op.eig_solve(pack(Bs), nrhs), systems, nrhs)):
        ref = direct.cholesky_solve(s.factors, B, s.sigma2)
        kappa = direct.condition_number(s.factors[0], s.sigma2)
        assert np.linalg.norm(X - ref) <= max(1e-12, 50 * kappa * 2.2e-16) * np.linalg.norm(ref)
        assert np.all(kron.relres(s.factors, X, B, s.sigma2) <= 1e-12)
    op.close()


@pytest.mark.parametrize("dims", [(1, 2), (2, 3), (15, 16), (17, 33), (64, 9), (65, 5), (128, 3), (129, 2),
                                  (139, 4), (140, 4), (141, 4)], ids=str)
def test_sizes(dims):
    rng = np.random.default_rng(sum(dims))
    _check([wl.random_system(rng, dims, sigma2=0.4, kind=k) for k in ("wishart", "rbf")])


def test_batch_on_both_sides_of_the_limit():
    rng = np.random.default_rng(4)
    _check([wl.random_system(rng, d, sigma2=0.3) for d in ((7,), (141, 2), (3, 4, 5), (40, 30), (2, 150), (1, 1))])


def test_scaled_factors():
    """Column norms of 1e-70 and 1e70: the rotation's squares would leave the range unscaled."""
    rng = np.random.default_rng(5)
    s = wl.random_system(rng, (20, 24), sigma2=0.2)
    s.factors = [[s.factors[0][0] * 1e-70, s.factors[0][1] * 1e70]]
    _check([s])


@pytest.mark.parametrize("dims", [(31, 3, 11), (32, 5, 7), (33, 1, 31), (2, 33, 33), (5, 31, 4), (33, 32), (3, 65)],
                         ids=str)
def test_division_in_the_last_product(dims):
    """The eigenvalues of two and three modes at the edges of the last product's tiles."""
    rng = np.random.default_rng(sum(dims) + 1)
    _check([wl.random_system(rng, dims, sigma2=0.4)], nrhs=3)
