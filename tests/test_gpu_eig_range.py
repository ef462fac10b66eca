"""Direct solves with factors at the ends of the FP64 range: the batched decomposition scales each factor
by a power of two, so the solve of (a K1) (x) (K2 / a) is that of K1 (x) K2 for any a.

Reference: the oracle's residual, at the bound of the unscaled solves (1e-12; kappa is below 100).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import kron

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("digits", [80, 100, 140, 250], ids=str)
@pytest.mark.parametrize("dims", [(20, 24), (3, 7, 5)], ids=str)
def test_factors_far_from_one(dims, digits):
    from gpu_util import make_op, pack, unpack
    rng = np.random.default_rng(digits + sum(dims))
    s = wl.random_system(rng, dims, sigma2=0.2)
    row = s.factors[0]
    row[0], row[1] = row[0] * 10.0 ** -digits, row[1] * 10.0 ** digits
    B = rng.standard_normal((2, s.n))
    op = make_op([s], prec="fp64")
    X = unpack(op.eig_solve(pack([B]), 2), [s], 2)[0]
    assert np.all(kron.relres(s.factors, X, B, s.sigma2) <= 1e-12)
    op.close()


def test_zero_factor():
    """A zero factor has eigenvalues of zero in any basis: the solve is b / sigma2."""
    from gpu_util import make_op, pack, unpack
    rng = np.random.default_rng(1)
    s = wl.random_system(rng, (6, 5), sigma2=0.5)
    s.factors[0][0] = np.zeros((6, 6))
    B = rng.standard_normal((2, s.n))
    op = make_op([s], prec="fp64")
    X = unpack(op.eig_solve(pack([B]), 2), [s], 2)[0]
    assert np.linalg.norm(X - B / 0.5) <= 1e-13 * np.linalg.norm(B / 0.5)
    op.close()
