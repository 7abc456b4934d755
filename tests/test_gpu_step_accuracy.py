"""GMRES(3) smoothing steps of smooth residuals against the same step in extended precision
(§5.3): the basis of such a residual is nearly dependent, and what a step loses there the rough
data of other tests do not show."""
import numpy as np
import pytest

import oracle as O
from paper_2308_13476_amd import workloads as W
from tests import extended as E
from tests.gpu_common import require_gpu, to_gpu, to_np

pytestmark = pytest.mark.gpu


def _smooth(S, l, f):
    f = np.ascontiguousarray(f)
    return to_np(S.smooth(l, to_gpu(np.zeros_like(f)), to_gpu(f), "gmres",
                          precision="fp64" if f.dtype == np.complex128 else "fp32_refined"))


def test_fp64_weights_of_a_smooth_residual():
    """The weights of a step come from the Gram matrix of its powers. On a fine grid at a low
    wavenumber, where |A r| is far below |A| |r|, entries formed from sums that were rounded
    before the shift of the basis was put in lose (shift |r| / |A r|)^2.

    Bound: 32 units of rounding (two applications of ten operations, the weights and the
    sums), amplified as vectors with a shift of 6 / h^2 amplify them."""
    require_gpu()
    from paper_2308_13476_amd.solver import Solver
    n, k = 1024, 20.48
    k2 = W.constant_k2(n, k)
    f = E.smooth_source(n)
    A = E.Matrix(O.helmholtz_matrix(k2, 1.0 / n))
    exact = E.gmres_step(A, np.zeros(f.size, E.LD), f.ravel().astype(E.LD))
    grow = E.amplification(A, f.ravel().astype(E.LD), exact, 6.0 * n * n)
    got = _smooth(Solver(to_gpu(k2), 1.0 / n, 1.0 / k), 0, f)
    assert E.distance(got, exact) <= 32 * 2.0 ** -53 * grow, (E.distance(got, exact), grow)
