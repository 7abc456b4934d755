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


# Bound of the tests below: no more than three times as far from the extended result as the
# oracle, which orthogonalises its vectors, is in the same precision (both are rounding that the
# operator amplifies alike; three covers the order of the sums), and eight units of rounding.
def _bound(reference, exact, dtype):
    return 3 * E.distance(reference, exact) + 8 * UNIT[dtype]


UNIT = {np.complex64: 2.0 ** -24, np.complex128: 2.0 ** -53}
BREAKDOWN = {np.complex64: 1e-6, np.complex128: 1e-14}


def _sources(n, k):
    return {"smooth": E.smooth_source(n), "narrow": E.smooth_source(n, width=0.05), "wave": E.smooth_source(n, k),
            "rough": W.random_complex((n + 1, n + 1), 7),
            "mixed": E.smooth_source(n) + 1e-2 * W.random_complex((n + 1, n + 1), 8)}


@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("n,kh", [(64, 0.3), (256, 0.1), (512, 0.02)])
def test_level0_steps_are_as_exact_as_the_oracles(n, kh, dtype):
    require_gpu()
    from paper_2308_13476_amd.solver import Solver
    k2 = W.constant_k2(n, kh * n)
    S = Solver(to_gpu(k2), 1.0 / n, 1.0 / (kh * n), precision="fp32_refined")
    A = O.helmholtz_matrix(k2, 1.0 / n)
    M, A = E.Matrix(A), A.astype(dtype)
    for name, f in _sources(n, kh * n).items():
        f = f.astype(dtype)
        exact = E.gmres_step(M, np.zeros(f.size, E.LD), f.ravel().astype(E.LD))
        ref = O.gmres_step(A, np.zeros(f.size, dtype), f.ravel(), breakdown=BREAKDOWN[dtype])
        got = E.distance(_smooth(S, 0, f), exact)
        assert got <= _bound(ref, exact, dtype), (name, got, E.distance(ref, exact))


# the residual that a step leaves by recurrence is what the next level gets
@pytest.mark.parametrize("n,kh,dtype", [(64, 0.3, np.complex128), (64, 0.3, np.complex64), (128, 0.1, np.complex64),
                                        (256, 0.05, np.complex64)])
def test_cycles_on_a_smooth_source_are_as_exact_as_the_oracles(n, kh, dtype):
    require_gpu()
    from paper_2308_13476_amd.solver import Solver
    k2 = W.constant_k2(n, kh * n)
    H = O.build_hierarchy(k2, 1.0 / n, 1.0 / (kh * n))
    S = Solver(to_gpu(k2), 1.0 / n, 1.0 / (kh * n), precision="fp32_refined")
    f = E.smooth_source(n).astype(dtype)
    exact = E.cycle(H, np.zeros(f.size, E.LD), f.ravel().astype(E.LD), 1, 0)
    fp32 = dtype == np.complex64
    ref = O.cycle(H, 0, np.zeros(f.size, dtype), f.ravel(), O.CycleOptions(smoother="gmres", nu1=1, nu2=0), fp32=fp32)
    got = E.distance(to_np(S.cycle(to_gpu(np.zeros_like(f)), to_gpu(f), smoother="gmres", nu_pre=1, nu_post=0,
                                   precision="fp32_refined" if fp32 else "fp64")), exact)
    assert got <= _bound(ref, exact, dtype), (got, E.distance(ref, exact))


@pytest.mark.parametrize("n,kh,transfer", [(128, 0.3, "bezier"), (256, 0.05, "bezier"), (64, 0.25, "linear")])
def test_fp32_steps_of_stored_levels_are_as_exact_as_the_oracles(n, kh, transfer):
    """Every level below the finest, on rough, smooth and restricted residuals."""
    require_gpu()
    from paper_2308_13476_amd.solver import Solver
    k2 = W.constant_k2(n, kh * n) if kh < 0.1 else W.random_k2(n, 31, 0.4 * kh * n, kh * n)
    H = O.build_hierarchy(k2, 1.0 / n, 1.0 / (kh * n), transfer=transfer)
    S = Solver(to_gpu(k2), 1.0 / n, 1.0 / (kh * n), transfer=transfer, precision="fp32_refined")
    dtype = np.complex64
    given = {"smooth": E.smooth_source(n).ravel(), "rough": W.random_complex((n + 1) ** 2, 7),
             "point": W.point_source_rhs(n, [W.center_node(n)])[0].ravel()}
    for l in range(1, H.levels - 1):
        n_l = H.n[l]
        given = {name: H.R[l - 1] @ (f - H.A[l - 1] @ O.gmres_step(H.A[l - 1], np.zeros_like(f), f))
                 for name, f in given.items()}
        own = {"smooth on the level": E.smooth_source(n_l), "rough on the level": W.random_complex((n_l + 1) ** 2, l)}
        M, A = E.Matrix(H.A[l]), H.A[l].astype(dtype)
        for name, f in {**given, **own}.items():
            f = f.reshape(n_l + 1, n_l + 1).astype(dtype)
            exact = E.gmres_step(M, np.zeros(f.size, E.LD), f.ravel().astype(E.LD))
            ref = O.gmres_step(A, np.zeros(f.size, dtype), f.ravel(), breakdown=BREAKDOWN[dtype])
            got = E.distance(_smooth(S, l, f), exact)
            assert got <= _bound(ref, exact, dtype), (l, name, got, E.distance(ref, exact))
