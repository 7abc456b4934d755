"""Smoothing steps whose Gram sums (§5.3) go through the one-block pre-reduction: more blocks
of the producing pass than the handle's block cap (one right-hand side), or than consumers of
a batch read themselves.

Blocks of the producers here (a cap of 64, and for the batch of nine consumers that read 64):
level 0 on 256 intervals 168, on 512 intervals 200, the FP64 product operator of level 1 on 128
intervals 99 (FP32 at most 64, not pre-reduced), the batch 72 on level 1."""
import numpy as np
import pytest

import oracle as O
from paper_2308_13476_amd import workloads as W
from tests import extended as E
from tests.gpu_common import require_gpu, to_gpu, to_np

pytestmark = pytest.mark.gpu


# rough residuals: the sums of all blocks matter alike. Bound: three times the distance of the
# oracle's step of the same precision from the step in extended precision, and eight units.
@pytest.mark.parametrize("n,level,env,batch", [(256, 0, {"HELMG_MAX_BLOCKS": "64"}, 1),
                                               (512, 0, {"HELMG_MAX_BLOCKS": "64"}, 1),
                                               (256, 1, {"HELMG_MAX_BLOCKS": "64", "HELMG_L1_PRODUCT": "2"}, 1),
                                               (256, 1, {}, 9)])
def test_steps_with_prereduced_sums(n, level, env, batch, monkeypatch):
    require_gpu()
    from paper_2308_13476_amd.solver import Solver
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    k2 = W.random_k2(n, 21, 0.1 * n, 0.25 * n)
    H = O.build_hierarchy(k2, 1.0 / n, 4.0 / n)
    S = Solver(to_gpu(k2), 1.0 / n, 4.0 / n, max_batch=batch, precision="fp32_refined")
    m = H.n[level] + 1
    f = W.random_complex((batch, m, m), 60 + level)
    M = E.Matrix(H.A[level])
    for dtype, unit in ((np.complex128, 2.0 ** -53), (np.complex64, 2.0 ** -24)):
        g = f.astype(dtype)
        got = to_np(S.smooth(level, to_gpu(np.zeros_like(g)), to_gpu(g), "gmres",
                             precision="fp64" if dtype == np.complex128 else "fp32_refined"))
        for b in range(0, batch, 4):
            r = g[b].ravel()
            exact = E.gmres_step(M, np.zeros(r.size, E.LD), r.astype(E.LD))
            ref = O.gmres_step(H.A[level].astype(dtype), np.zeros_like(r), r, breakdown=1e-14)
            bound = 3 * E.distance(ref, exact) + 8 * unit
            assert E.distance(got[b], exact) <= bound, (dtype, b, E.distance(got[b], exact), E.distance(ref, exact))
