"""The coarse tail where its setting is larger than the levels that its threads cover: the
first level of the tail has to be one of at most 34 intervals (§5 V/W cycles)."""
import numpy as np
import pytest

import oracle as O
from paper_2308_13476_amd import workloads as W
from tests.gpu_common import rel, require_gpu, to_gpu, to_np

pytestmark = pytest.mark.gpu


# 40, 20, 10, 5 and 36, 18, 9 intervals below the finest level (1681 and 1369 nodes, more than
# the tail's 1280), 32 (1089 nodes, two per thread) and 24 (625, one per thread)
@pytest.mark.parametrize("n,coarsest", [(80, 5), (160, 5), (72, 9), (128, 4), (96, 6)])
@pytest.mark.parametrize("tail", ["40", "64"])
def test_cycles_with_large_tail_settings(n, coarsest, tail, monkeypatch):
    require_gpu()
    from paper_2308_13476_amd.solver import Solver
    monkeypatch.setenv("HELMG_TAIL_N", tail)
    k2 = W.random_k2(n, 3, 8.0, 20.0)
    H = O.build_hierarchy(k2, 1.0 / n, 0.1, coarsest_n=coarsest)
    S = Solver(to_gpu(k2), 1.0 / n, 0.1, coarsest_n=coarsest, precision="fp32_refined")
    u, f = W.random_complex((1, n + 1, n + 1), 1), W.random_complex((1, n + 1, n + 1), 2)
    for smoother in ("gmres", "jacobi"):
        o = dict(cycle="W", smoother=smoother, nu_pre=1, nu_post=2)
        ref = O.cycle(H, 0, u[0].ravel(), f[0].ravel(), O.CycleOptions(gamma=2, smoother=smoother, nu1=1, nu2=2))
        assert rel(to_np(S.cycle(to_gpu(u), to_gpu(f), **o))[0], ref) <= 1e-10
        low = S.cycle(to_gpu(u.astype(np.complex64)), to_gpu(f.astype(np.complex64)), precision="fp32_refined", **o)
        assert rel(to_np(low)[0], ref) <= 1e-3  # FP32 residuals of rough data
