"""The dense coarse end of the cycle (AH_TAIL_MAX rows) against the same
hierarchy walked level by level with grid-wide kernels (AH_TAIL_MAX=0): odd
sizes, one or several levels inside it, vectors that leave LDS room for two
columns per workgroup or for one, level 0 inside it, one and three sweeps,
damped sweeps, forward and transposed, FP64 and FP32 cycles.

Tolerances: both form the same products in FP64 in other orders, 1e-12
relative; the walk of the FP32 cycle rounds to FP32 on every level, 1e-5."""
import numpy as np
import pytest
import torch

from workloads import square_tri_mesh, kuhn_cube_mesh
from workloads.problems import C1Advection1D, SmoothPlusFront
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def systems():
    cache = {}

    def get(kind, n, p):
        if (kind, n, p) not in cache:
            v, c = square_tri_mesh(n) if kind == "square" else kuhn_cube_mesh(n)
            prob = C1Advection1D(1e-4) if kind == "square" else SmoothPlusFront(1e-3, width=0.1)
            cache[kind, n, p] = gpu_system(v, c, prob, p)
        return cache[kind, n, p]
    return get


@pytest.mark.parametrize("kind,n,p,end,kw", [
    ("square", 5, 1, 2048, {}),                       # level 0 inside
    ("square", 9, 2, 2048, {"max_coarse": 5}),
    ("square", 31, 1, 2048, {"max_coarse": 1}),
    ("square", 31, 1, 2048, {"relax": 1}),
    ("square", 31, 1, 2048, {"omega": 0.7}),
    ("square", 40, 2, 8192, {}),                      # one column per workgroup
    ("cube", 5, 1, 2048, {"block_air": 1}),
    ("cube", 7, 1, 301, {"max_coarse": 17}),
    ("cube", 6, 1, 2048, {"relax": 2}),
    ("cube", 3, 2, 2048, {"theta": 0.5, "theta_r": 0.25})])
def test_dense_end_equals_the_walk(systems, monkeypatch, kind, n, p, end, kw):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, p, end, kw, flush=True)
    s = systems(kind, n, p)
    r = torch.as_tensor(np.random.default_rng(1).standard_normal(s.n), device="cuda")
    got = {}
    for e in (end, 0):
        monkeypatch.setenv("AH_TAIL_MAX", str(e))
        h = Hierarchy(s, adjoint=1, fp32_cycle=1, **kw)
        got[e] = [h.vcycle(r, precision=q, transpose=t) for q in (0, 1) for t in (False, True)]
    for k, (a, b) in enumerate(zip(got[end], got[0])):
        tol = 1e-12 if k < 2 else 1e-5
        assert float((a - b).norm()) <= tol * float(b.norm()), (k, float((a - b).norm() / b.norm()))
