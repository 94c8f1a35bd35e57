"""A zero right-hand side ends the solve at once; like every other solve it
returns with its stream idle, so a solve on another stream may use the shared
workspace next and gives what it gives alone, bit for bit."""
import numpy as np
import pytest
import torch

from workloads import kuhn_cube_mesh
from workloads.problems import SmoothPlusFront
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(noalloc=True, restart=20), dict(restart=20), dict(method=1)])
@pytest.mark.parametrize("delayed", [False, True])
def test_returns_idle_and_leaves_the_next_solve_alone(monkeypatch, kw, delayed):
    from paper_2010_11130_amd import Hierarchy
    print("case", kw, delayed, flush=True)
    monkeypatch.setenv("AH_DCGS_MIN", "0" if delayed else "1000000000")
    v, c = kuhn_cube_mesh(12)
    s = gpu_system(v, c, SmoothPlusFront(1e-3, width=0.1), 1)
    h = Hierarchy(s)
    zero = torch.zeros(s.n, dtype=torch.float64, device="cuda")
    rhs = torch.as_tensor(np.random.default_rng(3).standard_normal(s.n), device="cuda")
    outs = [torch.full_like(rhs, np.nan) for _ in range(3)]
    ref, info = h.solve(rhs, out=outs[0], tol=1e-9, **kw)
    assert info["converged"]
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(10):
        with torch.cuda.stream(a):
            x, info = h.solve(zero, out=outs[1], tol=1e-9, **kw)
            assert a.query() and info["converged"] and info["iters"] == 0
        with torch.cuda.stream(b):
            y, info = h.solve(rhs, out=outs[2], tol=1e-9, **kw)
        torch.cuda.synchronize()
        assert float(x.abs().max()) == 0.0 and torch.equal(y, ref)
        outs[1].fill_(np.nan)
        outs[2].fill_(np.nan)
        torch.cuda.synchronize()
