"""The scalars of an FGMRES step by copies (AH_POLL=0, the path of a thread without
a pinned buffer) and by the polled flag: the same solves bit for bit, forward
and adjoint, with restarts, a given start, step limits and a zero right-hand
side, in both orthogonalisations."""
import numpy as np
import pytest
import torch

from workloads import square_tri_mesh, kuhn_cube_mesh
from workloads.problems import C1Advection1D, SmoothPlusFront
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n", [("square", 13), ("cube", 6)])     # below and above the one-workgroup step
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("delayed", [False, True])
def test_copies_and_flag(monkeypatch, kind, n, precision, delayed):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, precision, delayed, flush=True)
    monkeypatch.setenv("AH_DCGS_MIN", "0" if delayed else "1000000000")
    v, c = square_tri_mesh(n) if kind == "square" else kuhn_cube_mesh(n)
    s = gpu_system(v, c, C1Advection1D(1e-4) if kind == "square" else SmoothPlusFront(1e-3, width=0.1), 1)
    rhs, x0 = (torch.as_tensor(r, device="cuda") for r in np.random.default_rng(5).standard_normal((2, s.n)))
    got = []
    for poll in ("1", "0"):
        monkeypatch.setenv("AH_POLL", poll)
        h = Hierarchy(s, max_coarse=8, adjoint=1, fp32_cycle=precision)
        kw = dict(tol=1e-9, precision=precision, maxit=500)
        runs = [h.solve(rhs, **kw), h.solve(rhs, x0=x0, restart=4, **kw), h.solve(rhs, noalloc=True, restart=30, **kw),
                h.solve(rhs, tol=1e-9, precision=precision, maxit=3), h.solve(torch.zeros_like(rhs), **kw),
                h.solve_adjoint(rhs, **kw)]
        got.append([(x, {k: i[k] for k in i if k != "t_solve_ms"}) for x, i in runs])
    for (x, i), (y, j) in zip(*got):
        assert torch.equal(x, y) and i == j, (i, j)
    assert got[0][0][1]["converged"] and got[0][3][1]["iters"] == 3
