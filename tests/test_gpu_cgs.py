"""FGMRES, with both orthogonalisations: the step's scalars reach the host through a
polled flag, or by copies where the thread has no pinned buffer; the solve at
the edges of its launch shapes (a handful of unknowns, row counts around a
block, around the step in one workgroup (2048 unknowns, 15 vectors), more
vectors than a combination's coefficient block holds), with a given start, a
zero right-hand side, step limits and restarts.

Tolerances: residuals are recomputed in FP64 from the exported system, twice
the requested tolerance; the two transports run the same kernels, so their
results agree bit for bit."""
import threading

import numpy as np
import pytest
import torch

from workloads import square_tri_mesh, kuhn_cube_mesh
from workloads.problems import C1Advection1D, SmoothPlusFront
from gpu_cases import gpu_system, to_scipy

pytestmark = pytest.mark.gpu


def system(kind, n, p):
    v, c = square_tri_mesh(n) if kind == "square" else kuhn_cube_mesh(n)
    return gpu_system(v, c, C1Advection1D(1e-4) if kind == "square" else SmoothPlusFront(1e-3, width=0.1), p)


def residual(s, x):
    ex = s.export()
    A = to_scipy(ex["rowptr"], ex["col"], ex["val"], s.n)
    b = ex["hhat"].cpu().numpy()
    return np.linalg.norm(b - A @ x.cpu().numpy()) / np.linalg.norm(b)


@pytest.mark.parametrize("kind,n,p", [("square", 1, 1), ("square", 3, 2), ("square", 13, 1), ("square", 18, 1),
                                      ("square", 19, 1), ("square", 40, 1), ("cube", 9, 1)])
@pytest.mark.parametrize("restart,relax", [(100, 0), (4, 0), (300, 1)])
@pytest.mark.parametrize("delayed", [False, True])
def test_solution_and_start(monkeypatch, kind, n, p, restart, relax, delayed):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, p, restart, relax, delayed, flush=True)
    monkeypatch.setenv("AH_DCGS_MIN", "0" if delayed else "1000000000")
    s = system(kind, n, p)
    # one F sweep per level converges slowly: more than 128 vectors in one combination
    h = Hierarchy(s, relax=relax, max_coarse=4, omega=0.5 if relax else 1.0)
    x, info = h.solve(tol=1e-9, restart=restart, maxit=3000)
    assert info["converged"] and residual(s, x) <= 2e-9
    y, again = h.solve(x0=x, tol=1e-9)
    assert again["iters"] == 0 and torch.equal(x, y)
    z, rest = h.solve(x0=0.5 * x, tol=1e-9, restart=restart, maxit=3000)
    assert rest["converged"] and residual(s, z) <= 2e-9


def test_limits_and_zero_rhs():
    from paper_2010_11130_amd import Hierarchy
    s = system("square", 13, 1)
    h = Hierarchy(s, max_coarse=8)
    x, info = h.solve(maxit=0)
    assert not info["converged"] and info["iters"] == 0 and float(x.abs().max()) == 0.0
    x, info = h.solve(maxit=2)
    assert not info["converged"] and info["iters"] == 2 and info["true_relres"] < 1.0
    x, info = h.solve(tol=1.0)
    assert info["converged"] and info["iters"] == 0 and float(x.abs().max()) == 0.0
    x, info = h.solve(torch.zeros(s.n, dtype=torch.float64, device="cuda"))
    assert info["converged"] and float(x.abs().max()) == 0.0


@pytest.mark.parametrize("delayed", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
def test_copied_scalars_give_the_polled_result(monkeypatch, precision, delayed):
    """A thread that has never set anything up has no pinned buffer, and the
    allocation-free solve must not make one."""
    from paper_2010_11130_amd import Hierarchy
    monkeypatch.setenv("AH_DCGS_MIN", "0" if delayed else "1000000000")
    s = system("cube", 4, 1)
    h = Hierarchy(s, fp32_cycle=1)
    kw = dict(noalloc=True, tol=1e-9, restart=30, precision=precision)
    outs = [torch.empty(s.n, dtype=torch.float64, device="cuda") for _ in range(2)]
    x, info = h.solve(out=outs[0], **kw)
    got = []
    t = threading.Thread(target=lambda: got.append(h.solve(out=outs[1], **kw)))
    t.start()
    t.join()
    assert info["converged"] and got[0][1]["iters"] == info["iters"] and torch.equal(outs[0], outs[1])
