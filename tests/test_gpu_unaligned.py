"""Caller's vectors at an odd offset (8-byte aligned views): every solve gives
what it gives with aligned ones, bit for bit, at the even block sizes whose
products load x in pairs and at an odd one."""
import numpy as np
import pytest
import torch

from workloads import square_tri_mesh, kuhn_cube_mesh
from workloads.problems import C1Advection1D, PolynomialProblem
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu


def odd(x):
    buf = torch.zeros(x.numel() + 1, dtype=torch.float64, device="cuda")
    buf[1:].copy_(x)
    assert buf[1:].data_ptr() % 16 == 8
    return buf[1:]


@pytest.mark.parametrize("kind,n,p", [("square", 8, 1), ("square", 6, 3), ("cube", 3, 1), ("cube", 3, 2),
                                      ("cube", 2, 3)])
@pytest.mark.parametrize("kw", [dict(), dict(noalloc=True, restart=5), dict(method=1)])
@pytest.mark.parametrize("delayed", [False, True])
def test_odd_offsets(monkeypatch, kind, n, p, kw, delayed):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, p, kw, delayed, flush=True)
    monkeypatch.setenv("AH_DCGS_MIN", "0" if delayed else "1000000000")
    v, c = square_tri_mesh(n) if kind == "square" else kuhn_cube_mesh(n)
    prob = C1Advection1D(1e-2) if kind == "square" else PolynomialProblem(2, p, 1e-2, seed=3, a_lin=np.zeros((2, 3)))
    s = gpu_system(v, c, prob, p)
    h = Hierarchy(s, max_coarse=8, adjoint=1)
    rhs, x0 = (torch.as_tensor(r, device="cuda") for r in np.random.default_rng(2).standard_normal((2, s.n)))
    got = []
    for f in (lambda t: t.clone(), odd):
        x, info = h.solve(f(rhs), x0=f(x0), out=f(rhs), tol=1e-9, **kw)
        assert info["converged"]
        got.append([x])
        if "noalloc" not in kw:
            lam, info = h.solve_adjoint(f(rhs), out=f(rhs), tol=1e-9, **kw)
            assert info["converged"]
            got[-1].append(lam)
    for a, b in zip(*got):
        assert torch.equal(a, b)
