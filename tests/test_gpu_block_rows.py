"""AH_FBB=0 (level 0 by rows) changes the path of odd facet sizes only: even ones
run by rows anyway and keep the copy in sweep order and its sweeps without an
interpolation pass, with the same results bit for bit."""
import numpy as np
import pytest
import torch

from workloads import kuhn_cube_mesh
from workloads.problems import PolynomialProblem
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p", [(4, 1), (3, 2), (2, 3)])     # facet sizes 3, 6, 10
@pytest.mark.parametrize("fp32", [0, 1])
def test_switch(monkeypatch, n, p, fp32):
    from paper_2010_11130_amd import Hierarchy
    print("case", n, p, fp32, flush=True)
    v, c = kuhn_cube_mesh(n)
    s = gpu_system(v, c, PolynomialProblem(2, p, 1e-2, seed=3, a_lin=np.zeros((2, 3))), p)
    monkeypatch.setenv("AH_TAIL_MAX", "0")
    r = torch.as_tensor(np.random.default_rng(1).standard_normal(s.n), device="cuda")
    z = {}
    for fbb in ("1", "0"):
        monkeypatch.setenv("AH_FBB", fbb)
        h = Hierarchy(s, block_air=1, max_coarse=8, fp32_cycle=fp32)
        assert h.info["level0_no_interp_pass"] == (1 if fbb == "1" or s.b % 2 == 0 else 0)
        z[fbb] = h.vcycle(r, precision=fp32)
    if s.b % 2 == 0:
        assert torch.equal(z["0"], z["1"])
    else:
        # other summation order: rounding of the cycle's precision
        assert float((z["0"] - z["1"]).norm()) <= (1e-4 if fp32 else 1e-11) * float(z["1"].norm())
