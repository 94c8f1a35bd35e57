"""The transposed operators of the adjoint cycle, whose rows are placed by
rank: 16 lanes per row for short rows, a wave per row otherwise, in chunks
where a row is longer than its lanes.  The transposed V-cycle must be the
transpose of the forward one on hierarchies whose coarse rows are shorter than
16, between and above 64 entries, and rebuilding it must give the same bits
(the scatter before the placement runs in no fixed order).

Tolerance: <Bx, y> and <x, B^T y> sum the same products in other orders, so
they differ by rounding: 1e-12 of ||Bx|| ||y|| for a few hundred operations
per entry in FP64."""
import numpy as np
import pytest
import torch

from workloads import square_tri_mesh, kuhn_cube_mesh, map_vertices_c5
from workloads.problems import C1Advection1D, GaussianSources, c5_sources
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh,n,p,air,longest", [
    ("square", 9, 1, {}, 0), ("cube", 5, 1, {}, 16), ("cube", 9, 2, {"theta": 0.5, "theta_r": 0.25}, 64),
    ("cube", 9, 1, {"block_air": 1}, 16)])
def test_transposed_cycle_is_the_transpose(mesh, n, p, air, longest):
    from paper_2010_11130_amd import Hierarchy
    print("case", mesh, n, p, air, flush=True)
    if mesh == "square":
        v, c = square_tri_mesh(n)
        prob = C1Advection1D(1e-4)
    else:
        v, c = kuhn_cube_mesh(n)
        v = map_vertices_c5(v)
        prob = GaussianSources(1e-3, c5_sources(8)[0], c5_sources(8)[2])
    s = gpu_system(v, c, prob, p)
    rng = np.random.default_rng(3)
    x, y = (torch.as_tensor(rng.standard_normal(s.n), device="cuda") for _ in range(2))
    h = Hierarchy(s, adjoint=1, max_coarse=8, **air)
    rows = max(int(torch.diff(h.level(l)["rowptr"]).max()) for l in range(h.info["levels"]))
    assert rows > longest
    bx, bty = h.vcycle(x), h.vcycle(y, transpose=True)
    gap = abs(float(bx @ y) - float(x @ bty))
    assert gap <= 1e-12 * float(bx.norm()) * float(y.norm()), gap
    again = Hierarchy(s, adjoint=1, max_coarse=8, **air).vcycle(y, transpose=True)
    assert torch.equal(again, bty)
