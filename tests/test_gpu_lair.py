"""lAIR restriction rows at the edges of their layouts: neighbourhoods of no
points, up to 8 and up to 16 (lanes of a group), and larger ones (a wave per
row); rows of facet blocks of every size.  The definition is checked on the
exported matrices: (R A)_ij = 0 for every point j of row i's neighbourhood,
except in rows without a local system (a one alone, or zeros after a singular
one), which the setup counts.

Tolerance: LU with partial pivoting solves a row of m <= 64 points with a
residual of a small multiple of m eps (|R| |A|)_ij; 1e-12 of that product."""
import numpy as np
import pytest
import scipy.sparse as sp

from workloads import square_tri_mesh, kuhn_cube_mesh
from workloads.problems import C1Advection1D, SmoothPlusFront
from gpu_cases import gpu_system, to_scipy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,p,air,most", [
    ("square", 2, 1, {}, 1), ("square", 13, 1, {}, 2), ("square", 12, 3, {"theta": 0.05}, 8),
    ("cube", 9, 1, {}, 8), ("cube", 5, 2, {"theta": 0.5, "theta_r": 0.05}, 16),
    ("square", 9, 1, {"block_air": 1}, 1), ("square", 9, 2, {"block_air": 1}, 1),
    ("square", 9, 3, {"block_air": 1}, 1), ("cube", 6, 1, {"block_air": 1}, 5),
    ("cube", 4, 2, {"block_air": 1}, 5), ("cube", 3, 3, {"block_air": 1}, 9)])
def test_rows_annihilate_their_neighbourhood(kind, n, p, air, most):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, p, air, flush=True)
    v, c = square_tri_mesh(n) if kind == "square" else kuhn_cube_mesh(n)
    prob = C1Advection1D(1e-4) if kind == "square" else SmoothPlusFront(1e-3, width=0.1)
    h = Hierarchy(gpu_system(v, c, prob, p), max_coarse=4, **air)
    without = widest = 0
    for l in range(h.info["levels"] - 1):
        lv = h.level(l)
        nc = h.info["n"][l + 1]
        A = to_scipy(lv["rowptr"], lv["col"], lv["val"], lv["n"])
        R = to_scipy(lv["Rptr"], lv["Rcol"], lv["Rval"], nc, lv["n"])
        ptr, col, val = (lv[k].cpu().numpy() for k in ("Rptr", "Rcol", "Rval"))
        row = np.repeat(np.arange(nc), np.diff(ptr))
        cf = lv["cf"].cpu().numpy()
        f = cf[col] == 0
        assert np.array_equal(np.bincount(row, weights=~f, minlength=nc), np.ones(nc))
        assert np.all(val[~f] == 1.0)
        solved = np.bincount(row, weights=f & (val != 0.0), minlength=nc) > 0
        without += int((~solved).sum())
        widest = max(widest, int(np.bincount(row, weights=f, minlength=nc).max()))
        at = f & solved[row]
        keep = sp.csr_matrix((np.ones(at.sum()), (row[at], col[at])), shape=R.shape)
        left = abs((R @ A).multiply(keep))
        scale = (abs(R) @ abs(A)).multiply(keep)
        assert (left - 1e-12 * scale).max() <= 0.0, (l, left.max())
    assert without == h.info["n_fallback"] and widest >= most
