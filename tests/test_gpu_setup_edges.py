"""Setup kernels at the edges of their layouts: the one-workgroup PMIS with its
lists in LDS, with only their offsets there and with both in global memory, and
as the end of grid-wide rounds; strength and one-point interpolation of rows longer than the entries a lane
keeps in registers; the register-held inverse of the coarsest matrix.

The splitting and the interpolation are compared exactly, with the grid-wide
rounds (AH_PMIS_WG_MAX=0) and with the definition on the exported matrices.  Tolerance of the inverse:
Gauss-Jordan elimination with partial pivoting is off by a small multiple of
n eps cond(A); 64 eps cond(A) for n <= 64."""
import numpy as np
import pytest
import torch

from workloads import square_tri_mesh, kuhn_cube_mesh, slab_prism_tet_mesh, stacked_prism_tet_mesh
from workloads.problems import C1Advection1D, SmoothPlusFront
from gpu_cases import gpu_system, to_scipy

pytestmark = pytest.mark.gpu

MESH = {"square": lambda n: square_tri_mesh(n), "cube": lambda n: kuhn_cube_mesh(n),
        "slab": lambda n: slab_prism_tet_mesh(n, 1.0 / 64), "stack": lambda n: stacked_prism_tet_mesh(*n)}


def problem(kind, n, p):
    v, c = MESH[kind](n)
    return v, c, C1Advection1D(1e-4) if kind == "square" else SmoothPlusFront(1e-3, width=0.1), p


@pytest.mark.parametrize("kind,n,p,air", [
    ("square", 1, 1, {}), ("square", 13, 1, {}), ("square", 36, 1, {}),      # everything in LDS
    ("cube", 6, 1, {"theta": 0.02}), ("slab", 8, 2, {"theta": 0.01}),        # lists too long for LDS
    ("stack", (3, 14), 2, {}),                                               # 8172 rows: offsets outside too
    ("cube", 9, 1, {"block_air": 1})])
def test_one_workgroup_rounds_give_the_same_split(monkeypatch, kind, n, p, air):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, p, air, flush=True)
    s = gpu_system(*problem(kind, n, p))
    if kind == "stack":
        assert s.n == 8172
    h = Hierarchy(s, max_coarse=2, **air)
    monkeypatch.setenv("AH_PMIS_WG_MAX", "0")
    ref = Hierarchy(s, max_coarse=2, **air)
    assert h.info["n"] == ref.info["n"]
    for l in range(h.info["levels"] - 1):
        a, b = h.level(l), ref.level(l)
        assert torch.equal(a["cf"], b["cf"]) and torch.equal(a["pcol"], b["pcol"]), l


@pytest.mark.parametrize("list_min", ["0", "1000000000"])
@pytest.mark.parametrize("kind,n,p,air", [("stack", (3, 15), 2, {}),              # 8748 rows
                                          ("square", 64, 3, {}), ("cube", 9, 2, {"theta": 0.02}),
                                          ("slab", 40, 2, {}), ("cube", 16, 1, {"block_air": 1})])
def test_last_rounds_in_one_workgroup_give_the_same_split(monkeypatch, kind, n, p, air, list_min):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, p, air, list_min, flush=True)
    monkeypatch.setenv("AH_PMIS_LIST_MIN", list_min)
    s = gpu_system(*problem(kind, n, p))
    got = {}
    for cap in ("8192", "50", "0"):
        monkeypatch.setenv("AH_PMIS_WG_MAX", cap)
        h = Hierarchy(s, max_coarse=2, **air)
        got[cap] = [(h.level(l)["cf"], h.level(l)["pcol"]) for l in range(h.info["levels"] - 1)]
    for cap in ("8192", "50"):
        assert len(got[cap]) == len(got["0"])
        for (a, pa), (b, pb) in zip(got[cap], got["0"]):
            assert torch.equal(a, b) and torch.equal(pa, pb)


@pytest.mark.parametrize("kind,n,p,theta,theta_r,longest", [("square", 9, 1, 0.25, 0.25, 8),
                                                            ("cube", 2, 3, 0.01, 0.01, 40),
                                                            ("cube", 9, 2, 0.5, 0.25, 64)])
def test_strength_and_interpolation_of_long_rows(kind, n, p, theta, theta_r, longest):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, p, theta, theta_r, flush=True)
    s = gpu_system(*problem(kind, n, p))
    h = Hierarchy(s, max_coarse=8, theta=theta, theta_r=theta_r)
    levels = [h.level(l) for l in range(h.info["levels"] - 1)]
    assert max(int(torch.diff(lv["rowptr"]).max()) for lv in levels) > longest
    for l, lv in enumerate(levels):
        ptr, col, val, cf, pcol, rptr = (lv[k].cpu().numpy() for k in ("rowptr", "col", "val", "cf", "pcol", "Rptr"))
        row = np.repeat(np.arange(lv["n"]), np.diff(ptr))
        off = np.where(col == row, 0.0, np.abs(val))
        top = np.maximum.reduceat(off, ptr[:-1])[row] * (1.0 - 1e-12)
        strong, strong_r = ((off > 0) & (off >= th * top) for th in (theta, theta_r))
        to_c = strong & (cf[col] == 1)
        best = np.maximum.reduceat(np.where(to_c, off, 0.0), ptr[:-1])
        near = np.flatnonzero(to_c & (off >= best[row] * (1.0 - 1e-12)))[::-1]
        want = np.full(lv["n"], -1)
        cidx = np.cumsum(cf == 1) - 1
        want[row[near]] = cidx[col[near]]   # the first of the row is written last
        want[cf == 1] = cidx[cf == 1]
        assert np.array_equal(pcol, want), l
        around = np.bincount(row, weights=strong_r & (cf[col] == 0), minlength=lv["n"]).astype(int)
        assert np.array_equal(np.diff(rptr), 1 + around[cf == 1]), l


@pytest.mark.parametrize("kind,n,p", [("square", 1, 1), ("square", 1, 3), ("square", 2, 2), ("square", 2, 3),
                                      ("square", 3, 1), ("cube", 1, 1), ("cube", 1, 2)])
def test_inverse_of_a_coarsest_matrix(monkeypatch, kind, n, p):
    from paper_2010_11130_amd import Hierarchy
    print("case", kind, n, p, flush=True)
    monkeypatch.setenv("AH_TAIL_MAX", "0")
    s = gpu_system(*problem(kind, n, p))
    assert s.n <= 64
    h = Hierarchy(s, max_coarse=64)
    assert h.info["levels"] == 1
    lv = h.level(0)
    A = to_scipy(lv["rowptr"], lv["col"], lv["val"], s.n).toarray()
    r = np.random.default_rng(2).standard_normal(s.n)
    x = h.vcycle(torch.as_tensor(r, device="cuda")).cpu().numpy()
    want = np.linalg.solve(A, r)
    assert np.linalg.norm(x - want) <= 64 * np.finfo(float).eps * np.linalg.cond(A) * np.linalg.norm(want)
