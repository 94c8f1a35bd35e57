"""Prefix sums of the setup at the edges of their launch shapes: one workgroup
up to 16384 values, small tiles of 4096 (a multiple of the tile, one row over),
large tiles above 1024 small ones.  The C points are numbered by a scan over
the level's points and the rows of R and of the coarse matrix are placed by
scans over its coarse points, so the exported hierarchy shows them: whole
numbers, exact."""
import pytest
import torch

from workloads import square_tri_mesh
from workloads.problems import C1Advection1D
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu


def increasing_within_rows(ptr, col):
    new = torch.zeros(col.numel() + 1, dtype=torch.bool, device=col.device)
    new[ptr[:-1]] = True
    return bool((torch.diff(col) > 0)[~new[1:-1]].all())


@pytest.mark.parametrize("n,p,rows", [(1, 1, 6), (52, 1, 16224), (53, 1, 16854), (64, 1, 24576), (64, 3, 49152),
                                      (591, 3, 4191372), (592, 3, 4205568)])
def test_numbering_and_row_pointers(n, p, rows):
    from paper_2010_11130_amd import Hierarchy
    print("case", n, p, flush=True)
    v, c = square_tri_mesh(n)
    s = gpu_system(v, c, C1Advection1D(1e-4), p)
    assert s.n == rows
    h = Hierarchy(s, max_coarse=2)
    assert h.info["n"][0] == rows
    for l in range(h.info["levels"]):
        lv = h.level(l)
        assert int(lv["rowptr"][0]) == 0 and int(lv["rowptr"][-1]) == lv["nnz"]
        assert int(torch.diff(lv["rowptr"]).min()) >= 1 and increasing_within_rows(lv["rowptr"], lv["col"])
        if l + 1 == h.info["levels"]:
            break
        c_pts = lv["cf"] == 1
        assert int(c_pts.sum()) == h.info["n"][l + 1]
        assert torch.equal(lv["pcol"][c_pts], (torch.cumsum(c_pts, 0) - 1)[c_pts].to(torch.int32))
        assert int(lv["Rptr"][0]) == 0 and int(lv["Rptr"][-1]) == lv["Rcol"].numel()
        # each row of R holds its C point and F points only
        row = torch.repeat_interleave(torch.arange(h.info["n"][l + 1], device="cuda"), torch.diff(lv["Rptr"]))
        at_c = c_pts[lv["Rcol"].long()]
        assert torch.equal(row[at_c].to(torch.int32), lv["pcol"][lv["Rcol"][at_c].long()])
        assert int(at_c.sum()) == h.info["n"][l + 1]
