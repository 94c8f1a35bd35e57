"""Reference tables and the caller's allocator: with one registered, every system
has its tables in memory from it (found there by the quadrature weights that
they hold) and gives all of it back; the library's own copy, used otherwise,
gives the same system bit for bit."""
import gc

import numpy as np
import pytest
import torch

from workloads import kuhn_cube_mesh
from workloads.problems import PolynomialProblem
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu


class Bump:
    """Device memory from one tensor, never reused; what is live is counted."""

    def __init__(self, nbytes):
        self.buf = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        self.at, self.live = 0, {}

    def alloc(self, ctx, nbytes, stream):
        at = (self.at + 255) // 256 * 256
        if at + nbytes > self.buf.numel():
            return None
        self.at = at + nbytes
        ptr = self.buf.data_ptr() + at
        self.live[ptr] = nbytes
        return ptr

    def free(self, ctx, ptr, nbytes, stream):
        assert self.live.pop(ptr) == nbytes

    def copies(self, w):
        """How often the values w stand in the memory handed out."""
        x = self.buf[:self.at].view(torch.float64)
        hit = torch.ones(x.numel() - len(w) + 1, dtype=torch.bool, device="cuda")
        for k, v in enumerate(w):
            hit &= x[k:k + hit.numel()] == v
        return int(hit.sum())


def export(s):
    return {k: v.cpu().numpy() for k, v in s.export().items()}


@pytest.mark.parametrize("p", [1, 3])
def test_tables_come_from_the_registered_allocator(p):
    from paper_2010_11130_amd import System, lib, quad_rule
    from paper_2010_11130_amd._lib import ALLOC_FN, FREE_FN
    prob = PolynomialProblem(2, p, 1e-2, seed=3, a_lin=np.zeros((2, 3)))
    v, c = kuhn_cube_mesh(2)
    s = gpu_system(v, c, prob, p)          # uploads the mesh, which is no matter of the allocator
    mesh, a = s.mesh, s._a
    want = export(System(mesh, p, 1e-2, a, None, None))
    del s
    gc.collect()
    bump = Bump(320 << 20)
    cbs = (ALLOC_FN(bump.alloc), FREE_FN(bump.free))
    assert lib().ah_set_allocator(cbs[0], cbs[1], None) == 0
    try:
        systems = [System(mesh, p, 1e-2, a, None, None) for _ in range(4)]
        torch.cuda.synchronize()
        assert bump.copies(quad_rule(3, p + 2)[1]) >= len(systems)
        got = export(systems[-1])
        del systems
        gc.collect()
        torch.cuda.synchronize()
        assert not bump.live
    finally:
        lib().ah_set_allocator(ALLOC_FN(), FREE_FN(), None)
    again = export(System(mesh, p, 1e-2, a, None, None))
    for k in want:
        assert np.array_equal(got[k], want[k]) and np.array_equal(again[k], want[k]), k
