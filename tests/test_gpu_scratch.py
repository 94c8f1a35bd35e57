"""Bounds of the memory that a call takes beside its results, counted by a
registered allocator."""
import contextlib

import numpy as np
import pytest
import torch

from workloads import kuhn_cube_mesh
from workloads.problems import PolynomialProblem
from gpu_cases import gpu_system

pytestmark = pytest.mark.gpu
CHUNK = 32 << 20       # smallest request of a library object


class Meter:
    """Device memory from torch, with the live and the largest live size, and
    what was taken and given back in order."""

    def __init__(self):
        self.sizes, self.live, self.peak, self.log = {}, 0, 0, []

    def alloc(self, ctx, nbytes, stream):
        ptr = torch.cuda.caching_allocator_alloc(int(nbytes), stream=int(stream or 0))
        self.sizes[ptr] = nbytes
        self.live += nbytes
        self.peak = max(self.peak, self.live)
        self.log.append((ptr, nbytes))
        return ptr

    def free(self, ctx, ptr, nbytes, stream):
        self.live -= self.sizes.pop(ptr)
        self.log.append((ptr, -nbytes))
        torch.cuda.caching_allocator_delete(ptr)


    def most_given_back(self):
        """The largest sum at one time of pieces that have been given back."""
        open_, pieces, at, most = {}, [], 0, 0
        for k, (ptr, size) in enumerate(self.log):
            if size > 0:
                open_[ptr] = k
            else:
                pieces += [(open_.pop(ptr), -size), (k, size)]
        for _, size in sorted(pieces):
            at += size
            most = max(most, at)
        return most


@contextlib.contextmanager
def metered():
    from paper_2010_11130_amd import lib
    from paper_2010_11130_amd._lib import ALLOC_FN, FREE_FN
    m = Meter()
    cbs = (ALLOC_FN(m.alloc), FREE_FN(m.free))
    assert lib().ah_set_allocator(cbs[0], cbs[1], None) == 0
    m.callbacks = cbs
    try:
        yield m
    finally:
        lib().ah_set_allocator(ALLOC_FN(), FREE_FN(), None)


@pytest.mark.parametrize("npts,K", [(1100000, 32768), (9 << 20, 300), (70000, 40000)])
def test_transposed_sources_in_pieces(npts, K):
    """More points than one piece holds: the partial sums stay within 32 MB or
    256 per centre, and the sums are those of the definition (tolerance: a few
    roundings of the argument |x - c|^2 / (2 w^2) per term, summed in absolute
    value; the sums run in blocks)."""
    from paper_2010_11130_amd import source_gauss_T
    print("case", npts, K, flush=True)
    rng = np.random.default_rng(K)
    X, cen = (torch.as_tensor(rng.uniform(0, 1, (m, 2)), device="cuda") for m in (npts, K))
    y = torch.as_tensor(rng.standard_normal(npts), device="cuda")
    w = 0.1
    with metered() as m:
        dc = source_gauss_T(X, cen, w, y)
    assert m.live == 0 and m.peak <= max(1 << 25, 256 * 8 * K) + CHUNK
    eps = 2.0 ** -52
    for k in [0, 1, K // 2, K - 1]:
        arg = ((X - cen[k]) ** 2).sum(1) / (2 * w * w)
        phi = torch.exp(-arg)
        bound = (16 * eps * (1 + arg) * phi + 64 * eps * phi) @ y.abs()
        assert float((dc[k] - y @ phi).abs()) <= float(bound)


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("block_scale", [False, True])
def test_assembly_needs_no_more_than_it_keeps(keep, block_scale):
    """The elements' parts of the diagonal blocks (79 MB here) are gone before
    the matrix is there."""
    print("case", keep, block_scale, flush=True)
    v, c = kuhn_cube_mesh(16)
    prob = PolynomialProblem(2, 3, 1e-2, seed=3, a_lin=np.zeros((2, 3)))
    with metered() as m:
        s = gpu_system(v, c, prob, 3, keep=keep, block_scale=block_scale)
        assert m.peak <= m.live + CHUNK
        del s
    assert m.live == 0


def test_setup_gives_the_coarsening_back(monkeypatch):
    """Scalar setup of 988,416 rows, 36.6M entries: beside what the hierarchy
    keeps, a level needs its strength mask (a byte per entry), row counters and
    offsets (24 bytes per row) and the chunk of its small buffers; the
    coarsening's packed columns (four bytes per entry) are gone by then."""
    from paper_2010_11130_amd import Hierarchy
    monkeypatch.setenv("AH_SWO", "0")       # no copies of the operators after the last level
    v, c = kuhn_cube_mesh(24)
    s = gpu_system(v, c, PolynomialProblem(2, 2, 1e-2, seed=3, a_lin=np.zeros((2, 3))), 2, keep=False)
    with metered() as m:
        h = Hierarchy(s)
        print("peak", m.peak >> 20, "kept", m.live >> 20, "MB", flush=True)
        assert m.peak <= m.live + s.nnz + 24 * s.n + 2 * CHUNK
        del h
    assert m.live == 0


def test_transposes_one_after_the_other():
    """The adjoint setup of an unscaled system, whose level-0 matrix is
    transposed entry by entry: one second copy of the entries at a time."""
    from paper_2010_11130_amd import Hierarchy
    v, c = kuhn_cube_mesh(32)
    s = gpu_system(v, c, PolynomialProblem(2, 2, 1e-2, seed=3, a_lin=np.zeros((2, 3))), 2, keep=False,
                   block_scale=False)
    with metered() as m:
        h = Hierarchy(s, adjoint=1)
        print("rows", s.n, "entries", s.nnz, "most", m.most_given_back() >> 20, "MB", flush=True)
        assert m.most_given_back() <= 12 * s.nnz + 4 * s.n + 2 * CHUNK
        del h
    assert m.live == 0
