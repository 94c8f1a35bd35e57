"""Element assembly over every orientation it can meet: meshes whose vertices
and cells are relabelled at random (so every facet-vertex permutation and
every local facet occurs), element counts that do not fill a workgroup of four,
velocity at vertices and at points, for every (dimension, degree); and a cell
given twice, whose off-diagonal blocks get two parts.

Against the oracle's Lagrange-basis quadrature.  Tolerances as in the assembly
parity test: 1e-12 of the largest entry (1e-11 for the block inverses), which
covers the condition of the element systems at these degrees."""
import numpy as np
import pytest
import torch

from oracle.drivers import setup_problem, direct_solve
from oracle import hdg
from workloads import square_tri_mesh, kuhn_cube_mesh
from workloads.problems import PolynomialProblem
from gpu_cases import gpu_system, to_scipy, rel_sparse_diff

pytestmark = pytest.mark.gpu


def shuffled(D, n, seed):
    v, c = square_tri_mesh(n) if D == 2 else kuhn_cube_mesh(n)
    rng = np.random.default_rng(seed)
    at = rng.permutation(len(v))
    w = np.empty_like(v)
    w[at] = v
    inner = np.all((w > 0) & (w < 1), axis=1)
    w[inner] += 0.1 / n * rng.uniform(-1, 1, (int(inner.sum()), D))
    return w, rng.permuted(at[c], axis=1).astype(np.int32)[rng.permutation(len(c))]


def check(s, o):
    ex = s.export()
    assert s.n == o.n
    assert rel_sparse_diff(to_scipy(ex["rowptr"], ex["col"], ex["val"], s.n), o.Shat) < 1e-12
    for name, ref, tol in (("hhat", o.Hhat, 1e-12), ("dinv", o.Dinv, 1e-11), ("lam_dir", o.lamD_full, 1e-12)):
        assert np.abs(ex[name].cpu().numpy() - ref).max() <= tol * max(np.abs(ref).max(), 1e-300), name


@pytest.mark.parametrize("at_points", [False, True])
@pytest.mark.parametrize("D,p,n", [(2, 1, 3), (2, 2, 3), (2, 3, 3), (3, 1, 3), (3, 2, 1), (3, 3, 1), (3, 3, 2)])
def test_random_orientations(D, p, n, at_points):
    print("case", D, p, n, at_points, flush=True)
    v, c = shuffled(D, n, 10 * D + p)
    prob = PolynomialProblem(D - 1, p + 1, 3e-2, seed=p)
    s = gpu_system(v, c, prob, p, at_points=at_points)
    o = setup_problem(v, c, prob, p)
    check(s, o)
    lam = direct_solve(o)
    u, ref = s.reconstruct(torch.as_tensor(lam, device="cuda")).cpu().numpy(), hdg.reconstruct(o, lam)
    assert np.abs(u - ref).max() <= 1e-11 * np.abs(ref).max()


@pytest.mark.parametrize("D,p", [(2, 2), (3, 1)])
def test_cell_given_twice(D, p):
    print("case", D, p, flush=True)
    v, c = shuffled(D, 2, 7)
    v, c = np.concatenate([v, v[c[0]] + 3.0]), np.concatenate([c, [np.arange(D + 1) + len(v)] * 2]).astype(np.int32)
    prob = PolynomialProblem(D - 1, p, 3e-2, seed=p)
    check(gpu_system(v, c, prob, p), setup_problem(v, c, prob, p))


@pytest.mark.parametrize("D,p", [(2, 2), (3, 2)])
def test_unscaled_keeps_the_diagonal_blocks(D, p):
    print("case", D, p, flush=True)
    v, c = shuffled(D, 2, 5)
    prob = PolynomialProblem(D - 1, p, 3e-2, seed=p)
    check(gpu_system(v, c, prob, p, block_scale=False), setup_problem(v, c, prob, p, block_scale=False))


def test_tables_shared_by_threads():
    """The reference tables are built once per (dimension, degree): threads on
    their own streams that all meet them first (after a trim) get the systems
    that a single thread gets."""
    import threading
    from paper_2010_11130_amd import pool_trim
    work = [(D, p) for D in (2, 3) for p in (1, 2, 3)] * 2
    data = [(shuffled(D, 2, 3), PolynomialProblem(D - 1, p, 3e-2, seed=p), p) for D, p in work]
    ref = [gpu_system(*vc, prob, p).export()["val"] for vc, prob, p in data]
    pool_trim()
    got = [None] * len(data)

    def run(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            got[k] = gpu_system(*data[k][0], data[k][1], data[k][2]).export()["val"]

    ths = [threading.Thread(target=run, args=(k,)) for k in range(len(data))]
    for t in ths:
        t.start()
    for t in ths:
        t.join()
    assert all(torch.equal(a, b) for a, b in zip(ref, got))
