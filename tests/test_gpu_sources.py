"""Gaussian sources and their transpose at the edges of the launch shapes:
points around a wave, a workgroup and the switch to several points per lane
(2^19), centres around the groups of eight and 64, arguments down to the
underflow of the exponential, and non-finite points.

Tolerance: the argument |x - c|^2 / (2 w^2) carries a few roundings, so phi is
off by a few eps (1 + argument); 16 of them per term, summed in absolute
value, with the rounding of the sums themselves (K or points terms, in blocks)
below that."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.mark.parametrize("npts", [1, 63, 65, 257, (1 << 19) - 1, (1 << 19) + 1])
@pytest.mark.parametrize("D,K", [(2, 1), (3, 7), (3, 9), (2, 65)])
def test_sources_and_transpose(npts, D, K):
    from paper_2010_11130_amd import source_gauss, source_gauss_T
    print("case", npts, D, K, flush=True)
    rng = np.random.default_rng(npts + K)
    X, cen = (torch.as_tensor(rng.uniform(0, 1, (m, D)), device="cuda") for m in (npts, K))
    c, y = (torch.as_tensor(rng.standard_normal(m), device="cuda") for m in (K, npts))
    w = 0.1
    arg = ((X[:, None, :] - cen) ** 2).sum(-1) / (2 * w * w)
    phi = torch.exp(-arg)
    off = 16 * EPS * (1 + arg) * phi
    f = source_gauss(X, cen, w, c)
    assert bool(((f - phi @ c).abs() <= off @ c.abs() + 1e-300).all())
    dc = source_gauss_T(X, cen, w, y)
    assert bool(((dc - y @ phi).abs() <= y.abs() @ off + 64 * EPS * (y.abs() @ phi)).all())


def test_underflow_and_nonfinite_points():
    from paper_2010_11130_amd import source_gauss
    r = np.array([0.0, 1e-9, 0.3, 26.0, 27.2, 27.3, 38.5, 1e100, np.inf, np.nan])   # exp(-r^2): subnormal from 26.7
    X = torch.as_tensor(np.stack([r, np.zeros_like(r)], 1), device="cuda")
    cen = torch.zeros((1, 2), dtype=torch.float64, device="cuda")
    f = source_gauss(X, cen, np.sqrt(0.5), torch.ones(1, device="cuda", dtype=torch.float64)).cpu().numpy()
    ref = np.exp(-(r * r))
    assert np.isnan(f[-1]) and np.all(f[6:-1] == 0.0)
    assert np.all(np.abs(f[:6] - ref[:6]) <= 16 * EPS * (1 + r[:6] ** 2) * ref[:6] + 2 * 5e-324)
