"""Launches of 2^32 threads and more: one grid dimension does not hold them, and
runs a part of them without an error.
The gathering interpolation runs 64 threads per point (over 2^26 points), the
cell-list pair sum up to 1024 per cell (over 161 cells per edge).  Points and
ions of the large call are compared with the same ones in a small call, which
evaluates each by itself in the same way: equal up to rounding of positions
that are not changed, so bit for bit."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_gather_of_more_points_than_one_grid_dimension_takes():
    from paper_2001_01583_amd import hpnfft as H
    M, N = (1 << 26) + 1000, (64, 64, 64)
    g = torch.Generator(device="cuda").manual_seed(11)
    x = torch.rand((M, 3), dtype=torch.float64, device="cuda", generator=g) - 0.5
    fh = torch.randn(N, dtype=torch.complex64, device="cuda", generator=g)
    plan = H.Plan(N, M, m=1, precision="f32", method="boxes")
    plan.set_points(x)
    out = plan.forward(fh)
    del plan
    for part in (slice(0, 2000), slice(M // 2, M // 2 + 2000), slice(M - 2000, M)):
        small = H.Plan(N, 2000, m=1, precision="f32", method="boxes")
        small.set_points(x[part].contiguous())
        assert torch.equal(out[part], small.forward(fh))


@pytest.mark.parametrize("nc", [170, 260])
def test_more_cells_than_one_grid_dimension_takes(nc):
    """Ions in the first and the last cells of the box, a few pairs each."""
    from paper_2001_01583_amd import ewald as E
    L, alpha, rcut = nc * 1.0001, 2.0, 1.0
    g = np.random.default_rng(nc)
    r = np.concatenate([g.random((40, 3)) * 2.0, L - g.random((40, 3)) * 2.0])
    q = g.uniform(0.5, 2.0, 80) * np.where(g.random(80) < 0.5, 1.0, -1.0)
    ew = E.Ewald(80, L, alpha, N=(16, 16, 16), m=2, rcut=rcut, real_method="cells")
    e, F = ew.real_space(torch.from_numpy(r).cuda(), torch.from_numpy(q).cuda())
    D = r[:, None] - r[None]
    D -= L * np.round(D / L)
    d = np.sqrt((D * D).sum(-1))
    near = (d < rcut) & (d > 0)
    d[~near] = 1.0
    ec = np.where(near, q[:, None] * q * np.vectorize(math.erfc)(alpha * d) / d, 0.0)
    f = np.where(near, (ec + q[:, None] * q * 2 * alpha / math.sqrt(math.pi) * np.exp(-(alpha * d) ** 2)) / d ** 2, 0.0)
    # (positions up to L and sums of at most 80 terms: L 2^-52 / rcut of a
    # distance, 1e-12 of a term)
    assert near.sum() > 100
    assert abs(float(e) - 0.5 * ec.sum()) <= 1e-12 * np.abs(ec).sum()
    Fr = (f[..., None] * D).sum(1)
    assert np.abs(F.cpu().numpy() - Fr).max() <= 1e-12 * np.abs(Fr).max()
