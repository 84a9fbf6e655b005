"""Cell-list pair sums of boxes with many cells and few ions each (workgroups of
256 threads, tiles of 1024 ions): empty cells, one ion, a cell whose neighbours
hold more than a tile, and mean occupations on both sides of 32 ions per cell,
where large workgroups take over.  Reference: the pair sum in float64 torch
operations; tolerance: sums of at most 2e4 terms of both signs, 1e-12 of the
largest force and of the sum of |terms| for the energy."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,M,crowd", [(10, 1, 0), (11, 2600, 0), (11, 300, 1500), (13, 900, 1030), (16, 20000, 0),
                                        (11, 11 ** 3 * 32 - 1, 0), (11, 11 ** 3 * 32, 0)])
def test_sparse_cells(nc, M, crowd):
    from paper_2001_01583_amd import ewald as E
    g = W.rng(8300 + M)
    L, rcut, alpha = nc * 1.001, 1.0, 2.0
    r = g.random((M, 3)) * L
    if crowd:  # around a corner of the box: four of the cells, across its faces
        r = np.concatenate([r, (g.random((crowd, 3)) * np.array([1.6, 1.6, 0.5]) - np.array([0.8, 0.8, 0.0])) % L])
    q = torch.from_numpy(np.where(g.random(len(r)) < 0.5, 1.0, -1.0) * g.uniform(0.5, 2.0, len(r))).cuda()
    r = torch.from_numpy(r).cuda()
    ew = E.Ewald(len(r), L, alpha, N=(16, 16, 16), m=2, rcut=rcut, real_method="cells")
    for _ in range(2):
        e, F = ew.real_space(r, q)
    U, A = 0.0, 0.0
    Fr = torch.empty_like(F)
    for a in range(0, len(r), 1024):
        D = r[a:a + 1024, None, :] - r[None]
        D -= L * torch.round(D / L)
        d2 = (D * D).sum(-1)
        d2[torch.arange(len(D)), torch.arange(a, a + len(D))] = math.inf
        near = d2 < rcut * rcut
        d = torch.sqrt(torch.where(near, d2, torch.ones_like(d2)))
        qq = torch.where(near, q[a:a + 1024, None] * q[None], torch.zeros_like(d))
        ec = qq * torch.erfc(alpha * d) / d
        f = (ec + qq * 2 * alpha / math.sqrt(math.pi) * torch.exp(-(alpha * d) ** 2)) / d ** 2
        U, A = U + 0.5 * float(ec.sum()), A + 0.5 * float(ec.abs().sum())
        Fr[a:a + 1024] = (f[..., None] * D).sum(1)
    big = float(Fr.abs().max())
    print("sparse cells nc=%d M=%d: energy %.2e force %.2e" % (nc, len(r), abs(float(e) - U) / max(A, 1e-300),
                                                               float((F - Fr).abs().max()) / max(big, 1e-300)))
    assert abs(float(e) - U) <= 1e-12 * A
    assert float((F - Fr).abs().max()) <= 1e-12 * big
