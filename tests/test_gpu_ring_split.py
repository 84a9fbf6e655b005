"""Ring sweeps whose items are cut to fewer blocks than a tile has: the
wavefronts left over then share the blocks' chunks of points.  All points lie
in k tap rows of one tile, so the heavy (tile, slab) pairs are cut between
rows; the first planes wrap around the torus.  Compared with the staged
sweeps: equal up to the order of the additions (the tolerances of the other
ring comparison)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 2e-6)])
@pytest.mark.parametrize("rows,per_row", [(1, 9000), (2, 2300), (3, 1100), (5, 700), (8, 300), (8, 37)])
def test_split_items(rows, per_row, prec, tol):
    from paper_2001_01583_amd import hpnfft as H
    N = (16, 16, 12)
    n = [2 * v for v in N]
    g = W.rng(7000 + 10 * rows + per_row)
    M = rows * per_row
    x = np.empty((M, 3))
    x[:, 0] = g.random(M) - 0.5
    x[:, 1] = (8 + np.repeat(np.arange(rows), per_row) + g.random(M)) / n[1] - 0.5
    x[:, 2] = (16 + 8 * g.random(M)) / n[2] - 0.5
    cd = torch.complex128 if prec == "f64" else torch.complex64
    f = torch.from_numpy(W.complex_normal(M, g)).cuda().to(cd)
    fh = torch.from_numpy(W.complex_normal(int(np.prod(N)), g).reshape(N)).cuda().to(cd)
    out = []
    for tiles in ((8, 16, 512), (8, 12, 512)):  # ring, staged
        plan = H.Plan(N, M, m=4, precision=prec, method="lines", tiles=tiles)
        plan.set_points(torch.from_numpy(x).cuda())
        out.append((plan.adjoint(f).cpu().numpy(), plan.forward(fh).cpu().numpy()))
    for a, b in zip(out[0], out[1]):
        d = np.linalg.norm((a - b).astype(np.complex128)) / np.linalg.norm(b.astype(np.complex128))
        print("rows %d per row %d %s: %.3e" % (rows, per_row, prec, d))
        assert d <= tol
