"""Ring sweeps (2m = 8) on grids whose n0 is no multiple of 8: the last group of
planes is cut, and periodic images carry their weights in another slot order.
Points at both ends of dim 0, a cluster there (items cut to fewer rows of
blocks), the smallest such grid, a single and several slabs.  Against the direct sums; tolerances: the window's a-priori
bound (3 E sqrt(inputs / 8)) plus 1e-12 (float64) or 2e-5 (float32) of rounding."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("points", ["uniform", "ends", "cluster"])
@pytest.mark.parametrize("N,Zs", [((10, 8, 12), 32), ((10, 10, 8), 8), ((18, 6, 10), 32), ((42, 8, 10), 16), ((30, 8, 8), 32),
                                  ((14, 12, 14), 8), ((50, 6, 8), 32), ((14, 10, 14), 16)])
def test_ring_planes(oracle_mod, N, Zs, points, prec):
    from paper_2001_01583_amd import hpnfft as H
    M, m = 3000, 4
    g = W.rng(9980 + N[0] + Zs)
    x = W.uniform_points(M, 3, g)
    if points == "ends":
        x[:, 0] = W.wrap_unit(0.5 + 0.04 * g.standard_normal(M))
    elif points == "cluster":
        x = W.wrap_unit(np.array([0.49, 0.1, -0.49]) + 0.02 * g.standard_normal((M, 3)))
    x[0], x[1] = -0.5, 0.5 - 1e-13
    cd = torch.complex128 if prec == "f64" else torch.complex64
    f = torch.from_numpy(W.complex_normal(M, g)).to(cd)
    fh = torch.from_numpy(W.complex_normal(math.prod(N), g).reshape(N)).to(cd)
    plan = H.Plan(N, M, m=m, precision=prec, method="lines", tiles=(8, Zs, 512))
    plan.set_points(torch.from_numpy(x).cuda())
    adj = plan.adjoint(f.cuda()).cpu().numpy().astype(np.complex128)
    fwd = plan.forward(fh.cuda()).cpu().numpy().astype(np.complex128)
    wide = [v.to(torch.complex128).numpy() for v in (f, fh)]
    ea = oracle_mod.rel_l2(adj.ravel(), np.ravel(oracle_mod.ndft_adjoint(N, x, wide[0])))
    ef = oracle_mod.rel_l2(fwd.ravel(), np.ravel(oracle_mod.ndft_forward(N, x, wide[1])))
    E, rnd = H.window_error_bound(m, 2.0), (1e-12 if prec == "f64" else 2e-5)
    ta, tf = (3 * E * math.sqrt(max(1.0, c / 8)) + rnd for c in (M, math.prod(N)))
    print("N=%s Zs=%d %s %s: adjoint %.2e (%.1e), forward %.2e (%.1e)" % (N, Zs, points, prec, ea, ta, ef, tf))
    assert ea <= ta and ef <= tf
