"""Gradient records in float64 (one lane per table entry, 16 points per
wavefront): point counts around 16 and 64, plans of one and two dimensions,
whose leading dims hold a unit impulse, and deterministic plans.  Gradients
against the direct sums; tolerances: the window's a-priori bound (3 E
sqrt(prod N / 8), times pi max n for a derivative) plus 1e-12 (1e-11) of
rounding."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("N,M,m", [((40,), 15, 8), ((36,), 65, 5), ((12, 20), 16, 4), ((18, 16), 17, 8),
                                   ((8, 10, 12), 63, 4), ((8, 16, 10), 64, 8), ((32, 30, 36), 1, 12)])
def test_tables(oracle_mod, N, M, m, det):
    from paper_2001_01583_amd import hpnfft as H
    d = len(N)
    g = W.rng(9970 + M + m)
    x = W.uniform_points(M, d, g)
    x[0] = -0.5
    f = W.complex_normal(M, g)
    fh = W.complex_normal(math.prod(N), g).reshape(N)
    plan = H.Plan(N, M, m=m, precision="f64", with_grad=True, deterministic=det)
    plan.set_points(torch.from_numpy(x).cuda())
    gf, gx = plan.adjoint_backward(torch.from_numpy(f).cuda(), torch.from_numpy(fh).cuda().reshape(-1))
    ref = np.ravel(oracle_mod.ndft_forward(N, x, fh))
    k = [np.arange(-v // 2, v // 2) for v in N]
    refx = np.stack([np.real(f * np.conj(np.ravel(oracle_mod.ndft_forward(
        N, x, fh * (2j * np.pi * k[t]).reshape([-1 if u == t else 1 for u in range(d)])))))
        for t in range(d)], 1)
    ef = oracle_mod.rel_l2(gf.cpu().numpy().ravel(), ref)
    ex = np.linalg.norm(gx.cpu().numpy().reshape(M, d) - refx) / np.linalg.norm(refx)
    e = 3 * H.window_error_bound(m, 2.0) * math.sqrt(max(1.0, math.prod(N) / 8))
    tf, tx = e + 1e-12, e * math.pi * 2 * max(N) + 1e-11
    print("N=%s M=%d m=%d: grad_f %.2e (%.1e), grad_x %.2e (%.1e)" % (N, M, m, ef, tf, ex, tx))
    assert ef <= tf and ex <= tx
