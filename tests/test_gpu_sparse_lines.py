"""Forward of float64 line-method plans of 2m = 8 on both sides of the density at
which ring sweeps take over from the gather (0.15 points per cell), alone and in
a batch, against the direct sums: the window's a-priori bound (3 E sqrt(max(1,
prod n / 8))) plus 1e-12 of rounding."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Ms", [((16, 16, 16), (1, 600, 4915, 4916)), ((12, 10, 18), (2592, 2593)),
                                  ((24, 8, 8), (1843, 1844))])
def test_sparse_lines(oracle_mod, N, Ms):
    from paper_2001_01583_amd import hpnfft as H
    g = W.rng(9970 + N[0])
    x = W.uniform_points(sum(Ms), 3, g)
    x[0], x[-1] = -0.5, [0.5 - 1e-13, -0.5, 0.5 - 1e-13]
    fh = W.complex_normal(int(np.prod(N)), g)
    tol = 3 * H.window_error_bound(4, 2.0) * math.sqrt(np.prod(N)) + 1e-12
    assert tol < 1e-2
    po, xs = 0, torch.from_numpy(x).cuda()
    ref = oracle_mod.ndft_forward(N, x, fh.reshape(N))
    for M in Ms:
        p = H.Plan(N, M, m=4, precision="f64", method="lines")
        p.set_points(xs[po:po + M].contiguous())
        e = oracle_mod.rel_l2(p.forward(torch.from_numpy(fh).cuda()).cpu().numpy(), ref[po:po + M])
        print("sparse lines N=%s M=%d: %.2e (bound %.1e)" % (N, M, e, tol))
        assert e <= tol
        po += M
    b = H.Plan([N] * len(Ms), list(Ms), m=4, precision="f64", method="lines")
    b.set_points(xs)
    out = b.forward(torch.from_numpy(np.tile(fh, len(Ms))).cuda()).cpu().numpy()
    assert oracle_mod.rel_l2(out, ref) <= tol
