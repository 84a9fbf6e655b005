"""FFT passes with every radix as the first, a middle and the last stage, a
single stage, dims of one element, and workgroups with a remainder of pencils
along rows and columns.  Against the direct sums; tolerances: the window's
a-priori bound (3 E sqrt(max(1, M / 8))) plus 1e-12 (float64) or 2e-5 (float32)
of rounding."""
import itertools
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

# grid edges 2 N: 4 | 8, 16, 32, 64 = 8, 8 2, 8 4, 8 8 | 12, 20, 28 = 4 3, 4 5,
# 4 7 | 36, 100, 196 = 4 3 3, 4 5 5, 4 7 7 | 24, 120, 112 = 8 3, 8 3 5, 8 2 7
EDGES = [(2, 2, 4), (4, 8, 16), (32, 4, 8), (6, 10, 14), (18, 50, 14), (98, 6, 10), (12, 60, 56)]
SIZES = [tuple(N) for e in EDGES for N in dict.fromkeys(itertools.islice(itertools.permutations(e), 0, 5, 2))]
SIZES += [(100,), (14,), (30, 84)]
# many pencils of 4 and of one element per workgroup, along rows and columns
SIZES += [(32, 32, 2), (2, 2, 500), (2, 500), (500, 2)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("N", SIZES)
def test_fft_stages(oracle_mod, N, prec):
    from paper_2001_01583_amd import hpnfft as H
    M, m = 64, min(8, min(N))
    g = W.rng(9900 + sum(N))
    x = W.uniform_points(M, len(N), g)
    f, fhat = W.complex_normal(M, g), W.complex_normal(math.prod(N), g)
    cd = torch.complex128 if prec == "f64" else torch.complex64
    f, fhat = (torch.from_numpy(v).to(cd) for v in (f, fhat))
    plan = H.Plan(N, M, m=m, precision=prec)
    plan.set_points(torch.from_numpy(x).cuda())
    adj = plan.adjoint(f.cuda()).cpu().numpy().astype(np.complex128).ravel()
    fwd = plan.forward(fhat.cuda()).cpu().numpy().astype(np.complex128).ravel()
    wide = [v.to(torch.complex128).numpy() for v in (f, fhat)]
    e = oracle_mod.rel_l2(adj, np.ravel(oracle_mod.ndft_adjoint(N, x, wide[0])))
    d = oracle_mod.rel_l2(fwd, np.ravel(oracle_mod.ndft_forward(N, x, wide[1])))
    E, rnd = H.window_error_bound(m, 2.0), (1e-12 if prec == "f64" else 2e-5)
    ta = 3 * E * math.sqrt(max(1.0, M / 8)) + rnd
    tf = 3 * E * math.sqrt(max(1.0, math.prod(N) / 8)) + rnd
    print("N=%s %s: adjoint %.2e (bound %.1e), forward %.2e (bound %.1e)" % (N, prec, e, ta, d, tf))
    assert e <= ta and d <= tf
