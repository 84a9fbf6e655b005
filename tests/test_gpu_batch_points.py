"""set_points of a batch as one pass over all transforms: point counts around
the wavefront's 64, box and line transforms in every order, and deterministic
plans.  Every transform against its direct sum;
tolerances: the window's a-priori bound (3 E sqrt(max(1, M / 8))) plus 1e-12
(float64) or 2e-5 (float32) of rounding."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

# (N, M): dense ones use lines, sparse ones boxes
LINES = [((8, 8, 8), 1200), ((12, 6, 10), 2049), ((16, 8, 4), 1023)]
BOXES = [((16, 16, 16), 1), ((24, 20, 18), 63), ((18, 16, 28), 64), ((32, 16, 16), 65)]
ORDERS = {"lines first": LINES + BOXES, "boxes first": BOXES + LINES,
          "mixed": [BOXES[0], LINES[0], BOXES[1], BOXES[2], LINES[1], BOXES[3], LINES[2]]}


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("prec,m", [("f32", 4), ("f64", 4), ("f64", 6)])
@pytest.mark.parametrize("order", sorted(ORDERS))
def test_batch_points(oracle_mod, order, prec, m, det):
    from paper_2001_01583_amd import hpnfft as H
    Ns, Ms = zip(*ORDERS[order])
    m = min(m, min(min(N) for N in Ns))
    g = W.rng(9950 + m)
    x = W.uniform_points(sum(Ms), 3, g)
    cd = torch.complex128 if prec == "f64" else torch.complex64
    f = torch.from_numpy(W.complex_normal(sum(Ms), g)).to(cd)
    plan = H.Plan(list(Ns), list(Ms), m=m, precision=prec, deterministic=det)
    for _ in range(2):  # (the second call finds the counters of the first)
        plan.set_points(torch.from_numpy(x).cuda())
    out = plan.adjoint(f.cuda()).cpu().numpy().astype(np.complex128).ravel()
    wide, po, fo = f.to(torch.complex128).numpy(), 0, 0
    for N, M in zip(Ns, Ms):
        F = math.prod(N)
        ref = np.ravel(oracle_mod.ndft_adjoint(N, x[po:po + M], wide[po:po + M]))
        e = oracle_mod.rel_l2(out[fo:fo + F], ref)
        tol = 3 * H.window_error_bound(m, 2.0) * math.sqrt(max(1.0, M / 8)) + (1e-12 if prec == "f64" else 2e-5)
        print("%s N=%s M=%d %s: %.2e (bound %.1e)" % (order, N, M, prec, e, tol))
        assert e <= tol
        po, fo = po + M, fo + F
