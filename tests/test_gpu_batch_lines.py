"""Batches whose line transforms are interpolated by one launch over all their
line groups (2m = 10 .. 16), beside box transforms that gather: transforms of
one and of several plane ranges, in every order.  A point's sums do not depend
on what else is in the plan, so forward and gradients equal those of single
plans bit for bit; the adjoint is compared with the direct sums (the window's
a-priori bound, 3 E sqrt(max(1, M / 8)), plus 1e-12 or 2e-5 of rounding)."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

# (N, M): dense ones use lines, sparse ones boxes
LINES = [((8, 8, 8), 1200), ((12, 16, 10), 4099), ((64, 12, 12), 12000), ((16, 12, 14), 4000)]
BOXES = [((16, 16, 16), 1), ((24, 20, 18), 63), ((18, 16, 28), 64)]
ORDERS = {"lines only": LINES, "lines first": LINES + BOXES, "boxes first": BOXES + LINES,
          "mixed": [BOXES[0], LINES[0], BOXES[1], BOXES[2], LINES[1], LINES[2], LINES[3]]}


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("m", [5, 6, 7, 8])
@pytest.mark.parametrize("order", sorted(ORDERS))
def test_batch_lines(oracle_mod, order, m, prec):
    from paper_2001_01583_amd import hpnfft as H
    Ns, Ms = zip(*ORDERS[order])
    g = W.rng(9960 + m)
    cd = torch.complex128 if prec == "f64" else torch.complex64
    x = W.uniform_points(sum(Ms), 3, g)
    f = torch.from_numpy(W.complex_normal(sum(Ms), g)).to(cd).cuda()
    fh = torch.from_numpy(W.complex_normal(sum(math.prod(N) for N in Ns), g)).to(cd).cuda()
    xg = torch.from_numpy(x).cuda()
    plan = H.Plan(list(Ns), list(Ms), m=m, precision=prec, with_grad=True)
    assert plan.m == m and plan.method == ("lines" if order == "lines only" else "mixed")
    plan.set_points(xg)
    adj, fwd = plan.adjoint(f).cpu().numpy().astype(np.complex128).ravel(), plan.forward(fh)
    gf, gx = plan.adjoint_backward(f, fh)
    assert torch.equal(gf, plan.adjoint_backward(f, fh, need_x=False)[0])
    po, fo = 0, 0
    for N, M in zip(Ns, Ms):
        P, F = slice(po, po + M), slice(fo, fo + math.prod(N))
        one = H.Plan(N, M, m=m, precision=prec, with_grad=True, method="lines" if (N, M) in LINES else "boxes")
        one.set_points(xg[P].contiguous())
        for a, b in zip((one.forward(fh[F]), *one.adjoint_backward(f[P].contiguous(), fh[F])), (fwd[P], gf[P], gx[P])):
            if N == (8, 8, 8):
                assert float((a - b).norm()) <= (1e-12 if prec == "f64" else 2e-6) * float(b.norm())
            else:
                assert torch.equal(a, b)
        ref = np.ravel(oracle_mod.ndft_adjoint(N, x[P], f[P].cpu().numpy().astype(np.complex128)))
        tol = 3 * H.window_error_bound(m, 2.0) * math.sqrt(max(1.0, M / 8)) + (1e-12 if prec == "f64" else 2e-5)
        assert oracle_mod.rel_l2(adj[F], ref) <= tol
        po, fo = P.stop, F.stop
