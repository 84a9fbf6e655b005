"""Interpolation by gathering (one wavefront per point, every window width,
box and line records): the forward of sparse sets and of deterministic plans,
and the gradients of every plan, against the direct sums.  Grids as small as
the window, edges that are no multiple of 2m, points at both ends of the
domain, more workgroups than one share per XCD and fewer (M = 1).  Tolerances:
the window's a-priori bound (d E, times 2 pi n / 2 for a derivative) plus
1e-12 (float64) or 2e-5 (float32) of rounding."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _tol(H, m, prec, n, grad):
    e = 3 * H.window_error_bound(m, 2.0)
    # the bound is relative to ||input||_1; the inputs here are N(0, 1), so
    # relative to the result's l2 norm it grows by at most sqrt(#inputs)
    e *= math.sqrt(float(np.prod(n)) / 8)
    return e * (math.pi * max(n) if grad else 1.0) + (1e-12 if prec == "f64" else 2e-5) * (10 if grad else 1)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("method", ["boxes", "lines"])
@pytest.mark.parametrize("N,M,m", [((8, 8, 8), 1, 8), ((8, 10, 14), 333, 8), ((12, 6, 10), 500, 5), ((6, 10, 4), 777, 2),
                                   ((10, 12, 14), 1000, 7), ((12, 8, 16), 2049, 4), ((16, 18, 20), 100, 9),
                                   ((4, 6, 4), 64, 1), ((6, 8, 12), 129, 3), ((16, 14, 12), 400, 6)])
def test_gather(oracle_mod, N, M, m, method, prec):
    from paper_2001_01583_amd import hpnfft as H
    g = W.rng(9000 + M + m)
    x = W.uniform_points(M, 3, g)
    x[0] = -0.5
    x[-1] = [0.5 - 1e-13, -0.5, 0.5 - 1e-13] if M > 1 else -0.5
    cd = torch.complex128 if prec == "f64" else torch.complex64
    f = torch.from_numpy(W.complex_normal(M, g)).to(cd)
    fh = torch.from_numpy(W.complex_normal(int(np.prod(N)), g).reshape(N)).to(cd)
    f64, fh64 = (v.to(torch.complex128).numpy() for v in (f, fh))
    n = [2 * v for v in N]
    plan = H.Plan(N, M, m=m, precision=prec, method=method, with_grad=True)
    plan.set_points(torch.from_numpy(x).cuda())
    gf, gx = plan.adjoint_backward(f.cuda(), fh.cuda().reshape(-1))
    ref = oracle_mod.ndft_forward(N, x, fh64)
    k = [np.arange(-v // 2, v // 2) for v in N]
    refx = np.stack([np.real(f64 * np.conj(oracle_mod.ndft_forward(
        N, x, fh64 * (2j * np.pi * k[t]).reshape([-1 if u == t else 1 for u in range(3)])))) for t in range(3)], 1)
    ef = oracle_mod.rel_l2(gf.cpu().numpy().astype(np.complex128), ref)
    ex = np.linalg.norm(gx.cpu().numpy().astype(np.float64) - refx) / np.linalg.norm(refx)
    print("gather %s N=%s M=%d m=%d %s: grad_f %.2e grad_x %.2e" % (method, N, M, m, prec, ef, ex))
    assert ef <= _tol(H, m, prec, n, False) and ex <= _tol(H, m, prec, n, True)
    if method == "boxes":
        for det in (False, True):
            p = H.Plan(N, M, m=m, precision=prec, method=method, deterministic=det)
            p.set_points(torch.from_numpy(x).cuda())
            out = p.forward(fh.cuda()).cpu().numpy().astype(np.complex128)
            assert oracle_mod.rel_l2(out, ref) <= _tol(H, m, prec, n, False)


@pytest.mark.parametrize("N,Zs", [((18, 12, 10), 8), ((24, 10, 8), 16), ((20, 10, 10), 24)])
def test_float32_gradient_sums_do_not_depend_on_slabs_met(N, Zs):
    """Float32 line gradients sum a window in the parts its slabs cut it into:
    a point whose window meets one slab only is summed as one part, whatever
    the slab depth, so plans of different depths agree bit for bit there."""
    from paper_2001_01583_amd import hpnfft as H
    M = 3000
    g = W.rng(9500 + Zs)
    x = W.uniform_points(M, 3, g)
    f = torch.from_numpy(W.complex_normal(M, g)).cuda().to(torch.complex64)
    fh = torch.from_numpy(W.complex_normal(int(np.prod(N)), g)).cuda().to(torch.complex64)
    n0 = 2 * N[0]
    out = []
    for zs in (Zs, 32):  # (gradient plans take slabs of up to 32 planes here)
        p = H.Plan(N, M, m=4, precision="f32", method="lines", with_grad=True, tiles=(8, zs, 512))
        p.set_points(torch.from_numpy(x).cuda())
        out.append([v.cpu().numpy() for v in p.adjoint_backward(f, fh)])
    first = np.floor(x[:, 0] * n0).astype(int) % n0 - 3
    whole = (first >= 0) & (first + 7 < n0) & (first // Zs == (first + 7) // Zs) & (first // 32 == (first + 7) // 32)
    assert whole.any()
    for a, b in zip(out[0], out[1]):
        assert np.array_equal(a[whole], b[whole])
        assert np.linalg.norm((a - b).astype(np.complex128)) <= 2e-6 * np.linalg.norm(b.astype(np.complex128))
