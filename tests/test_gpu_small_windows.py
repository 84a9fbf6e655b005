"""Spreads, interpolations and gradients against the windowed sums they stand for,
evaluated on the CPU with the library's window and roll-off factors: these agree to
rounding at every cut-off, where the direct sums differ by the window's error (25%
at m = 1).  Tolerances: 1e-12 (float64; ten times that for a gradient, whose terms
cancel) or 2e-5 (float32) of the result's l2 norm; every one far below the 1 that
an output of zeros would have.  And a NaN coordinate in the direct pair sum."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _windowed(H, N, x, f, fh, m):
    """(adjoint of f, forward of fh, derivatives of the forward (M, 3))."""
    n = [2 * v for v in N]
    phi, dphi, cell, roll = [], [], [], []
    for t in range(3):
        v = x[:, t] * n[t]
        c = np.floor(v)
        taps = np.arange(2 * m)
        p, d = H.window_eval(m, 2.0, ((v - c)[:, None] + (m - 1 - taps)[None, :]).ravel())
        phi.append(np.asarray(p).reshape(-1, 2 * m))
        dphi.append(np.asarray(d).reshape(-1, 2 * m) * n[t])
        cell.append(((c[:, None] - m + 1 + taps) % n[t]).astype(int))
        roll.append(np.asarray(H.window_rolloff(m, 2.0, n[t], N[t])))
    idx = np.ix_(*[np.arange(-v // 2, v // 2) % w for v, w in zip(N, n)])
    R = roll[0][:, None, None] * roll[1][None, :, None] * roll[2][None, None, :]
    grid = np.zeros(n, dtype=np.complex128)
    at = [(cell[0][j][:, None, None], cell[1][j][None, :, None], cell[2][j][None, None, :]) for j in range(len(x))]
    w = [np.einsum("a,b,c->abc", phi[0][j], phi[1][j], phi[2][j]) for j in range(len(x))]
    for j in range(len(x)):
        np.add.at(grid, at[j], f[j] * w[j])
    adj = np.fft.fftn(grid)[idx] * R
    grid = np.zeros(n, dtype=np.complex128)
    grid[idx] = fh * R
    grid = np.fft.ifftn(grid) * grid.size
    fwd = np.array([(grid[a] * v).sum() for a, v in zip(at, w)])
    der = np.empty((len(x), 3), dtype=np.complex128)
    for t in range(3):
        P = [dphi[u] if u == t else phi[u] for u in range(3)]
        for j in range(len(x)):
            der[j, t] = (grid[at[j]] * np.einsum("a,b,c->abc", P[0][j], P[1][j], P[2][j])).sum()
    return adj, fwd, der


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("how", ["boxes", "lines", "deterministic"])
@pytest.mark.parametrize("N,M,m", [((4, 6, 4), 64, 1), ((2, 2, 4), 40, 1), ((10, 8, 18), 333, 1), ((6, 10, 4), 300, 2),
                                   ((16, 12, 14), 65, 2), ((6, 8, 12), 129, 3), ((18, 20, 16), 400, 3),
                                   ((12, 8, 10), 257, 4), ((12, 14, 10), 200, 5), ((18, 20, 18), 150, 9)])
def test_windowed_sums(N, M, m, how, prec):
    from paper_2001_01583_amd import hpnfft as H
    g = W.rng(9100 + M + m)
    x = W.uniform_points(M, 3, g)
    x[0], x[-1] = -0.5, [0.5 - 1e-13, -0.5, 0.5 - 1e-13]
    x[1:M // 3] = W.wrap_unit(np.array([-0.49, 0.1, 0.49]) + 0.03 * g.standard_normal((M // 3 - 1, 3)))
    cd = torch.complex128 if prec == "f64" else torch.complex64
    f = torch.from_numpy(W.complex_normal(M, g)).to(cd)
    fh = torch.from_numpy(W.complex_normal(int(np.prod(N)), g).reshape(N)).to(cd)
    wf, wfh = (v.to(torch.complex128).numpy() for v in (f, fh))
    adj, fwd, der = _windowed(H, N, x, wf, wfh, m)
    refs = [adj, fwd, fwd, np.real(wf[:, None] * np.conj(der))]
    plan = H.Plan(N, M, m=m, precision=prec, with_grad=True,
                  **(dict(deterministic=True) if how == "deterministic" else dict(method=how)))
    plan.set_points(torch.from_numpy(x).cuda())
    gf, gx = plan.adjoint_backward(f.cuda(), fh.cuda().reshape(-1))
    outs = [plan.adjoint(f.cuda()), plan.forward(fh.cuda()), gf, gx]
    plain = H.Plan(N, M, m=m, precision=prec,
                   **(dict(deterministic=True) if how == "deterministic" else dict(method=how)))
    plain.set_points(torch.from_numpy(x).cuda())
    refs, outs = refs + [adj, fwd], outs + [plain.adjoint(f.cuda()), plain.forward(fh.cuda())]
    for k, (a, b) in enumerate(zip(outs, refs)):
        e = np.linalg.norm(a.cpu().numpy().astype(np.complex128) - b) / np.linalg.norm(b)
        print("windowed %s N=%s M=%d m=%d %s output %d: %.2e" % (how, N, M, m, prec, k, e))
        assert e <= (2e-5 if prec == "f32" else 1e-11 if k == 3 else 1e-12)


def test_nan_coordinate_reaches_the_direct_sum():
    from paper_2001_01583_amd import ewald as E
    g = W.rng(8200)
    r, q = torch.from_numpy(g.random((300, 3)) * 10.0).cuda(), torch.from_numpy(g.uniform(0.5, 2.0, 300)).cuda()
    r[17, 1] = math.nan
    ew = E.Ewald(300, 10.0, 1.0, N=(16, 16, 16), m=2, rcut=3.3, real_method="direct")
    e, F = ew.real_space(r, q)  # (a separation that is not a number is no distance beyond the cut-off)
    assert math.isnan(float(e)) and bool(torch.isnan(F).all(dim=1).all())
