"""Real-space pair kernels (Eq. (11)) at the edges of their tiles: one ion,
queues that never fill, more partners than one LDS tile holds (4096), ions
past the last whole group of 256, pair distances from 1e-6 to beyond the
cut-off (alpha r up to 12), and NaN coordinates.  Reference: the pair sum in
float64 torch operations.  Tolerance: sums of at most 2e4 terms of both signs,
1e-12 of the largest force and of the sum of |terms| for the energy."""
import ctypes
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _reference(r, q, L, alpha, rcut):
    D = r[:, None, :] - r[None, :, :]
    D -= L * torch.round(D / L)
    d2 = (D * D).sum(-1)
    near = (d2 < rcut * rcut) & ~torch.eye(len(r), dtype=torch.bool, device=r.device)
    d = torch.sqrt(torch.where(near, d2, torch.ones_like(d2)))
    qq = q[:, None] * q[None, :]
    ec = torch.where(near, torch.erfc(alpha * d) / d, torch.zeros_like(d))
    g = torch.where(near, qq * (ec + 2 * alpha / math.sqrt(math.pi) * torch.exp(-alpha * alpha * d2)) / d ** 2,
                    torch.zeros_like(d))
    return 0.5 * (qq * ec).sum(), 0.5 * (qq * ec).abs().sum(), (g[..., None] * D).sum(1)


def _run(r, q, L, alpha, rcut, method):
    from paper_2001_01583_amd import ewald as E
    ew = E.Ewald(len(r), L, alpha, N=(16, 16, 16), m=2, rcut=rcut, real_method=method)
    return ew.real_space(r, q)


def _ions(M, L, close, g):
    r = g.random((M, 3)) * L
    if close:  # partners at every distance scale
        k = M // 2
        step = g.standard_normal((k, 3))
        step /= np.linalg.norm(step, axis=1, keepdims=True)
        r[:k] = r[M - k:] + step * 10.0 ** g.uniform(-6, 0, (k, 1))
    q = np.where(g.random(M) < 0.5, 1.0, -1.0) * g.uniform(0.5, 2.0, M)
    return torch.from_numpy(r).cuda(), torch.from_numpy(q).cuda()


@pytest.mark.parametrize("method", ["direct", "cells"])
@pytest.mark.parametrize("M,L,rcut,alpha,close", [
    (1, 10.0, 3.0, 1.0, False), (2, 10.0, 3.0, 1.0, True), (65, 10.0, 3.2, 1.5, True), (257, 12.0, 4.0, 0.3, False),
    (4097, 12.0, 4.0, 3.0, True), (5000, 9.0, 2.9, 1.0, False), (3000, 30.0, 3.0, 4.0, True)])
def test_pair_sums(M, L, rcut, alpha, close, method):
    r, q = _ions(M, L, close, W.rng(8000 + M))
    e, F = _run(r, q, L, alpha, rcut, method)
    er, ea, Fr = _reference(r, q, L, alpha, rcut)
    big = max(float(Fr.abs().max()), 1e-300)
    print("pairs %s M=%d: energy %.2e force %.2e" % (method, M, abs(float(e - er)) / max(float(ea), 1e-300),
                                                     float((F - Fr).abs().max()) / big))
    assert abs(float(e - er)) <= 1e-12 * float(ea)
    assert float((F - Fr).abs().max()) <= 1e-12 * big if M > 1 else float(F.abs().max()) == 0.0


@pytest.mark.parametrize("method", ["direct", "cells"])
def test_pair_nan_reaches_the_sums(method):
    r, q = _ions(300, 10.0, False, W.rng(8100))
    q[17] = float("nan")
    e, F = _run(r, q, 10.0, 1.0, 3.3, method)
    assert math.isnan(float(e)) and bool(torch.isnan(F[17]).all())
