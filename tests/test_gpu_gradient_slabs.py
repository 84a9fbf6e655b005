"""Float32 gradients of 2m = 8 line plans for every kind of cut a window can have:
slabs shallower than the window, slabs whose depth is no power of two, grids
that end within a slab, windows that wrap.  A point whose window meets one slab
only is summed as one part, bit for bit as in a plan with deeper slabs there;
all others to a few roundings of the 512 taps (2e-6 in the l2 norm)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [(4, 6, 5 * 2), (18, 12, 10), (30, 8, 8), (50, 4, 4)])
@pytest.mark.parametrize("Zs", [2, 3, 5, 7, 11, 12, 20, 24])
def test_gradient_slabs(N, Zs):
    from paper_2001_01583_amd import hpnfft as H
    M, n0 = 4001, 2 * N[0]
    g = W.rng(9700 + Zs)
    x = W.uniform_points(M, 3, g)
    x[0] = -0.5
    f = torch.from_numpy(W.complex_normal(M, g)).cuda().to(torch.complex64)
    fh = torch.from_numpy(W.complex_normal(int(np.prod(N)), g)).cuda().to(torch.complex64)
    out = []
    for zs in (Zs, 32):
        p = H.Plan(N, M, m=4, precision="f32", method="lines", with_grad=True, tiles=(8, zs, 512))
        p.set_points(torch.from_numpy(x).cuda())
        out.append([v.cpu().numpy() for v in p.adjoint_backward(f, fh)])
    first = np.floor(x[:, 0] * n0).astype(int) % n0 - 3
    whole = (first >= 0) & (first + 7 < n0) & (first // Zs == (first + 7) // Zs) & (first // 32 == (first + 7) // 32)
    assert whole.any() or Zs < 8 or N[0] < 6
    for a, b in zip(out[0], out[1]):
        assert np.array_equal(a[whole], b[whole])
        assert np.linalg.norm((a - b).astype(np.complex128)) <= 2e-6 * np.linalg.norm(b.astype(np.complex128))
    one = H.Plan(N, M, m=4, precision="f64", method="boxes", with_grad=True)
    one.set_points(torch.from_numpy(x).cuda())
    for a, b in zip(out[0], one.adjoint_backward(f.to(torch.complex128), fh.to(torch.complex128))):
        b = b.cpu().numpy()
        assert np.linalg.norm(a - b) <= 2e-5 * np.linalg.norm(b)
