"""GPU tests of the periodic box's transforms (csrc/fourier.h) at every size: each mix of radices, rows per block
and thread groups, every combination of outputs, against numpy's FFTs and the multiplier in FP64.

Bar: an FFT's error is a few roundings (2.2e-16) per radix-2 stage of the largest value; 2e-15 per stage over the
4 lg M stages of a forward and an inverse 2-D transform.  Point values (non-uniform FFT) add 1e-14 of sum |u^|
(its kernel's truncation)."""
import numpy as np
import pytest
import torch

from paper_1908_07392_amd import mhlp

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("M", [16, 32, 64, 128, 256, 512, 1024, 2048])
def test_particular_at_every_size(M):
    rng = np.random.default_rng(M)
    x0, y0, Lb, alpha, n = -1.0, 0.5, 3.0, 7.0, 37
    F = rng.standard_normal((2, M, M))
    px, py = x0 + Lb * rng.uniform(-0.2, 1.2, n), y0 + Lb * rng.uniform(-0.2, 1.2, n)
    k = 2 * np.pi / Lb * np.fft.fftfreq(M, 1.0 / M)
    k1, k2 = np.meshgrid(k, k, indexing="xy")
    kk = np.where(k1 * k1 + k2 * k2 > 0, k1 * k1 + k2 * k2, 1.0)
    f = np.fft.fft2(F) / M ** 2
    f[:, M // 2, :] = f[:, :, M // 2] = 0.0
    div = (k1 * f[0] + k2 * f[1]) / kk
    den = alpha ** 2 + np.where(k1 * k1 + k2 * k2 > 0, kk, 0.0)
    uh = np.stack([(f[0] - k1 * div) / den, (f[1] - k2 * div) / den])
    gh = np.stack([1j * k1 * uh[0], 1j * k2 * uh[0], 1j * k1 * uh[1], 1j * k2 * uh[1]])
    u, g = np.fft.ifft2(uh).real * M ** 2, np.fft.ifft2(gh).real * M ** 2
    ex, ey = np.exp(1j * np.outer(px - x0, k)), np.exp(1j * np.outer(py - y0, k))
    up = np.stack([np.einsum("pj,ji,pi->p", ey, c, ex, optimize=True).real for c in uh])
    bar = 4 * np.log2(M) * 2e-15
    B = mhlp.Box(M, x0, y0, Lb, alpha)
    for want_u, want_grad, points in ((True, True, True), (True, False, False), (False, True, False),
                                      (False, False, True), (True, False, True)):
        pts = dict(px=_t(px), py=_t(py)) if points else {}
        ru, rg, rp = B.particular(_t(F), want_u=want_u, want_grad=want_grad, **pts)
        if want_u:
            assert np.abs(ru.cpu().numpy() - u).max() <= bar * np.abs(u).max()
        if want_grad:
            assert np.abs(rg.cpu().numpy() - g).max() <= bar * np.abs(g).max()
        if points:
            assert np.abs(rp.cpu().numpy() - up).max() <= bar * np.abs(up).max() + 1e-14 * np.abs(uh).sum()
    B.set_point_method(0)
    rp = B.particular(_t(F), want_u=False, px=_t(px), py=_t(py))[2]
    assert np.abs(rp.cpu().numpy() - up).max() <= bar * np.abs(up).max() + 1e-14 * np.abs(uh).sum()
