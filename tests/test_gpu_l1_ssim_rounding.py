"""Rounding of the magnitude-spectrum loss's gradient: no further from 64 bits
than the plain FP32 evaluation, every map filtered apart (the two variances
too) with one rounding per tap, which is emulated here on the same inputs.
"""
import numpy as np
import pytest
import torch

import paper_2511_22793_amd as gs

pytestmark = pytest.mark.gpu

TAPS = np.exp(-(np.arange(11) - 5.0) ** 2 / (2 * 1.5 ** 2))
TAPS /= TAPS.sum()
LAMBDA = 0.2


def _filter(v):
    taps = TAPS.astype(v.dtype).astype(np.float64)
    for axis in (2, 1):
        pad = [(0, 0)] * 3
        pad[axis] = (5, 5)
        p = np.pad(v, pad).astype(np.float64)
        out = np.zeros_like(v)
        for k, w in enumerate(taps):  # a fused multiply-add per tap
            out = (w * np.take(p, range(k, k + v.shape[axis]), axis) + out).astype(v.dtype)
        v = out
    return v


def _gradient(x, y, dt):
    x, y, one = x.astype(dt), y.astype(dt), dt(1)
    c1, c2 = dt(0.01) ** 2, dt(0.03) ** 2
    mx, my = _filter(x), _filter(y)
    sxx, syy, sxy = _filter(x * x) - mx * mx, _filter(y * y) - my * my, _filter(x * y) - mx * my
    a1, a2, b1, b2 = 2 * mx * my + c1, 2 * sxy + c2, mx * mx + my * my + c1, sxx + syy + c2
    s = a1 * a2 / (b1 * b2)
    d = s * (my * (2 / a1 - 2 / a2) - 2 * mx * (one / b1 - one / b2))
    g = _filter(d) + 2 * x * _filter(-s / b2) + y * _filter(2 * s / a2)
    return (dt(1 - LAMBDA) * np.sign(x - y) - dt(LAMBDA) * g) / dt(x.size)


def _spectra(seed, S, H, W):
    """Blobs of a few paths, and a noisy estimate of them."""
    r = np.random.default_rng(seed)
    yy, xx = np.mgrid[:H, :W]
    z = np.zeros((S, H, W))
    for _ in range(48):
        cx, cy, wx, wy = r.uniform(0, W), r.uniform(0, H), r.uniform(W / 90, W / 12), r.uniform(H / 45, H / 6)
        blob = np.exp(-0.5 * ((xx - cx) / wx) ** 2 - 0.5 * ((yy - cy) / wy) ** 2)
        z += r.uniform(-1, 1, (S, 1, 1)) * blob
    z = np.abs(z) / np.abs(z).max()
    return np.clip(z + r.normal(0, 0.05, z.shape), 0, 1).astype(np.float32), z.astype(np.float32)


@pytest.mark.parametrize("S,H,W", [(8, 90, 360), (6, 75, 333)])
def test_gradient_no_further_off_than_plain_fp32(S, H, W):
    x, y = _spectra(H, S, H, W)
    d = gs.loss_l1_ssim(torch.from_numpy(x[:, None]).cuda(), torch.from_numpy(y[:, None]).cuda(), LAMBDA)[3]
    got = d[:, 0].double().cpu().numpy()
    ref = _gradient(x, y, np.float64)
    err, plain = float(np.linalg.norm(got - ref)), float(np.linalg.norm(_gradient(x, y, np.float32) - ref))
    assert err <= plain
