"""Rounding of the attribute gradients summed over the image.

A Gaussian that covers the whole image takes a term from every 64 pixels of
every receiver; the terms are summed per tile before they join the Gaussian's
FP32 sum, which would round four times as often without.  The scene: K faint
Gaussians that cover the image, a wall that stops every pixel, and thousands
behind it that no pixel reaches.  The reference sums the same weights (a
forward of one-hot attributes gives them) in FP64; the tolerance is the
geometric mean of the errors of FP32 sums of the tiles' and of the 64-pixel
boxes' terms, in a random order.
"""
import numpy as np
import pytest
import torch

import paper_2511_22793_amd as gs
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

H, W, K, WALL, BEHIND, B = 90, 360, 24, 12, 3000, 8


def _scene():
    rng = np.random.default_rng(5)
    n = K + WALL + BEHIND
    d = rng.normal(size=(n, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    d[:, 2] = np.abs(d[:, 2])  # the upper half space
    r = np.concatenate([np.linspace(2.0, 3.0, K), np.full(WALL, 4.0), np.linspace(6.0, 8.0, BEHIND)])
    q = rng.normal(size=(4, n))
    return {"mean": (d * r[:, None]).T.astype(np.float32).copy(),
            "log_scale": np.broadcast_to(np.log(5 * r), (3, n)).astype(np.float32).copy(),
            "quat": (q / np.linalg.norm(q, axis=0)).astype(np.float32),
            "opacity_logit": np.where(np.arange(n) < K, -4.0, 8.0).astype(np.float32)}


def _rms(x, ref):
    return float(np.sqrt((((x - ref) / ref) ** 2).mean()))


def _running(terms, rng):
    """Each column's FP32 running sum over the rows in a random order."""
    t = terms[rng.permutation(len(terms))].astype(np.float32)
    return np.add.accumulate(t, axis=0, dtype=np.float32)[-1].astype(np.float64)


# (channels, complex, channel group, tile): one value per entry, butterfly
# groups, matrix-core groups, more than one group
@pytest.mark.parametrize("F,cplx,group,tile", [(1, False, 0, (16, 16)), (1, False, 0, (32, 8)), (3, False, 0, (16, 16)),
                                               (3, False, 1, (16, 16)), (8, True, 0, (16, 16)),
                                               (35, True, 0, (8, 32))])
def test_attribute_gradients_sum_per_tile(F, cplx, group, tile):
    sc = to_dev(_scene())
    n = K + WALL + BEHIND
    gen = torch.Generator(device="cuda").manual_seed(F)
    rx = 0.05 * torch.randn(B, 3, generator=gen, device="cuda")
    grid = gs.Grid(H, W, *tile)
    prm = gs.Params(pair_capacity=n * 200, chan_group=group)
    eye = torch.zeros(n, K, device="cuda")
    eye[:K] = torch.eye(K, device="cuda")
    w, _ = gs.forward(sc, eye, rx, grid=grid, params=gs.Params(pair_capacity=n * 200, chan_group=1))
    attr = torch.rand((n, F, 2) if cplx else (n, F), generator=gen, device="cuda")
    out, ws = gs.forward(sc, attr, rx, grid=grid, params=prm, is_complex=cplx)
    up = torch.rand(out.shape, generator=gen, device="cuda")
    got = gs.backward(ws, sc, attr, rx, out, up, is_complex=cplx)["d_attr"].reshape(n, -1)
    assert int(ws.view("n_last", 0, H * W).max()) <= K + WALL
    assert float(got[K + WALL:].abs().max()) == 0.0
    got = got[:K].double().cpu().numpy()
    # the terms of every 64-pixel box: [receiver, tile row, tile column, box, K, columns]
    th, tw = tile
    bh = max(1, 64 // tw)
    up = up.permute(0, 1, 4, 2, 3).reshape(B, -1, H, W) if cplx else up
    pad = (0, -W % tw, 0, -H % th)
    w, up = (torch.nn.functional.pad(x.double(), pad) for x in (w, up))
    ty, tx = w.shape[2] // th, w.shape[3] // tw
    split = lambda x: x.reshape(B, -1, ty, th // bh, bh, tx, tw).permute(0, 2, 5, 3, 1, 4, 6).flatten(-2)  # noqa: E731
    box = (split(w) @ split(up).transpose(-1, -2)).reshape(B * ty * tx, th // bh, -1).cpu().numpy()
    ref = box.sum((0, 1))
    rng = np.random.default_rng(1)
    per_tile = box.astype(np.float32).sum(1, dtype=np.float32)
    e_tile = np.mean([_rms(_running(per_tile, rng), ref) for _ in range(4)])
    e_box = np.mean([_rms(_running(box.reshape(-1, box.shape[-1]), rng), ref) for _ in range(4)])
    assert e_box > 1.5 * e_tile  # the two can be told apart
    assert _rms(got.reshape(-1), ref) <= np.sqrt(e_tile * e_box)
