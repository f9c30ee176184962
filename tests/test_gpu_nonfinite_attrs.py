"""Attributes that are not finite reach the pixels that composite them: a
pixel that stopped in front of such a Gaussian holds the same bits as with its
attributes zero, also beside pixels of its tile that go on; and one behind
every pixel's stop changes nothing, in any form of the compositing.  Which
pixels composite a Gaussian: a render of one-hot attributes, one channel at a
time.
"""
import numpy as np
import pytest
import torch

import paper_2511_22793_amd as gs
import synth
from gpu_util import to_dev
from paper_2511_22793_amd import serve

pytestmark = pytest.mark.gpu

H, W, N = 45, 180, 64
VALUES = (float("nan"), float("inf"), -float("inf"))


def _scene(wall):
    """Eight faint Gaussians, sixteen opaque ones (wall: wider than the image,
    so that every pixel stops at the second, else small, so that some pixels
    stop and others do not), and faint ones behind, all of these as wide as
    the image."""
    rng = np.random.default_rng(2)
    d = rng.normal(size=(N, 3))
    d[:, 2] = np.abs(d[:, 2])
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    r = np.linspace(2.0, 5.0, N)
    opaque = (np.arange(N) >= 8) & (np.arange(N) < 24)
    scale = np.log(np.where(opaque, 50.0 if wall else 0.6, 5.0) * r)
    return to_dev({"mean": (d * r[:, None]).T.astype(np.float32).copy(),
                   "log_scale": np.broadcast_to(scale, (3, N)).astype(np.float32).copy(),
                   "quat": np.tile(np.array([[1.0], [0], [0], [0]], np.float32), (1, N)),
                   "opacity_logit": np.where(opaque, 8.0, -2.0).astype(np.float32)})


def _params(group=0):
    return gs.Params(pair_capacity=N * 64 * 4, chan_group=group)


def _weighs(sc, rx, grid):
    """[receivers, N, H, W]: the pixel composites the Gaussian."""
    hot = torch.eye(N, device="cuda")
    return gs.forward(sc, hot, rx, grid=grid, params=_params(1))[0] != 0.0


def _attrs(F, cplx, seed, where):
    a = torch.from_numpy(synth.channel_attrs(N, F, cplx, seed=seed)).cuda()
    bad, zero = a.clone(), a.clone()
    for k, g in enumerate(where):
        bad[g] = VALUES[k % 3]
        zero[g] = 0.0
        if k % 4 == 3:  # a single channel
            bad[g] = 0.0
            bad[g].view(-1)[-1] = VALUES[0]
    return bad, zero


def _check(out, ref, hit):
    """out, ref: [sets, F, H, W(, 2)]; hit: [sets, H, W]."""
    clean = ~hit[:, None].expand(out.shape[:4])
    same = torch.equal(out[clean], ref[clean])
    assert same
    if bool(hit.any()):
        assert not bool(torch.isfinite(out[~clean]).any())


RX = torch.tensor([[0.0, 0.0, 0.0], [0.1, -0.05, 0.02]])


# row forms, matrix-core blocks that are partly filled, 64-bit addressing
# ("odd": a spectrum that only 4-byte accesses reach)
@pytest.mark.parametrize("F,cplx,group,tile,odd", [(1, False, 0, (16, 16), False), (2, True, 0, (8, 16), False),
                                                   (7, False, 0, (8, 8), False), (9, False, 0, (16, 16), False),
                                                   (5, True, 0, (8, 32), False), (16, True, 4, (16, 16), False),
                                                   (5, True, 0, (16, 16), True), (24, False, 0, (16, 16), False)])
def test_stopped_pixels_beside_others(F, cplx, group, tile, odd):
    sc, rx, grid = _scene(False), RX.cuda(), gs.Grid(H, W, *tile)
    w = _weighs(sc, rx, grid)
    where = [g for g in range(24, N, 5)]
    hit = w[:, where].any(1)  # the others stopped in front of them all
    assert 0.05 < float(hit.float().mean()) < 0.95
    bad, zero = _attrs(F, cplx, F, where)
    bad[where] = torch.where(torch.isfinite(bad[where]), VALUES[0], bad[where])  # every channel
    shape = (2, F, H, W) + ((2,) if cplx else ())
    size = int(np.prod(shape))
    buf = torch.empty(size + 1, device="cuda")[int(odd):][:size].view(shape)
    ref, _ = gs.forward(sc, zero, rx, grid=grid, params=_params(group), is_complex=cplx)
    gs.forward(sc, bad, rx, grid=grid, params=_params(group), is_complex=cplx, out=buf)
    _check(buf, ref, hit)
    batch = serve.Batch([serve.Job(sc, bad, rx, cplx, grid, _params(group))])
    batch.run()
    _check(batch.spectra[0], ref, hit)
    # the fused loss, one receiver
    ws = gs.prepare(sc, rx[:1].contiguous(), grid=grid, params=_params())
    out = gs.blend_loss(ws, bad, torch.rand(ref[:1].shape, device="cuda"), is_complex=cplx)[0]
    _check(out, ref[:1], hit[:1])


@pytest.mark.parametrize("F,cplx,tile", [(1, False, (16, 16)), (8, False, (8, 8)), (5, True, (16, 16)),
                                         (16, False, (16, 16)), (16, True, (8, 16)), (64, True, (16, 16))])
def test_behind_every_stop(F, cplx, tile):
    sc, rx, grid = _scene(True), torch.zeros(2, 3, device="cuda"), gs.Grid(H, W, *tile)
    w = _weighs(sc, rx, grid)
    where = torch.nonzero(~w.any(3).any(2).any(0))[:, 0].tolist()[1:]  # from the first one behind the stops on
    assert where[0] == 10
    bad, zero = _attrs(F, cplx, F, where)
    none = torch.zeros(2, H, W, dtype=torch.bool, device="cuda")
    ref, _ = gs.forward(sc, zero, rx, grid=grid, params=_params(), is_complex=cplx)
    out, _ = gs.forward(sc, bad, rx, grid=grid, params=_params(), is_complex=cplx)
    _check(out, ref, none)
    ws = gs.prepare(sc, rx[:1].contiguous(), grid=grid, params=_params())
    sets = torch.stack([bad, bad])
    shared = gs.blend(ws, sets, n_sets=2, is_complex=cplx).clone()
    _check(shared, ref[:1].expand_as(shared), none)
    up = torch.rand(out.shape, device="cuda")
    out, ws = gs.forward(sc, bad, rx, grid=grid, params=_params(), is_complex=cplx)
    for g in gs.backward(ws, sc, bad, rx, out, up, is_complex=cplx).values():
        assert bool(torch.isfinite(g).all())
