"""The forms of the compositing against each other.

Every form adds a pixel's entries in list order as one chain of fused
multiply-adds, so the matrix-core form (blocks of 16 or 32 columns, step
counts rounded up with zero weights, weight buffers flushed in between,
64-bit addressing) must give the bits of the one-channel-at-a-time form.  The
dealt and the counted part of the persistent launch must give those of the
grid-mapped one whatever the number of workgroups.
"""
import numpy as np
import pytest
import torch

import paper_2511_22793_amd as gs
import synth
from gpu_util import to_dev
from paper_2511_22793_amd import serve

pytestmark = pytest.mark.gpu

RX = np.array([[0.1, -0.2, 0.3], [2.5, -1.0, 1.4]], np.float32)


def _scene(n, seed, faint):
    sc = synth.scene(n, seed=seed, lo=[-3, -3, 0.1], hi=[3, 3, 2.5], log_scale_mean=-0.8 if faint else -1.3)
    if faint:  # walks of several weight buffers
        sc["opacity_logit"] = np.full(n, -4.0, np.float32)
    return to_dev(sc)


# (channels, complex, tile, Gaussians, faint, grid): channel floats 9 (one
# masked block), 10, 24, 48 (blocks of 16), 32, 128 (blocks of 32), 16 real
CASES = [
    (9, False, (16, 16), 300, False, (90, 360)),
    (5, True, (8, 16), 700, False, (75, 333)),
    (12, True, (8, 8), 20, False, (45, 180)),
    (24, True, (32, 8), 1500, True, (45, 180)),
    (16, True, (16, 16), 1500, True, (50, 130)),
    (64, True, (8, 32), 1200, False, (50, 130)),
    (16, False, (16, 16), 5, False, (33, 70)),
]


@pytest.mark.parametrize("F,cplx,tile,n,faint,hw", CASES)
def test_column_blocks_match_single_channels(F, cplx, tile, n, faint, hw):
    sc = _scene(n, 3 * n + F, faint)
    grid = gs.Grid(hw[0], hw[1], tile[0], tile[1])
    rx = torch.from_numpy(RX).cuda()
    attr = torch.from_numpy(synth.channel_attrs(n, F, cplx, seed=n)).cuda()
    ref, wr = gs.forward(sc, attr, rx, grid=grid, params=gs.Params(chan_group=1), is_complex=cplx)
    out, ws = gs.forward(sc, attr, rx, grid=grid, is_complex=cplx)
    assert torch.equal(out, ref)
    # a spectrum (and attributes) that only 4-byte accesses reach
    odd = torch.empty(out.numel() + 1, device="cuda")[1:].view(out.shape)
    aodd = torch.empty(attr.numel() + 1, device="cuda")[1:].view(attr.shape)
    aodd.copy_(attr)
    gs.forward(sc, aodd, rx, grid=grid, is_complex=cplx, out=odd)
    assert torch.equal(odd, ref)
    P = hw[0] * hw[1]
    for q in range(2):
        for k in ("T_final", "n_last", "n_contrib"):
            assert torch.equal(ws.view(k, q, P), wr.view(k, q, P))
    if faint:
        assert int(ws.view("n_contrib", 0, P).max()) > 128


@pytest.mark.parametrize("workgroups", [1, 7, 100_000])
def test_persistent_items_dealt_and_counted(workgroups):
    jobs = []
    for i, (F, cplx, n) in enumerate(((1, False, 400), (5, True, 300), (16, True, 500), (64, True, 200))):
        jobs.append(serve.Job(_scene(n, 40 + i, False), torch.from_numpy(synth.channel_attrs(n, F, cplx, seed=i)).cuda(),
                              torch.from_numpy(RX).cuda(), cplx, gs.Grid(45, 180)))
    b = serve.Batch(jobs, workgroups=workgroups)
    for s in b.spectra:
        s.fill_(-1.0)
    b.run()
    for j, s in zip(b.jobs, b.spectra):
        ref, _ = gs.forward(j.scene, j.attr, j.rx, grid=j.grid, params=j.params, is_complex=j.is_complex)
        assert torch.equal(s, ref)
