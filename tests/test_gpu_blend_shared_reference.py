"""Compositing of attribute sets over one shared geometry (the matrix-core
form, all columns of all sets after a pixel's walk) against the row form, one
channel of one set at a time (GS_OPT_BLEND_PER_GROUP with a channel group of
1): another kernel with its own walk loop and sums.  Both add a pixel's
entries in list order as one chain of fused multiply-adds, so spectra and
pixel state are the same bits, also past several weight buffers of 64 entries,
in partly filled column blocks and with the sets' columns cut into ranges.
"""
import numpy as np
import pytest
import torch

import paper_2511_22793_amd as gs
import synth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

STATE = ("T_final", "n_last", "n_contrib")


# (sets, channels, complex, tile (h, w), Gaussians, faint, (H, W))
CASES = [
    (16, 64, True, (16, 16), 3000, False, (90, 360)),   # the training shape
    (3, 8, True, (8, 32), 400, False, (90, 360)),       # 16 columns a set
    (1, 16, False, (8, 8), 300, False, (90, 360)),      # one block
    (2, 48, False, (32, 8), 500, False, (75, 333)),
    (3, 12, True, (16, 8), 400, False, (75, 333)),      # 24 columns: the second block partly filled
    (2, 9, False, (16, 16), 700, False, (45, 180)),
    (2, 16, True, (16, 16), 1500, True, (45, 180)),     # walks past several weight buffers
    (3, 5, True, (8, 16), 1500, True, (45, 180)),
    (3, 8, True, (16, 16), 5, False, (33, 70)),         # tiles without entries
]


@pytest.mark.parametrize("S,F,cplx,tile,n,faint,hw", CASES)
def test_shared_geometry_matches_single_channels(S, F, cplx, tile, n, faint, hw):
    sc = synth.scene(n, seed=7 * n + F, lo=[-3, -3, 0.1], hi=[3, 3, 2.5], log_scale_mean=-0.8 if faint else -1.3)
    if faint:
        sc["opacity_logit"] = np.full(n, -4.0, np.float32)
    sc, rx = to_dev(sc), torch.tensor([[0.1, -0.2, 0.3]]).cuda()
    attr = torch.from_numpy(np.stack([synth.channel_attrs(n, F, cplx, seed=10 * F + s) for s in range(S)])).cuda()
    grid, P = gs.Grid(hw[0], hw[1], *tile), hw[0] * hw[1]
    res = []
    for prm in (gs.Params(), gs.Params(blend_per_group=True, chan_group=1)):
        ws = gs.prepare(sc, rx, grid=grid, params=prm)
        out = gs.blend(ws, attr, n_sets=S, is_complex=cplx).clone()
        res.append((out, [ws.view(k, 0, P).clone() for k in STATE]))
    same = [torch.equal(a, b) for a, b in zip([res[0][0], *res[0][1]], [res[1][0], *res[1][1]])]
    assert all(same)
    if faint:
        assert int(res[0][1][2].max()) > 128
