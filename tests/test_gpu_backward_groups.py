"""The compositing backward's channel groups and its split of a walk.

Groups: a partly filled last group below and above the matrix-core limit
(10, 33 and 66 channel floats, 3 and 5 reals), a requested group.  Walks:
more than one 64-entry batch per tile, and counts of entries that leave the
four waves uneven quarters (48, 65 and 150 Gaussians, most of them reaching
every pixel box).  Tolerances as for the other backward tests: FP32 sums
against FP64, 2e-4 of the tensor's maximum, 2e-3 relative on entries above
1% of it.
"""
import numpy as np
import pytest
import torch

import paper_2511_22793_amd as gs
import synth
from gpu_util import oracle_params, to_dev
from test_gpu_backward import NAMES, close_scene, compare, torch_grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx,F,th,tw,group,n", [(False, 3, 16, 16, 0, 65), (False, 5, 8, 8, 0, 150),
                                                  (True, 5, 8, 32, 0, 48), (False, 33, 8, 16, 0, 150),
                                                  (True, 33, 16, 16, 0, 65), (True, 32, 16, 16, 64, 150),
                                                  (True, 4, 4, 64, 2, 65)])
def test_channel_groups_match_autograd_reference(cplx, F, th, tw, group, n):
    sc = close_scene(n, F + n)
    attr = synth.channel_attrs(n, F, cplx, seed=F)
    rx = [0.2, -0.1, 0.05]
    G = np.random.default_rng(F).normal(size=(F, 90, 360, 2) if cplx else (F, 90, 360))
    prm = gs.Params(T_min=0.0, chan_group=group)  # no stop: every walk reaches the end of its list
    ref = torch_grads(sc, attr, rx, G, oracle_params(prm), cplx=cplx)
    dev = to_dev(sc)
    a = torch.from_numpy(np.ascontiguousarray(attr, np.float32)).cuda()
    rx_t = torch.tensor([rx], dtype=torch.float32).cuda()
    out, ws = gs.forward(dev, a, rx_t, grid=gs.Grid(90, 360, th, tw), params=prm, is_complex=cplx)
    g = gs.backward(ws, dev, a, rx_t, out, torch.from_numpy(G[None].astype(np.float32)).cuda(), is_complex=cplx)
    for k in NAMES + ("attr",):
        compare(g["d_" + k].cpu().numpy(), ref[k], k)
