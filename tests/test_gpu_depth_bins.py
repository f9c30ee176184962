"""The depth order where a bin of the splitter sort takes 16 keys per thread
(2049 to 4096 keys) and just beyond: scenes built so that one bin holds
everything that the sample left out, and an ordinary scene whose largest bin
is of that size."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_22793_amd as gs
import synth
import test_gpu_depth_order as depth
from gpu_util import to_dev
from test_depth_bins_cpu import _largest_bin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4100, 4160, 4161])  # bins of 4036, 4096 and 4097 keys
def test_one_large_bin(n):
    depth.test_depth_order_exact(n, "missed")


def test_ordinary_scene_with_a_large_bin():
    n, rx = 2 ** 19, np.array([[0.5, -0.25, 0.1]], np.float32)
    sc = synth.scene(n, seed=52)
    sc["log_scale"] = np.full_like(sc["log_scale"], -6.0)
    p = oracle.project(sc, rx[0], 32, 64)
    order = oracle.depth_order(p)
    key = np.full(n, 0xFFFFFFFF, np.uint32)
    key[order] = p["r32"][order].view(np.uint32)
    assert 2048 < _largest_bin(key) <= 4096
    ws = gs.prepare(to_dev(sc), torch.from_numpy(rx).cuda(), grid=gs.Grid(32, 64),
                    params=gs.Params(pair_capacity=16 * n + 4096, forward_only=True))
    got = ws.view("order", 0, n, torch.int32).cpu().numpy()
    assert np.array_equal(got, np.concatenate([order, np.setdiff1d(np.arange(n), order)]))
