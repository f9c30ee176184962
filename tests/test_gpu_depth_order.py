"""The depth order (exact, ties by index) at the edges of its paths: ranking
all against all (up to 4096 keys), sampled splitters (up to 2^19), the radix sort
beyond; equal distances; and a scene built so that the sample misses almost
every key's range, which leaves one bin too large for a workgroup's LDS.
Bit-exact against a stable sort of the oracle's FP32 distances.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_22793_amd as gs
import synth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


def _sample_places(n):
    bins = 16
    while bins < 1024 and n // bins > 320:
        bins *= 2
    m = 4 * bins
    i = np.arange(m, dtype=np.uint64)
    h = (i * 0x9E3779B1) & 0xFFFFFFFF
    return (i * n // m + (h * (n // m) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("n,kind", [(1, "plain"), (65, "ties"), (512, "plain"), (513, "ties"),
                                    (2048, "plain"), (2049, "plain"), (4095, "plain"), (4096, "ties"),
                                    (4097, "plain"), (6145, "ties"), (20_000, "missed"), (9000, "missed"),
                                    (2 ** 19, "plain"), (2 ** 19 + 1, "ties")])
def test_depth_order_exact(n, kind):
    sc = synth.scene(n, seed=n % 97)
    rx = np.array([[0.0, 0.0, 0.0], [0.5, -0.25, 0.1]], np.float32)
    rng = np.random.default_rng(n)
    if kind == "ties":  # a few distinct places
        sc["mean"] = np.ascontiguousarray(sc["mean"][:, rng.integers(0, min(n, 37), n)])
    if kind == "missed":  # the sampled keys far away, all others close together
        far = np.zeros(n, bool)
        far[_sample_places(n)] = True
        d = rng.normal(size=(n, 3))
        d[:, 2] = np.abs(d[:, 2]) + 0.1
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        sc["mean"] = (d * np.where(far, 9.0 + rng.random(n), 3.0 + 0.01 * rng.random(n))[:, None]).T.astype(np.float32).copy()
    sc["log_scale"] = np.full_like(sc["log_scale"], -6.0)  # few tiles each
    prm = gs.Params(pair_capacity=16 * n + 4096, forward_only=True)
    ws = gs.prepare(to_dev(sc), torch.from_numpy(rx).cuda(), grid=gs.Grid(32, 64), params=prm)
    torch.cuda.synchronize()
    for q in range(2):
        p = oracle.project(sc, rx[q], 32, 64)
        order = oracle.depth_order(p)
        culled = np.setdiff1d(np.arange(n), order)
        got = ws.view("order", q, n, torch.int32).cpu().numpy()
        keys = ws.view("keys", q, n, torch.int32).cpu().numpy().view(np.uint32)
        assert np.array_equal(got, np.concatenate([order, culled]))
        assert np.array_equal(keys[:len(order)], p["r32"][order].view(np.uint32))
        assert np.all(keys[len(order):] == 0xFFFFFFFF)
        # the scan of the tile counts behind it (8193 block sums at the largest)
        tiles = ws.view("tinfo", q, 4 * n, torch.int32).cpu().numpy().reshape(n, 4)[:, 3]
        f = ws.flags()[q]
        assert f["n_visible"] == len(order) and f["n_pairs"] == int(tiles[order].astype(np.int64).sum())
