"""The training pass's pairs of groups and target loads at their edges: an odd
tile width inside the image (single-word target loads), groups of a tile
partly or wholly outside the image, tiles of one group, and pairs whose
members fall in different walk classes (a faint cluster over a few rows:
walks of more than 64, 128 and 256 entries next to short ones).  Against the
unfused path, with the tolerances of the other training tests.
"""
import numpy as np
import pytest

import paper_2511_22793_amd as gs
import synth
from test_gpu_train_fused import _check_against_unfused, _run_both, _targets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,tile,faint", [(45, 75, (16, 16), 0), (33, 71, (8, 16), 100), (24, 41, (8, 8), 200),
                                            (90, 90, (16, 16), 110), (90, 90, (16, 16), 220), (90, 90, (16, 16), 420)])
def test_pairs_match_unfused_path(H, W, tile, faint):
    S, F, n = 3, 8, 160
    sc = synth.scene(n, seed=H + faint)
    if faint:
        # small and faint, close together: many entries over few pixels
        a = synth.scene(faint, seed=W, lo=[1.5, 1.4, 1.2], hi=[1.7, 1.6, 1.3], log_scale_mean=-2.5)
        a["opacity_logit"] = np.full(faint, -4.0, np.float32)
        sc = {k: np.ascontiguousarray(np.concatenate([a[k], sc[k]], axis=-1)) for k in sc}
    attrs = np.stack([synth.channel_attrs(n + faint, F, True, seed=7 + s) for s in range(S)])
    fused, ref, ws = _run_both(sc, attrs, [0.0, 0.0, 0.0], _targets(S, F, H, W, 5), gs.Grid(H, W, *tile), gs.Params())
    if faint > 200 and H == 90:
        stops = ws.view("n_last", 0, H * W).cpu().numpy()
        assert stops.max() > (256 if faint > 400 else 128) and np.median(stops) <= 128
    _check_against_unfused(fused, ref, S)
