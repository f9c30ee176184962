"""Adam on elements that are not finite: the limits of its definition.  An
infinite or NaN gradient gives NaN, a second moment that overflowed makes no
update, a large finite gradient an ordinary one."""
import numpy as np
import pytest
import torch

from paper_2511_22793_amd import mlp as gm

pytestmark = pytest.mark.gpu

INF = float("inf")
# p, g, m, v
ROWS = np.array([[0.5, INF, 0.0, 0.0], [0.5, -INF, 0.1, 0.2], [0.5, float("nan"), 0.0, 0.0], [0.5, 1e-3, 0.1, INF],
                 [0.5, 0.0, 0.0, INF], [0.5, 1e3, 0.1, INF], [0.5, 1e15, 0.0, 0.0], [0.5, 0.25, 0.1, 0.01],
                 [0.5, 1e-20, 0.0, 0.0]], np.float32)


@pytest.mark.parametrize("step", [1, 40])
@pytest.mark.parametrize("pad", [0, 1])  # the vector and the element loads
def test_adam_limits(step, pad):
    p, g, m, v = (torch.from_numpy(np.concatenate([np.zeros(pad, np.float32), c])).cuda()[pad:] for c in ROWS.T.copy())
    lr, b1, b2, eps = 0.01, float(np.float32(0.9)), float(np.float32(0.999)), float(np.float32(1e-15))
    gm.adam_step([(p, g, m, v, None, lr)], step)
    q, h, m0, v0 = ROWS.T.astype(np.float64)
    with np.errstate(all="ignore"):
        m1, v1 = b1 * m0 + (1 - b1) * h, b2 * v0 + (1 - b2) * h * h
        ref = q - float(np.float32(lr)) * (m1 / (1 - b1 ** step)) / (np.sqrt(v1 / (1 - b2 ** step)) + eps)
    got = p.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    ok = ~np.isnan(ref)
    # one rounding of p, the estimates' 48 bits far below it
    assert np.all(np.abs(got[ok] - ref[ok]) <= np.spacing(np.abs(ref[ok]).astype(np.float32)))
    assert np.all(got[3:6] == 0.5)
