"""The attribute network's row tiles: row counts at the edges of the 16-, 64-
and 128-row tiles, both output widths, and attributes that are only 8-byte
aligned (narrow stores and loads).  Rows are independent, so the outputs of the
first r rows are those of the whole list bit for bit and no other row is
written; the weight gradients of the first r rows and of the rest add up to
the whole's: FP32 sums in another order, 2e-4 of each tensor's maximum (as the
other gradient tests); a row's own embedding gradient differs by the order of
its few terms, 1e-5.
"""
import pytest
import torch

from paper_2511_22793_amd import mlp as gm
from test_gpu_mlp import setup

pytestmark = pytest.mark.gpu


def _run(d, lst, r, up, off):
    n, S, F = d["n"], d["S"], d["F"]
    rows = gm.Rows(d["rows"].tx, lst, torch.tensor([r], dtype=torch.int32, device="cuda"), row_cap=n // 2)
    st = gm.State(S, n // 2, n_partial=8, n_chan=F)

    def shifted(t):
        buf = torch.zeros(t.numel() + off, device="cuda")
        buf[off:] = t.flatten()
        return buf[off:].view(t.shape)

    attr = shifted(torch.zeros(S, n, F, 2, device="cuda"))
    gm.forward(d["net"], gm.embed(d["net"], d["E_bf"]), d["mean"], rows, attr, st)
    g = gm.backward(d["net"], d["E_bf"], d["mean"], rows, shifted(up), st)
    torch.cuda.synchronize()
    return attr, g


@pytest.mark.parametrize("F,off", [(64, 0), (32, 0), (64, 2)])
@pytest.mark.parametrize("r", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129])
def test_row_tiles(r, F, off):
    d = setup(n=300, S=2, seed=11, F=F)
    N = d["n"] // 2
    lst = d["rows"].list
    up = torch.randn(2, d["n"], F, 2, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    full, gf = _run(d, lst, N, up, 0)
    head, gh = _run(d, lst, r, up, off)
    tail, gt = _run(d, lst[r:].contiguous(), N - r, up, off)
    at = lst.long()
    for out, rows in ((head, at[:r]), (tail, at[r:])):
        assert torch.equal(out[:, rows], full[:, rows])
        rest = torch.ones(d["n"], dtype=torch.bool, device="cuda")
        rest[rows] = False
        assert not out[:, rest].any()
    for k in ("W1", "b1", "W2", "b2", "W3", "b3"):
        assert float((gh[k] + gt[k] - gf[k]).abs().max()) <= 2e-4 * float(gf[k].abs().max()), k
    scale = float(gf["E"][at].abs().max())
    assert float((gh["E"][at[:r]] - gf["E"][at[:r]]).abs().max()) <= 1e-5 * scale
    assert float((gt["E"][at[r:]] - gf["E"][at[r:]]).abs().max()) <= 1e-5 * scale
