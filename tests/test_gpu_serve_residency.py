"""The persistent compositing launch keeps the chip's waves in flight whatever
its workgroup size: its LDS is that of the waves launched and of the forms its
jobs take.  (The matrix-core form's registers allow two waves per SIMD, 8 per
CU; the row form runs four.)  And the spectra are those of the grid-mapped
launches at every size."""
import pytest
import torch

import paper_2511_22793_amd as gs
import synth
from gpu_util import to_dev
from paper_2511_22793_amd import serve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(8, 8), (8, 16), (16, 16)])
@pytest.mark.parametrize("channels,waves", [(((1, False),), 16), (((7, False), (2, True)), 16),
                                            (((16, True),), 8), (((1, False), (5, True), (16, True)), 8)])
def test_waves_per_cu(tile, channels, waves):
    jobs = []
    rx = torch.tensor([[0.1, -0.2, 0.3], [2.5, -1.0, 1.4]]).cuda()
    for i, (F, cplx) in enumerate(channels):
        sc = to_dev(synth.scene(600, seed=i, lo=[-3, -3, 0.1], hi=[3, 3, 2.5], log_scale_mean=-1.3))
        jobs.append(serve.Job(sc, torch.from_numpy(synth.channel_attrs(600, F, cplx, seed=i)).cuda(), rx, cplx,
                              gs.Grid(45, 180, *tile)))
    b = serve.Batch(jobs)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert b.info.block == tile[0] * tile[1]
    assert b.info.workgroups * (b.info.block // 64) >= waves * cus
    b.run()
    for j, s in zip(b.jobs, b.spectra):
        ref, _ = gs.forward(j.scene, j.attr, j.rx, grid=j.grid, params=j.params, is_complex=j.is_complex)
        assert torch.equal(s, ref)
