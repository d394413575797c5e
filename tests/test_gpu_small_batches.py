"""Batches on both sides of the lines at which ray generation and the queues
change (2^18 paths: small sorting windows, dense queues filled by atomics):
one job in one batch, in a mix whose batches are larger, and in a context
whose batches are smaller gives the same field and signatures, bit for bit,
with and without next-event estimation, in every phase mode."""
import numpy as np
import pytest

import scenes
from scenes import jobs

pytestmark = pytest.mark.gpu


def _job(w, h, spp, T, mode, nee=0, n_ch=1):
    gw, gh = jobs.grf_size(w, h, 8e-6, 638e-9, 32e-3)
    j = dict(jobs.JOB_DEFAULTS)
    j.update(width=w, height=h, lambdas=jobs.RGB[:n_ch], comps=list(range(n_ch)), spp=spp, max_bounces=4, T=T, seed=3,
             grf_seed=4, grf_w=gw, grf_h=gh, phase_mode=mode, nee=nee)
    return j


@pytest.mark.parametrize("w,h,spp", [(16, 8, 1), (64, 64, 64), (513, 8, 64), (33, 31, 257), (100, 100, 27)])
@pytest.mark.parametrize("mode,nee", [(jobs.PHASE_FP64, 0), (jobs.PHASE_SPLIT, 1), (jobs.PHASE_FP32, 0)])
def test_same_in_any_batch(w, h, spp, mode, nee):
    import paper_2606_14173_amd as hpt
    sc = scenes.scene_mid(2)
    j = dict(_job(w, h, spp, 3, mode, nee), debug=4)
    other = _job(256, 200, 32, 1, mode, nee)
    got = []
    for budget in (0, 256 << 20):                      # batches of 2^26 and of 2^16 paths
        with hpt.Context(0, budget) as ctx:
            sid = ctx.upload_scene(sc)
            got.append(ctx.trace(sid, j, sigsum=True))
            ids = [ctx.submit(sid, other), ctx.submit(sid, j), ctx.submit(sid, other)]
            for i in ids:
                ctx.wait(i)
            got.append((ctx.read_field(ids[1], j), ctx.read_sigsum(ids[1], j)))
    assert np.abs(got[0][0]).max() > 0
    for f, s in got[1:]:
        assert np.array_equal(f.view(np.uint32), got[0][0].view(np.uint32)) and np.array_equal(s, got[0][1])
