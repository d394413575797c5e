"""Occlusion queries of next-event estimation that travel with the path's next
ray: dense and compacted queues (up to 2^18 paths a batch and more), paths
absorbed while their query is open (GGX lobes below the surface), and batches of
several scenes. Bars as for next-event estimation elsewhere; jobs in a mixed
batch equal themselves alone bit for bit."""
import numpy as np
import pytest

import scenes
from scenes import jobs
from parity_util import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2606_14173_amd as hpt
    c = hpt.Context(0)
    yield c
    c.close()


def _rays(ctx, sid, job):
    jid = ctx.submit(sid, job)
    ctx.wait(jid)
    rays = ctx.stats(jid)["rays"]
    ctx.release_job(jid)
    return rays


@pytest.mark.parametrize("crop,spp", [((250, 250, 9, 7), 5), ((236, 236, 72, 64), 24)])
def test_queries_match_oracle(ctx, crop, spp):
    sc = scenes.scene_mid(1)
    job = jobs.job_for_config(1, T=2, nee=1, crop=crop, spp=spp)
    sid = ctx.upload_scene(sc)
    Ug, recg, ctg = gpu_run(ctx, sid, job)
    rays = [_rays(ctx, sid, dict(job, nee=n)) for n in (0, 1)]
    ctx.release_scene(sid)
    assert rays[0] == rays[1]   # the same paths; occlusion queries are no rays
    Uo, reco, cto = oracle_run(sc, job)
    r = compare(Ug, recg, ctg, Uo, reco, cto)
    same = recg["sig"] == reco["sig"]
    print("paths %d match %.5f err/rms %.2e absorbed %d" % (r["n_paths"], r["match"], r["err"],
                                                            (reco["kind"] == 7).sum()))
    assert r["ok"]
    assert np.array_equal(recg["kind"][same], reco["kind"][same])
    assert np.array_equal(recg["n_hits"][same], reco["n_hits"][same])


@pytest.mark.parametrize("w,h,spp", [(24, 20, 8), (128, 96, 24)])
def test_scenes_in_one_batch_match_alone(ctx, w, h, spp):
    sids = [ctx.upload_scene(s) for s in (scenes.scene_tiny(0), scenes.scene_mid(1), scenes.scene_tiny(0))]
    reqs = [(sid, jobs.job_for_config(0, T=2, nee=n, seed=11 + k, max_bounces=4, width=w, height=h, spp=spp))
            for k, (sid, n) in enumerate([(sids[0], 1), (sids[1], 1), (sids[2], 1), (sids[0], 1)])]
    alone = [ctx.trace(sid, j) for sid, j in reqs]
    jids = [ctx.submit(sid, j) for sid, j in reqs]
    for jid, (sid, j), a in zip(jids, reqs, alone):
        ctx.wait(jid)
        got = ctx.read_field(jid, j)
        ctx.release_job(jid)
        assert np.array_equal(got.view(np.uint32), a.view(np.uint32))
    for sid in sids:
        ctx.release_scene(sid)
