"""Pixel order, sample split and random-field wrap at odd sizes: crops one pixel
wide or high, with partial tiles and a short last band, sample counts that are no
power of two, and field grids from one texel to just the hologram, in which nearly
every image point falls outside and wraps. Bars as for the rest of the tracer
(identical path signatures, field error against the oracle)."""
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


@pytest.mark.parametrize("w,h,spp,gw,gh", [(1, 1, 5, 1, 1), (7, 9, 3, 7, 9), (8, 8, 1, 8, 11), (33, 17, 6, 64, 17),
                                           (1, 41, 7, 3, 4096), (65, 1, 2, 127, 2)])
def test_odd_sizes_match_oracle(ctx, w, h, spp, gw, gh):
    sc = scenes.scene_tiny(0)
    job = jobs.job_for_config(0, T=2, width=w, height=h, spp=spp, grf_w=gw, grf_h=gh, max_bounces=3,
                              phase_mode=jobs.PHASE_SPLIT)
    sid = ctx.upload_scene(sc)
    r = compare(*gpu_run(ctx, sid, job), *oracle_run(sc, job))
    ctx.release_scene(sid)
    print("paths %d match %.5f err/rms %.2e" % (r["n_paths"], r["match"], r["err"]))
    assert r["ok"]
