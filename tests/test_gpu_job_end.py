"""A job that ends without having run (cancelled before any batch took it, or
failed with its first batch) leaves nothing behind that still writes the
caller's field: its set-up waits for the caller's stream and then clears the
field, so the job ends after both, and what the caller puts into the field once
hpt_job_wait has returned stays there."""
import pytest

import scenes
from scenes import jobs

pytestmark = pytest.mark.gpu


def _job(w, h, spp, bounces):
    gw, gh = jobs.grf_size(w, h, 8e-6, 520e-9, 52e-3)
    j = dict(jobs.JOB_DEFAULTS)
    j.update(width=w, height=h, lambdas=[520e-9], comps=[1], spp=spp, max_bounces=bounces, T=1, seed=1, grf_seed=7,
             grf_w=gw, grf_h=gh, phase_mode=jobs.PHASE_SPLIT)
    return j


def _submit_behind_busy_stream(ctx, sid, job):
    """(job, its field, an event that a stream reaches after about half a
    second; the job was submitted on that stream)."""
    import torch
    field = torch.ones((1, job["T"], job["height"], job["width"]), dtype=torch.complex64, device="cuda:0")
    a = torch.randn(4096, 4096, device="cuda:0")
    (a @ a).sum()
    torch.cuda.synchronize()
    s, busy = torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(s):
        for _ in range(400):
            a = a @ a * 1e-3
        busy.record()
        jid = ctx.submit(sid, job, field=field)
    return jid, field, busy


def _ended(ctx, jid, field, busy, name):
    """Wait for the job, which ends with `name`, and give its field to other work."""
    import torch
    import paper_2606_14173_amd as hpt
    with pytest.raises(hpt.HptError) as e:
        ctx.wait(jid)
    through = busy.query()
    assert e.value.name == name
    ctx.release_job(jid)
    field.fill_(2.0)
    torch.cuda.synchronize()
    assert through
    return field


def test_cancelled_before_any_batch_took_it():
    """Batches of 2^16 paths, which each unit of the first job fills: the
    second job is admitted but in no batch until the first is through."""
    import torch
    import paper_2606_14173_amd as hpt
    with hpt.Context(0, 256 << 20) as ctx:
        assert ctx.ctx_stats()["batch_capacity_paths"] == 1 << 16
        sid = ctx.upload_scene(scenes.scene_mid(1))
        long, small = _job(512, 512, 256, 6), _job(64, 64, 16, 2)
        ctx.trace(sid, small)                       # its random field is resident
        first = ctx.submit(sid, long)
        while ctx.ctx_stats()["jobs_running"] < 1:
            pass
        jid, field, busy = _submit_behind_busy_stream(ctx, sid, small)
        while ctx.ctx_stats()["jobs_running"] == 1 and ctx.ctx_stats()["jobs_queued"]:
            pass
        ctx.cancel(jid)
        _ended(ctx, jid, field, busy, "HPT_ECANCELED")
        ctx.cancel(first)
        with pytest.raises(hpt.HptError):
            ctx.wait(first)
        ctx.release_job(first)
        ctx.trace(sid, small)
        torch.cuda.synchronize()
        assert bool((field == 2.0).all())


def test_failed_with_its_first_batch():
    import torch
    import paper_2606_14173_amd as hpt
    with hpt.Context(0) as ctx:
        sid = ctx.upload_scene(scenes.scene_tiny(0))
        small = _job(64, 64, 16, 2)
        ctx.trace(sid, small)
        ctx.debug_fail_batches(1)
        jid, field, busy = _submit_behind_busy_stream(ctx, sid, small)
        _ended(ctx, jid, field, busy, "HPT_EDEVICE")
        ctx.trace(sid, small)
        torch.cuda.synchronize()
        assert bool((field == 2.0).all())
