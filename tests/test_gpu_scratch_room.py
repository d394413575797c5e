"""The work buffer that a large call leaves for the next ones, where the budget
is tight: a small call that runs at the same time holds no more of it than it
needs, so that an encoding or a job that fits beside the small call is not
refused."""
import threading
import time

import numpy as np
import pytest

import scenes
from scenes import jobs

pytestmark = pytest.mark.gpu
D, LAM = 8e-6, 520e-9
ROOM = 41 << 20


def _context():
    """A context with ROOM bytes beside its batch buffers (at their smallest,
    2^16 paths, under any budget this small)."""
    import paper_2606_14173_amd as hpt
    with hpt.Context(0, 64 << 20) as c:
        used = c.ctx_stats()["used_bytes"]
    return hpt.Context(0, used + ROOM)


def _fields(n, h, w, seed):
    import torch
    rng = np.random.default_rng(seed)
    u = (rng.normal(size=(n, h, w)) + 1j * rng.normal(size=(n, h, w))).astype(np.complex64)
    return torch.from_numpy(u).to("cuda:0")


def _leave_large_buffer(c):
    import torch
    base = c.ctx_stats()["used_bytes"]
    src, out = _fields(8, 200, 300, 1), torch.empty((1, 5, 200, 300), dtype=torch.float32, device="cuda:0")
    c.reconstruct(src, 1, 8, 300, 200, D, [LAM], [1e-3 * k for k in range(1, 6)], 0.02, out)
    return base, c.ctx_stats()["used_bytes"] - base


class _SmallCall(threading.Thread):
    """Two 64 x 64 fields, propagated on a stream that is busy for about half a second."""

    def __init__(self, c):
        import torch
        super().__init__()
        self.c, self.src = c, _fields(2, 64, 64, 2)
        self.dst, self.a = torch.empty_like(self.src), torch.randn(4096, 4096, device="cuda:0")
        self.error = None
        (self.a @ self.a).sum()
        torch.cuda.synchronize()
        self.start()
        time.sleep(0.15)   # it has its work buffer now

    def run(self):
        import torch
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(400):
                    self.a = self.a @ self.a * 1e-3
                self.c.asm_propagate(self.src, self.dst, 2, 64, 64, D, LAM, 1e-3)
        except Exception as e:
            self.error = e

    def end(self):
        import torch
        self.join()
        assert self.error is None
        ref = torch.empty_like(self.src)
        self.c.asm_propagate(self.src, ref, 2, 64, 64, D, LAM, 1e-3)
        assert torch.equal(self.dst, ref)


def _encode(c, src):
    import torch
    n, h, w = src.shape
    ph = torch.empty((n, h, w), dtype=torch.float32, device="cuda:0")
    c.encode_phase(src, ph, n, w, h, D, LAM, -4e-3, 2, 0.05)
    return ph


def test_encoding_beside_a_small_call():
    """800 x 600: 24 bytes a pixel, a row buffer of 600 x 2048 and a quarter of
    2048 x 2048 factors, 30 MB in all."""
    import torch
    import paper_2606_14173_amd as hpt
    src = _fields(1, 600, 800, 3)
    with hpt.Context(0) as big:
        ref = _encode(big, src)
    with _context() as c:
        _, left = _leave_large_buffer(c)
        assert left > ROOM - (30 << 20)          # beside it the encoding would not fit
        small = _SmallCall(c)
        got = _encode(c, src)
        small.end()
        assert torch.equal(got, ref)


def test_job_beside_a_small_call():
    """A random-field table of 600 x 600 x 4 and its scratch: 35 MB."""
    gw = gh = 600
    j = dict(jobs.JOB_DEFAULTS)
    j.update(width=64, height=64, lambdas=[LAM], comps=[1], spp=4, max_bounces=2, T=4, seed=1, grf_seed=7, grf_w=gw,
             grf_h=gh, phase_mode=jobs.PHASE_SPLIT)
    with _context() as c:
        sid = c.upload_scene(scenes.scene_tiny(0))
        _, left = _leave_large_buffer(c)
        assert left > ROOM - 96 * gw * gh        # beside it the table would not fit
        small = _SmallCall(c)
        U = c.trace(sid, j)
        small.end()
        assert np.isfinite(U).all() and np.abs(U).max() > 0


def test_job_that_takes_the_rest_of_an_ample_budget():
    """Less than half of the budget is in use, but the job's table and scratch
    (24 bytes a point and frame) leave 30 MB of it."""
    import paper_2606_14173_amd as hpt
    with hpt.Context(0, 64 << 20) as c:
        used = c.ctx_stats()["used_bytes"]
    room = used + (192 << 20)
    side = int(np.sqrt((room - (30 << 20)) / (24 * 8)))
    assert side <= 4096
    j = dict(jobs.JOB_DEFAULTS)
    j.update(width=64, height=64, lambdas=[LAM], comps=[1], spp=4, max_bounces=2, T=8, seed=1, grf_seed=7, grf_w=side,
             grf_h=side, phase_mode=jobs.PHASE_SPLIT)
    with hpt.Context(0, used + room) as c:
        sid = c.upload_scene(scenes.scene_tiny(0))
        before, left = _leave_large_buffer(c)
        assert left > 30 << 20 and 2 * (before + left) <= used + room
        small = _SmallCall(c)
        U = c.trace(sid, j)
        small.end()
        assert np.isfinite(U).all() and np.abs(U).max() > 0


def test_buffer_is_given_up():
    """Nothing of it is lost to the budget's count when its room is needed."""
    with _context() as c:
        base, left = _leave_large_buffer(c)
        assert left > 0
        _encode(c, _fields(1, 600, 800, 3))
        _encode(c, _fields(1, 16, 16, 3))
        assert c.ctx_stats()["used_bytes"] - base <= ROOM
        sid = c.upload_scene(scenes.scene_mid(1))
        c.build_cache(sid, res=32, bins=8, spb=1, max_bounces=2, seed=7)   # 12.6 MB and the scene's
        info = c.scene_info(sid)
        assert c.ctx_stats()["used_bytes"] <= base + ROOM and info["device_bytes"] > 0
