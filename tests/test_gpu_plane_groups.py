"""Focal stacks whose planes and frames are taken a few at a time, because the
budget has no room for more (a plane's transfer function is then tabulated again
for every group of frames), against an ample budget and the FP64 oracle.

Bars: the fields are the same bits, so only the order in which T positive
intensities are added differs: each of the at most T additions and T products
with the weight rounds by 2^-24 of the sum on either side, 4 T 2^-24 in all.
Against the oracle the bar of the other focal stacks, 2e-5 of the mean times the
root of the largest to the mean intensity."""
import numpy as np
import pytest

from oracle import asm as oasm
from oracle import recon as orecon

pytestmark = pytest.mark.gpu
D, LAM = 8e-6, [638e-9, 450e-9]
DIST = [2e-3, -1e-3, 5e-3, 9e-3]
T = 5


def _tight(need):
    import paper_2606_14173_amd as hpt
    with hpt.Context(0, 64 << 20) as c:
        used = c.ctx_stats()["used_bytes"]
    return hpt.Context(0, used + need)


@pytest.mark.parametrize("h,w", [(200, 150), (129, 257), (601, 260)])
def test_planes_and_frames_a_few_at_a_time(h, w):
    import torch
    import paper_2606_14173_amd as hpt
    px, py = oasm.padded_size(w), oasm.padded_size(h)
    one, tab = 8 * h * px, 8 * (px // 2 + 1) * (py // 2 + 1)
    rng = np.random.default_rng(h)
    u = (rng.normal(size=(2, T, h, w)) + 1j * rng.normal(size=(2, T, h, w))).astype(np.complex64)
    src = torch.from_numpy(u).to("cuda:0")

    def stack(c):
        out = torch.empty((2, len(DIST), h, w), dtype=torch.float32, device="cuda:0")
        c.reconstruct(src, 2, T, w, h, D, LAM, DIST, 0.02, out)
        return out.cpu().numpy().astype(np.float64)

    with hpt.Context(0) as big:
        ref = stack(big)
    exact = orecon.focal_stack(u.astype(np.complex128), D, LAM, DIST, na=0.02)
    bar = 2e-5 * np.sqrt(exact.max() / exact.mean())
    assert np.abs(ref - exact).max() / exact.mean() <= bar
    # planes and frames at a time: 1 and 1, 3 and 1, 4 and 1, 4 and 2
    for planes, frames in ((1, 1), (3, 1), (4, 1), (4, 2)):
        need = (planes + 1) * frames * one + planes * tab + 3 * 256
        with _tight(need) as c:
            got = stack(c)
        rel = (np.abs(got - ref) / ref).max()
        err = np.abs(got - exact).max() / exact.mean()
        print("%dx%d, %d planes, %d frames: %.2e from the ample budget's, %.2e from the oracle's" % (h, w, planes, frames,
                                                                                                 rel, err), flush=True)
        assert rel <= 4 * T * 2.0 ** -24 and err <= bar
    with _tight(2 * one + tab) as c, pytest.raises(hpt.HptError, match="EBUDGET"):
        stack(c)
