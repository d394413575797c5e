"""Fields whose row spectra lie in tiles (columns padded to 2048 and more, rows to
512 and more), at the shortest and longest sizes of each padded length, odd heights
(workgroups of two rows cross from one field to the next) and just outside the
rule: propagation and a focal stack of two planes against the FP64 oracle.

Bar: that of the untiled transforms (at most 52 butterfly levels of 2^-24 with
random signs, the largest of 10^7 values within 6 of that, and the twiddles'
rounding): 1e-5 x RMS; an intensity has twice a field's relative error."""
import numpy as np
import pytest

from oracle import asm as oasm
from oracle import recon as orecon

pytestmark = pytest.mark.gpu
D, LAM, TOL = 8e-6, 520e-9, 1e-5


@pytest.fixture(scope="module")
def ctx():
    import paper_2606_14173_amd as hpt
    c = hpt.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("h,w", [(513, 129), (1024, 128), (701, 257), (515, 600), (513, 1025), (1025, 130), (1027, 513),
                                 (2048, 200), (2049, 140)])
def test_tiled_fields(ctx, h, w):
    import torch
    n = 3 if h * w < 400000 else 2
    rng = np.random.default_rng(h + w)
    u = (rng.normal(size=(n, h, w)) + 1j * rng.normal(size=(n, h, w))).astype(np.complex64)
    src = torch.from_numpy(u).to("cuda:0")
    dst = torch.empty_like(src)
    ctx.asm_propagate(src, dst, n, w, h, D, LAM, 1e-3, True)
    ref = oasm.propagate(u, D, LAM, 1e-3)
    err = np.abs(dst.cpu().numpy() - ref).max() / np.sqrt(np.mean(np.abs(ref) ** 2))
    dist = [1e-3, -2e-3]
    out = torch.empty((1, 2, h, w), dtype=torch.float32, device="cuda:0")
    ctx.reconstruct(src, 1, n, w, h, D, [LAM], dist, 0.02, out)
    ref = orecon.focal_stack(u.astype(np.complex128)[None], D, [LAM], dist, na=0.02)
    err_i = np.abs(out.cpu().numpy() - ref).max() / ref.mean()
    print("%dx%d: %.2e, stack %.2e" % (h, w, err, err_i), flush=True)
    assert err <= TOL
    assert err_i <= 2 * TOL * np.sqrt(ref.max() / ref.mean())
