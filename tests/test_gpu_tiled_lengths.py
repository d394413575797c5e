"""Tiled row spectra at the lengths and in the kernels that the propagation of
short rows does not reach: rows padded to 8192 (one row to a workgroup) and, in
the encoding's own row kernels, every tiled length with an odd number of rows
(the last pair of rows is half empty), where Adam's kernel also rewrites the
spectra in place. Against the FP64 oracle.

Bars: propagation and focal stacks as at the other tiled sizes, 1e-5 x RMS (at
most 52 butterfly levels of 2^-24 with random signs, the largest of 10^7 values
within 6 of that, and the twiddles' rounding) and twice that for an intensity.
Encoding as at the untiled sizes: phases within 1e-3 rad on 99.9 % of the pixels
(a pixel whose gradient is within rounding of zero may step the other way), losses
within 1e-4 + 1e-3 x the oracle's."""
import numpy as np
import pytest

from oracle import asm as oasm
from oracle import encode as oenc
from oracle import recon as orecon

pytestmark = pytest.mark.gpu
D, LAM, TOL = 8e-6, 520e-9, 1e-5


@pytest.fixture(scope="module")
def ctx():
    import paper_2606_14173_amd as hpt
    c = hpt.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("h,w,n", [(513, 2049, 2), (601, 4096, 2), (1025, 2050, 1)])
def test_rows_of_8192(ctx, h, w, n):
    import torch
    assert oasm.padded_size(w) == 8192
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


@pytest.mark.parametrize("h,w", [(701, 257), (515, 600), (513, 1025), (1027, 513), (513, 2049), (2049, 140), (2049, 257)])
def test_encoding_in_tiles(ctx, h, w):
    import torch
    rng = np.random.default_rng(h * 7 + w)
    y, x = np.mgrid[0:h, 0:w]
    u = 0.3 * (rng.normal(size=(2, h, w)) + 1j * rng.normal(size=(2, h, w)))
    for f in range(2):
        for _ in range(3):
            cy, cx, s = rng.uniform(0, h), rng.uniform(0, w), rng.uniform(1.5, 6.0)
            u[f] += np.exp(-((y - cy) ** 2 + (x - cx) ** 2) / (2 * s * s) + 2j * np.pi * rng.uniform())
    u = u.astype(np.complex64)
    src = torch.from_numpy(u).to("cuda:0")
    ph = torch.empty((2, h, w), dtype=torch.float32, device="cuda:0")
    loss = ctx.encode_phase(src, ph, 2, w, h, D, LAM, -6e-3, 3, 0.05)
    phi_o, loss_o = oenc.encode(u.astype(np.complex128), D, LAM, -6e-3, 3, 0.05)
    d = np.abs(np.angle(np.exp(1j * (ph.cpu().numpy().astype(np.float64) - phi_o))))
    print("%dx%d: p99.9 %.2e, loss %s vs %s" % (h, w, np.percentile(d, 99.9), loss, loss_o), flush=True)
    assert np.percentile(d, 99.9) <= 1e-3
    assert np.all(np.abs(loss - loss_o) <= 1e-4 + 1e-3 * loss_o)
