"""Line FFTs of the propagation at the edges of every padded length, against
the FP64 oracle: the shortest and the longest field that each padded length
2 .. 8192 takes, along each axis; plane groups and transfer functions under a
budget that has room for one at a time; work buffers kept between calls.

Bar: a path through the transforms has at most 2 log2 Px + 2 log2 Py <= 52
butterfly levels, each rounding by at most 2^-24 of the RMS with random signs:
52^0.5 x 6e-8 = 4e-7 x RMS, and the largest of up to 10^6 values lies within
6 of that: 3e-6 x RMS; 1e-5 leaves room for the twiddles' own rounding."""
import threading

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


def _fields(n, h, w, seed):
    rng = np.random.default_rng(seed)
    return (rng.normal(size=(n, h, w)) + 1j * rng.normal(size=(n, h, w))).astype(np.complex64)


def _asm(ctx, u, z, band=True):
    import torch
    n, h, w = u.shape
    src = torch.from_numpy(u).to("cuda:0")
    dst = torch.empty_like(src)
    ctx.asm_propagate(src, dst, n, w, h, D, LAM, z, band)
    return dst.cpu().numpy()


def _close(got, ref, label):
    err = np.abs(got - ref).max() / np.sqrt(np.mean(np.abs(ref) ** 2))
    print("%s: %.2e" % (label, err), flush=True)
    assert err <= TOL, label


@pytest.mark.parametrize("lg", range(1, 14))
def test_every_padded_length(ctx, lg):
    """Rows and columns of the shortest (N/4 + 1) and the longest (N/2) field
    padded to N = 2^lg; three fields, so that a column group takes several."""
    n = 1 << lg
    for m in sorted({max(1, n // 4 + 1), n // 2}):
        assert oasm.padded_size(m) == n
        for h, w in ((m, 5), (7, m)):
            u = _fields(3, h, w, seed=lg * 100 + h)
            _close(_asm(ctx, u, 1e-3), oasm.propagate(u, D, LAM, 1e-3), "%dx%d" % (h, w))


@pytest.mark.parametrize("h,w", [(64, 300), (300, 64), (520, 130)])
def test_many_planes_at_once(ctx, h, w):
    import torch
    u = _fields(6, h, w, seed=h).reshape(2, 3, h, w)
    lam, dist = [638e-9, 450e-9], [1e-3 * k for k in range(-3, 6)]
    out = torch.empty((2, len(dist), h, w), dtype=torch.float32, device="cuda:0")
    ctx.reconstruct(torch.from_numpy(u).to("cuda:0"), 2, 3, w, h, D, lam, dist, 0.02, out)
    ref = orecon.focal_stack(u.astype(np.complex128), D, lam, dist, na=0.02)
    # an intensity |u|^2 doubles the field's relative error
    err = np.abs(out.cpu().numpy() - ref).max() / ref.mean()
    assert err <= 2 * TOL * np.sqrt(ref.max() / ref.mean())


def _tight(need):
    """A context whose budget leaves `need` bytes beside its batch buffers (at
    their smallest, 2^16 paths, under any budget this small)."""
    import paper_2606_14173_amd as hpt
    with hpt.Context(0, 64 << 20) as c:
        used = c.ctx_stats()["used_bytes"]
    c = hpt.Context(0, used + need)
    assert c.ctx_stats()["used_bytes"] == used
    return c


@pytest.mark.parametrize("h,w", [(200, 150), (129, 257)])
def test_room_for_one_of_each(h, w):
    """Where the budget has room for one field, one plane and one transfer
    function, results are those of an ample budget, bit for bit; with room for
    none the calls are refused."""
    import torch
    import paper_2606_14173_amd as hpt
    px, py = oasm.padded_size(w), oasm.padded_size(h)
    one, tab = 8 * h * px, 8 * (px // 2 + 1) * (py // 2 + 1)
    need = 24 * h * w + one + 24 * h + 24 + tab + 16 * 256 + tab // 2   # encoding: the largest of the three
    u = _fields(2, h, w, seed=w)
    src = torch.from_numpy(u).to("cuda:0")
    dist = [2e-3, -1e-3, 5e-3]

    def all_three(c):
        a, ph = torch.empty_like(src), torch.empty((2, h, w), dtype=torch.float32, device="cuda:0")
        st = torch.empty((1, 3, h, w), dtype=torch.float32, device="cuda:0")
        c.asm_propagate(src, a, 2, w, h, D, LAM, 3e-3)
        c.reconstruct(src, 1, 2, w, h, D, [LAM], dist, 0.02, st)
        loss = c.encode_phase(src, ph, 2, w, h, D, LAM, -4e-3, 4, 0.05)
        return a.cpu(), ph.cpu(), loss

    with hpt.Context(0) as big:
        ref = all_three(big)
    with _tight(need) as c:
        got = all_three(c)
        assert all(torch.equal(x, y) for x, y in zip(ref[:2], got[:2]))
        assert np.allclose(ref[2], got[2], rtol=1e-12)
    with _tight(one // 2) as c, pytest.raises(hpt.HptError, match="EBUDGET"):
        c.asm_propagate(src, torch.empty_like(src), 2, w, h, D, LAM, 3e-3)
    phi_o, _ = oenc.encode(u.astype(np.complex128), D, LAM, -4e-3, 4, 0.05)
    d = np.abs(np.angle(np.exp(1j * (ref[1].numpy().astype(np.float64) - phi_o))))
    assert np.percentile(d, 99.9) <= 1e-3


def test_calls_of_several_threads_and_sizes(ctx):
    """Work buffers are kept between calls: calls of changing sizes, one after
    another and from four threads at once, give what each gives alone."""
    jobs = [(64, 64, 1e-3), (300, 200, -2e-3), (31, 500, 5e-3), (200, 300, 4e-3)]
    data = [_fields(3, h, w, seed=k) for k, (h, w, _) in enumerate(jobs)]
    alone = [_asm(ctx, u, z) for u, (_, _, z) in zip(data, jobs)]
    again = [_asm(ctx, u, z) for u, (_, _, z) in zip(data, jobs)]
    wrong = []

    def work(k):
        for _ in range(20):
            if not np.array_equal(_asm(ctx, data[k], jobs[k][2]), alone[k]):
                wrong.append(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert all(np.array_equal(a, b) for a, b in zip(alone, again)) and not wrong
