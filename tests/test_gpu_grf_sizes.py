"""Random-field tables of Eq. 4 for grids of every kind of size (powers of two,
their multiples, odd composites, primes, one texel, the largest line) against
the oracle's FP64 inverse FFT.

Bar: a table value is an FP64 sum (error of order 1e-15) rounded once to
float32, so it is within half a unit in the last place: 2^-24 of the largest
component, which lies below 8 for these sizes: 4.8e-7."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2606_14173_amd as hpt
    c = hpt.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("gw,gh,T", [(1, 1, 2), (2, 3, 1), (8, 16, 3), (64, 64, 1), (97, 31, 2), (127, 128, 5),
                                     (243, 125, 2), (360, 224, 4), (4096, 3, 1), (5, 4096, 2), (4093, 2, 1),
                                     (2, 3571, 1), (832, 832, 1), (2187, 7, 3)])
def test_grf_sizes(ctx, gw, gh, T):
    got = ctx.grf(gw, gh, T, 5).astype(np.complex128)
    ref = oracle.grf_table(gw, gh, T, 5)
    err = max(np.abs(got.real - ref.real).max(), np.abs(got.imag - ref.imag).max())
    print("%dx%d T=%d: %.2e, largest %.2f" % (gw, gh, T, err, np.abs(ref).max()), flush=True)
    assert np.abs(ref).max() < 8 and err <= 4.8e-7
