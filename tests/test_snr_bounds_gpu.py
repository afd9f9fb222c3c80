"""The fused boxcar / S/N kernel's sums of squares at the limits of what they
hold, against the oracle: S/N within 1e-5 relative (float32 results), peak
indices exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _check(dd, widths, threads, pad=0):
    import torch
    import paper_1811_04165_amd as amber
    tiles = None if threads is None else amber.make_tiles(snr_threads=threads)
    rows = np.full((dd.shape[0], dd.shape[1] + pad), 1 << 30, dtype=np.int32)
    rows[:, :dd.shape[1]] = dd
    s, p = amber.integrate_snr(torch.from_numpy(rows).cuda(), dd.shape[1], widths, tiles=tiles)
    for k, w in enumerate(widths):
        ref_s, ref_p = oracle.snr(oracle.boxcar(dd, w))
        np.testing.assert_allclose(s[k].cpu().numpy().astype(np.float64), ref_s, rtol=1e-5, atol=1e-6)
        np.testing.assert_array_equal(p[k].cpu().numpy(), ref_p)


def test_lane_sums_between_63_and_64_bits():
    """Rows centred on a first sample of 0: one wavefront's lane adds 168
    squares of 512 * 6e5, 1.6e19, below the bound of 1.8e19 and above 2^63."""
    print("[case] lane sums past 63 bits", flush=True)
    rng = np.random.default_rng(1)
    dd = rng.integers(598000, 602000, size=(3, 256 * 44)).astype(np.int32)
    dd[:, 0] = 0
    assert 164 * (512 * 598000) ** 2 > 2 ** 63 and 176 * (512 * 602000) ** 2 < 1.8e19
    _check(dd, (512,), 64)


POW2 = tuple(1 << k for k in range(11))


@pytest.mark.parametrize("n_out,widths,threads,low,high", [
    (120000, (1, 512, 700, 1024), 128, 150000, 250000),   # a wide boxcar and a long row
    (120003, POW2, 128, 150000, 250000),
    (6000, (1, 3, 64), 64, 7900000, 8000000),             # the narrow form
    (5001, POW2[:7], 128, 19000000, 20000000),            # samples past 2^23: every width again, more than a sweep takes
    (1030, (1024, 1023), 512, 2085000, 2090000),          # more wavefronts than blocks
    (1030, (1024,), 128, 2085000, 2090000),
    (300, (64,), 64, 33000000, 33500000),                 # boxcars just below 2^31
])
def test_rows_far_from_their_first_sample(n_out, widths, threads, low, high):
    """Sums that 64 bits do not hold about the first sample (0, and a common
    one in the second row) are taken again in FP64 by all wavefronts."""
    print("[case] far rows", n_out, widths, threads, flush=True)
    rng = np.random.default_rng([n_out, len(widths)])
    dd = rng.integers(low, high, size=(5, n_out)).astype(np.int32)
    dd[0, 0] = 0
    dd[2:, 0] = 0
    dd[3, 1:] = low                                       # ties
    dd[4, n_out - 1] = high                               # the last sample
    for pad in (0, 3, (-n_out) % 4):
        _check(dd, widths, threads, pad)
