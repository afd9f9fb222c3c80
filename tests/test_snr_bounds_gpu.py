"""The fused boxcar / S/N kernel's sums of squares at the limits of what they
hold, against the oracle: S/N within 1e-5 relative (float32 results), peak
indices exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _check(dd, widths, threads):
    import torch
    import paper_1811_04165_amd as amber
    tiles = None if threads is None else amber.make_tiles(snr_threads=threads)
    s, p = amber.integrate_snr(torch.from_numpy(dd).cuda(), dd.shape[1], widths, tiles=tiles)
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
