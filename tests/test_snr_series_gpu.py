"""S/N of materialised boxcar series against the oracle: rows around the
256-value blocks, more wavefronts than blocks, rows of any alignment, ties
within a group of four and across blocks, maxima at the row's end, signed
values.  S/N within 1e-5 relative, peak indices exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [64, 128, 1024])
@pytest.mark.parametrize("n_out", [1, 3, 255, 256, 257, 1029, 5121])
def test_series(n_out, threads):
    import torch
    import paper_1811_04165_amd as amber
    print("[case] series", n_out, threads, flush=True)
    rng = np.random.default_rng([n_out, threads])
    widths = tuple(w for w in (1, 2, 5, 64, 255) if w <= n_out and 32 * w <= 32 * threads)
    n_dm = 6
    dd = rng.integers(-200000, 250000, size=(n_dm, n_out)).astype(np.int32)
    dd[1] = 7                                   # constant: the first index, S/N 0
    dd[2, n_out - 1] = 900000                   # the last value
    dd[3, n_out // 2:] = 900000                 # ties over many blocks
    dd[4, [min(2, n_out - 1), n_out // 3, n_out - 1]] = 900000
    series = [oracle.boxcar(dd, w) for w in widths]
    for stride in (n_out, (n_out + 3) // 4 * 4, (n_out + 3) // 4 * 4 + 3):
        box = np.full((len(widths), n_dm, stride), 1 << 30, dtype=np.int32)
        for k, w in enumerate(widths):
            box[k, :, :n_out - w + 1] = series[k]
        s, p = amber.snr(torch.from_numpy(box).cuda(), n_out, widths, tiles=amber.make_tiles(snr_threads=threads))
        for k in range(len(widths)):
            ref_s, ref_p = oracle.snr(series[k])
            np.testing.assert_allclose(s[k].cpu().numpy().astype(np.float64), ref_s, rtol=1e-5, atol=1e-6)
            np.testing.assert_array_equal(p[k].cpu().numpy(), ref_p)
