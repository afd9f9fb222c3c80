"""Decimated S/N over wavefront spans against the oracle: bins that cross
chunks and spans (or hold whole spans), rows of exactly one or more chunks and
just beside them, more wavefronts than chunks, factor 1 in any place and twice,
up to 16 factors, ties, rows of any alignment.  S/N within 1e-5 relative
(float32 results of FP64 sums), peak indices exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dm,n_out,factors,threads,ties", [
    (37, 12208, (1, 10, 20, 40, 80, 160, 320, 640, 1280, 3200), None, False),
    (5, 4096, (1, 2, 4, 1024, 4096, 3, 1023, 1025), 512, False),   # four whole chunks, the row one bin
    (5, 8192, (7, 1, 1, 64, 65, 2048, 2049, 4095), 512, False),
    (5, 8193, (2048, 4096, 8), 256, False),
    (3, 5000, (2500, 4096, 5, 1, 1000), 1024, True),
    (2, 25600, tuple(range(1, 17)), 256, False),
    (2, 2047, tuple(range(3, 16)), 64, True),
    (4, 3, (1, 2, 3), None, False),
    (4, 1, (1,), 64, False),
    (4100, 1024, (1024, 512, 341), None, False),                   # one wavefront a row
    (3, 1025, (1024, 1025, 1), 128, False),
])
def test_spans(n_dm, n_out, factors, threads, ties):
    import torch
    import paper_1811_04165_amd as amber
    print("[case] decimated spans", n_dm, n_out, factors, threads, ties, flush=True)
    rng = np.random.default_rng([n_dm, n_out])
    dd = rng.integers(150000, 250000, size=(n_dm, n_out)).astype(np.int32)
    if ties:
        dd[:] = 200000
        dd[1, n_out // 2:n_out // 2 + 50] += 5
    ref = [oracle.snr(oracle.downsample(dd, f)) for f in factors]
    tiles = None if threads is None else amber.make_tiles(snr_threads=threads)
    for pad in (0, 3, (-n_out) % 4):
        rows = np.full((n_dm, n_out + pad), 1 << 20, dtype=np.int32)
        rows[:, :n_out] = dd
        try:
            s, p = amber.downsample_snr(torch.from_numpy(rows).cuda(), n_out, factors, tiles=tiles)
        except amber.AmberError:
            assert threads is not None and threads * 16 < 2 * max(factors)  # the factor's limit for explicit tiles
            continue
        for k in range(len(factors)):
            np.testing.assert_allclose(s[k].cpu().numpy().astype(np.float64), ref[k][0], rtol=1e-5, atol=1e-6)
            np.testing.assert_array_equal(p[k].cpu().numpy(), ref[k][1])
