"""Decimated S/N with automatic tiles where the number of wavefronts per row
changes (more than 12 factors, short rows, many rows), against the oracle: S/N
within 1e-5 relative (float32 results of FP64 sums), peak indices exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dm,n_out,factors", [
    (1024, 1300, tuple(range(1, 14))), (1025, 1300, tuple(range(1, 14))), (2049, 1030, tuple(range(2, 18))),
    (300, 1200, tuple(range(1, 17))), (300, 1024, (1, 7, 600)), (5, 3000, (1, 10, 1500)),
])
def test_automatic_wavefronts(n_dm, n_out, factors):
    import torch
    import paper_1811_04165_amd as amber
    print("[case] decimated, automatic", n_dm, n_out, len(factors), flush=True)
    rng = np.random.default_rng([n_dm, n_out])
    dd = rng.integers(150000, 250000, size=(n_dm, n_out)).astype(np.int32)
    s, p = amber.downsample_snr(torch.from_numpy(dd).cuda(), n_out, factors)
    for k, f in enumerate(factors):
        ref_s, ref_p = oracle.snr(oracle.downsample(dd, f))
        np.testing.assert_allclose(s[k].cpu().numpy().astype(np.float64), ref_s, rtol=1e-5, atol=1e-6)
        np.testing.assert_array_equal(p[k].cpu().numpy(), ref_p)
