"""S/N of materialised series that hold the type's lowest value, as masks do:
rows of nothing else (S/N 0, peak 0), rows with one other value and ordinary
ones, at lengths below, at and beyond a block of 256 and of every work-group
size.  S/N within 1e-5 relative, peak indices exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

LOWEST = np.iinfo(np.int32).min


@pytest.mark.parametrize("threads", [64, 128, 1024])
@pytest.mark.parametrize("n_out", [1, 3, 255, 256, 1029])
def test_lowest_values(n_out, threads):
    import torch
    import paper_1811_04165_amd as amber
    print("[case] lowest values", n_out, threads, flush=True)
    rng = np.random.default_rng([n_out, threads])
    box = rng.integers(-200000, 250000, size=(1, 6, n_out)).astype(np.int32)
    box[0, 0] = LOWEST
    box[0, 2] = LOWEST
    box[0, 2, n_out - 1] = LOWEST + 1
    box[0, 3, :n_out // 2] = LOWEST
    box[0, 5] = LOWEST
    ref_s, ref_p = oracle.snr(box[0])
    assert ref_s[0] == 0.0 and ref_p[0] == 0 and ref_p[2] == n_out - 1
    s, p = amber.snr(torch.from_numpy(box).cuda(), n_out, (1,), tiles=amber.make_tiles(snr_threads=threads))
    np.testing.assert_allclose(s[0].cpu().numpy().astype(np.float64), ref_s, rtol=1e-5, atol=1e-6)
    np.testing.assert_array_equal(p[0].cpu().numpy(), ref_p)
