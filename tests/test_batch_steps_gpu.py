"""Beams of a batch whose tiles differ only in the steps that their boxcar /
S/N kernel does not have run in one launch each of both kernels."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths", [(1, 2, 4), (1, 100, 300)])
def test_steps_do_not_split_launches(widths):
    import torch
    import paper_1811_04165_amd as amber
    print("[case] batch steps", widths, flush=True)
    rng = np.random.default_rng(2)
    beams, refs = [], []
    for n_out in (700, 901):
        d, info = amber.delay_table(1250.0 + np.arange(32) * 300.0 / 32, 81.92e-6, 6, 0.0, 0.5)
        n_in = n_out + info.max_delay
        x = rng.integers(0, 256, size=(32, (n_in + 31) // 4 * 4), dtype=np.uint8)
        refs.append(oracle.dedisperse(d, x, n_in, n_out))
        beams.append(dict(delays=torch.from_numpy(d).cuda(), info=info, x=torch.from_numpy(x).cuda(), n_in=n_in,
                          n_out=n_out, dd=torch.zeros((6, n_out), dtype=torch.int32, device="cuda"),
                          snr=torch.zeros((len(widths), 6), dtype=torch.float32, device="cuda"),
                          peak=torch.zeros((len(widths), 6), dtype=torch.int32, device="cuda")))
    batch = amber.Batch(beams, widths, tiles=[amber.make_tiles(boxcar_step=s) for s in (8, 2)])
    assert batch.launches() == (1, 1)
    batch.run()
    torch.cuda.synchronize()
    for b, dd in zip(beams, refs):
        for k, w in enumerate(widths):
            s, p = oracle.snr(oracle.boxcar(dd, w))
            np.testing.assert_allclose(b["snr"][k].cpu().numpy().astype(np.float64), s, rtol=1e-5, atol=1e-6)
            np.testing.assert_array_equal(b["peak"][k].cpu().numpy(), p)
    batch.close()
