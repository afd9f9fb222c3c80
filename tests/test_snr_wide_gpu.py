"""The fused boxcar / S/N kernel's wide form (widths up to 1024, up to 16 of
them) against the oracle: row lengths around its blocks and lookahead, widths
at the edges of both forms and of a read's alignment, every work-group size,
rows of any alignment, ties, and rows far from the sample they are centred on
(sums of squares beyond 64 bits).  S/N within 1e-5 relative, as the narrow
form (float32 results of exact sums), peak indices exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

POW2 = tuple(1 << k for k in range(11))


@pytest.fixture(scope="module")
def amber():
    import paper_1811_04165_amd as amber
    return amber


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


@pytest.mark.parametrize("n_dm,n_out,widths,threads,kind", [
    (37, 1024, POW2, None, "noise"),              # the longest window is the row
    (5, 1023, POW2[:10], 64, "noise"),
    (7, 1281, POW2[:9], 128, "noise"),
    (9, 5000, POW2, 1024, "ties"),                # more threads than the wide form takes
    (7, 24576, POW2, None, "zero first"),
    (3, 999, (1, 3, 5, 9, 20, 45, 77, 300, 999), None, "noise"),
    (5, 2500, (1000, 1024, 1023, 517, 2, 256, 257, 255, 1, 64, 65, 66, 128), 256, "far"),
    (4, 7000, tuple(range(1, 17)), None, "noise"),  # more than 8 widths, none above 64
    (4, 7000, tuple(range(50, 66)), None, "noise"),
    (3, 300, (65,), 64, "noise"),
    (3, 6001, (65, 1024), 512, "beyond 64 bits"),
])
def test_wide_widths(amber, torch, n_dm, n_out, widths, threads, kind):
    print("[case] wide", n_dm, n_out, widths, threads, kind, flush=True)
    rng = np.random.default_rng([n_dm, n_out, len(widths)])
    dd = rng.integers(150000, 250000, size=(n_dm, n_out)).astype(np.int32)
    if kind == "ties":
        dd[:] = 200000
        dd[1, 500:700] += 5
    elif kind == "zero first":
        dd[:, 0] = 0
    elif kind == "far":
        dd[:, :10] = -3000000
        dd[2] = 7
    elif kind == "beyond 64 bits":
        dd[:, 0] = 2000000
        dd[:, 1:] -= 1800000
    ref_s, ref_p = np.empty((len(widths), n_dm)), np.empty((len(widths), n_dm), dtype=np.int32)
    for k, w in enumerate(widths):
        ref_s[k], ref_p[k] = oracle.snr(oracle.boxcar(dd, w))
    tiles = None if threads is None else amber.make_tiles(snr_threads=threads)
    for pad in (0, 3, (-n_out) % 4):
        rows = np.full((n_dm, n_out + pad), 1 << 30, dtype=np.int32)
        rows[:, :n_out] = dd
        s, p = amber.integrate_snr(torch.from_numpy(rows).cuda(), n_out, widths, tiles=tiles)
        np.testing.assert_allclose(s.cpu().numpy().astype(np.float64), ref_s, rtol=1e-5, atol=1e-6)
        np.testing.assert_array_equal(p.cpu().numpy(), ref_p)


def test_wide_widths_of_a_batch(amber, torch):
    """More than 8 widths up to 64, and wide ones, over a table of beams."""
    for widths in (tuple(range(1, 13)), (1, 2, 100, 1024)):
        print("[case] wide batch", widths, flush=True)
        rng = np.random.default_rng(len(widths))
        beams, dds = [], []
        for n_dm, n_out in ((3, 1100), (5, 2051)):
            f = 1250.0 + np.arange(16) * 300.0 / 16
            d, info = amber.delay_table(f, 81.92e-6, n_dm, 0.0, 0.5)
            n_in = n_out + info.max_delay
            x = rng.integers(0, 256, size=(16, (n_in + 31) // 4 * 4), dtype=np.uint8)
            dds.append(oracle.dedisperse(d, x, n_in, n_out))
            beams.append(dict(delays=torch.from_numpy(d).cuda(), info=info, x=torch.from_numpy(x).cuda(), n_in=n_in,
                              n_out=n_out, dd=torch.zeros((n_dm, n_out), dtype=torch.int32, device="cuda"),
                              snr=torch.zeros((len(widths), n_dm), dtype=torch.float32, device="cuda"),
                              peak=torch.zeros((len(widths), n_dm), dtype=torch.int32, device="cuda")))
        batch = amber.Batch(beams, widths)
        batch.run()
        torch.cuda.synchronize()
        for b, dd in zip(beams, dds):
            for k, w in enumerate(widths):
                s, p = oracle.snr(oracle.boxcar(dd, w))
                np.testing.assert_allclose(b["snr"][k].cpu().numpy().astype(np.float64), s, rtol=1e-5, atol=1e-6)
                np.testing.assert_array_equal(b["peak"][k].cpu().numpy(), p)
        batch.close()
