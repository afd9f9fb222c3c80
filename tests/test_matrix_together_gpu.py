"""Beams that run together on the matrix cores: one launch per form of the
kernel or per explicit tile set, in batches and in the streaming service, and
the oracle's results, bit for bit (S/N within 1e-5, peaks exactly)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

WIDTHS = (1, 2, 4, 8)


@pytest.fixture(scope="module")
def amber():
    import paper_1811_04165_amd as amber
    return amber


def _freqs(n_chan):
    return 1250.0 + np.arange(n_chan) * 300.0 / n_chan


@pytest.mark.parametrize("beams,launches", [
    # (channels, DMs, samples, DM step) of each beam
    ([(256, 64, 1500, 0.1), (300, 40, 2700, 0.1), (512, 96, 611, 0.2)], 1),
    ([(256, 64, 1500, 0.1), (512, 70, 900, 0.4), (300, 33, 2000, 0.1), (384, 64, 700, 0.5), (128, 40, 900, 0.5)], 4),
])
def test_batch_launches(amber, beams, launches):
    import torch
    print("[case] matrix beams together", beams, flush=True)
    rng = np.random.default_rng(len(beams))
    made, refs = [], []
    for n_chan, n_dm, n_out, step in beams:
        d, info = amber.delay_table(_freqs(n_chan), 81.92e-6, n_dm, 0.0, step)
        n_in = n_out + info.max_delay
        x = rng.integers(0, 256, size=(n_chan, (n_in + 31) // 4 * 4), dtype=np.uint8)
        refs.append(oracle.dedisperse(d, x, n_in, n_out))
        made.append(dict(delays=torch.from_numpy(d).cuda(), info=info, x=torch.from_numpy(x).cuda(), n_in=n_in,
                         n_out=n_out, dd=torch.full((n_dm, n_out), -1, dtype=torch.int32, device="cuda"),
                         snr=torch.zeros((len(WIDTHS), n_dm), dtype=torch.float32, device="cuda"),
                         peak=torch.zeros((len(WIDTHS), n_dm), dtype=torch.int32, device="cuda")))
    batch = amber.Batch(made, WIDTHS)
    assert batch.launches() == (launches, 1)
    batch.run()
    torch.cuda.synchronize()
    for p, ref in zip(made, refs):
        np.testing.assert_array_equal(p["dd"].cpu().numpy(), ref)
    batch.close()


@pytest.mark.parametrize("tiles", [False, True])
def test_streamed_beams(amber, tiles):
    """Chunks of several beams fused into one launch group, with automatic
    tiles and with one explicit set of 32 trials that one beam cannot run on the
    matrix cores."""
    L, n_chunks = 1200, 4
    t = amber.make_tiles(dms_per_block=16, dms_per_thread=2, samples_per_thread=4, channel_unroll=8) if tiles else None
    print("[case] streamed matrix beams", tiles, flush=True)
    rng = np.random.default_rng(3)
    geoms = [(256, 64, 0.1), (255 if tiles else 300, 40, 0.1), (512, 70, 0.4)]
    data = []
    for n_chan, n_dm, step in geoms:
        d, info = amber.delay_table(_freqs(n_chan), 81.92e-6, n_dm, 0.0, step)
        x = rng.integers(0, 256, size=(n_chan, n_chunks * L), dtype=np.uint8)
        data.append((d, info, x, oracle.dedisperse(d, x, n_chunks * L, n_chunks * L - info.max_delay)))
    with amber.Server(max_inflight=8, max_batch=8, n_streams=2) as srv:
        for (n_chan, n_dm, step), _ in zip(geoms, data):
            srv.add_beam(_freqs(n_chan), 81.92e-6, n_dm, 0.0, step, L, WIDTHS, tiles=t)
        for k in range(n_chunks):
            for b, (_, _, x, _) in enumerate(data):
                srv.submit(b, x[:, k * L:(k + 1) * L])
        results = [srv.wait(60.0) for _ in range(n_chunks * len(geoms))]
    assert all(r is not None for r in results)
    for r in results:
        dd, mx = data[r["beam"]][3], data[r["beam"]][1].max_delay
        t0, n = amber.chunk_span(r["seq"], L, mx)
        assert (r["t_first"], r["n_out"]) == (t0, n) and r["has_snr"] == 1
        for k, w in enumerate(WIDTHS):
            s, p = oracle.snr(oracle.boxcar(dd[:, t0:t0 + n], w))
            np.testing.assert_allclose(r["snr"][k].astype(np.float64), s, rtol=1e-5, atol=1e-6)
            np.testing.assert_array_equal(r["peak"][k], p)
