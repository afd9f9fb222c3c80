"""Dedispersion on the matrix cores for any order of the channels, against the
CPU oracle, bit for bit: descending bands from DM 0, whose windows begin before
the first sample and whose remainders take several passes, sub-bands listed one
after the other or in turn, and no order at all."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _band(n_chan, order):
    f = 1250.0 + np.arange(n_chan) * 300.0 / n_chan
    if order == "desc":
        return f[::-1].copy()
    if order.startswith("blocks"):   # sub-bands in ascending order, each descending
        return f.reshape(int(order[6:]), -1)[:, ::-1].reshape(-1).copy()
    if order.startswith("turns"):    # one channel of each sub-band in turn
        return f.reshape(int(order[5:]), -1).T.reshape(-1).copy()
    if order == "shuffled":
        return np.random.default_rng(n_chan).permutation(f)
    return f


CASES = [
    # n_chan, n_dm, n_out, first DM, DM step, order
    (256, 31, 700, 0.0, 0.5, "desc"),
    (256, 64, 641, 0.0, 0.5, "desc"),
    (288, 33, 300, 0.0, 0.25, "desc"),
    (768, 64, 900, 0.0, 0.5, "desc"),
    (768, 40, 515, 0.0, 0.5, "blocks4"),
    (1536, 64, 700, 0.0, 0.1, "turns3"),
    (384, 64, 700, 0.0, 0.1, "turns3"),
    (384, 64, 700, 0.0, 0.1, "shuffled"),
    (1536, 33, 515, 0.0, 0.5, "turns2"),
    (1536, 33, 515, 0.0, 2.0, "shuffled"),
    (2304, 33, 300, 0.0, 0.25, "shuffled"),   # more channels than are sorted together
    (387, 70, 643, 57.3, 0.35, "shuffled"),
    (300, 40, 200, 0.0, 0.25, "blocks2"),     # a group on both sides of the sub-bands' border
    (1536, 40, 300, 0.0, 0.5, "turns128"),    # groups that sweep over a quarter of the band
]


@pytest.mark.parametrize("zapped", [False, True])
@pytest.mark.parametrize("n_chan,n_dm,n_out,dm0,step,order", CASES)
def test_any_order(n_chan, n_dm, n_out, dm0, step, order, zapped):
    import torch
    import paper_1811_04165_amd as amber
    print("[case] matrix order", n_chan, n_dm, n_out, dm0, step, order, zapped, flush=True)
    rng = np.random.default_rng([n_chan, n_dm, n_out])
    d, info = amber.delay_table(_band(n_chan, order), 81.92e-6, n_dm, dm0, step)
    n_in = n_out + info.max_delay
    # no byte to spare after the last row
    x = rng.integers(0, 256, size=(n_chan, max(32, (n_in + 3) // 4 * 4)), dtype=np.uint8)
    keep = (rng.random(n_chan) > 0.15).astype(np.uint8) if zapped else None
    ref = oracle.dedisperse_masked(d, x, n_in, n_out, keep) if zapped else oracle.dedisperse(d, x, n_in, n_out)
    dd = amber.dedisperse(torch.from_numpy(d).cuda(), info, torch.from_numpy(x).cuda(), n_in, n_out,
                          keep=None if keep is None else torch.from_numpy(keep).cuda())
    np.testing.assert_array_equal(dd.cpu().numpy(), ref)


def test_rows_that_limit_what_is_sorted_together():
    """Rows so far apart that 32-bit offsets reach 224 of 320 shuffled channels."""
    import torch
    import paper_1811_04165_amd as amber
    n_chan, n_dm, n_out, stride = 320, 33, 300, (1 << 24) + 256
    print("[case] matrix order, far rows", flush=True)
    rng = np.random.default_rng(5)
    d, info = amber.delay_table(_band(n_chan, "shuffled"), 81.92e-6, n_dm, 0.0, 0.5)
    n_in = n_out + info.max_delay
    x = rng.integers(0, 256, size=(n_chan, (n_in + 3) // 4 * 4), dtype=np.uint8)
    far = torch.zeros((n_chan, stride), dtype=torch.uint8, device="cuda")
    far[:, :x.shape[1]] = torch.from_numpy(x).cuda()
    dd = amber.dedisperse(torch.from_numpy(d).cuda(), info, far, n_in, n_out)
    np.testing.assert_array_equal(dd.cpu().numpy(), oracle.dedisperse(d, x, n_in, n_out))


@pytest.mark.parametrize("zapped", [False, True])
def test_table_of_no_dispersion_law(zapped):
    """Channels that move as far at other trials, which no order makes alike."""
    import torch
    import paper_1811_04165_amd as amber
    n_chan, n_dm, n_out = 288, 96, 1100
    print("[case] matrix order, no law", zapped, flush=True)
    rng = np.random.default_rng(6)
    i = np.arange(n_dm)[:, None]
    late = (np.arange(n_chan) % 2 == 1)[None, :]
    d = np.where(late, 10 * np.clip(i - 16, 0, 16), 10 * np.minimum(i, 16)).astype(np.int32)
    d += (np.arange(n_chan) % 7).astype(np.int32)[None, :]
    _, info = amber.delay_table(_band(n_chan, "asc"), 81.92e-6, n_dm, 0.0, 0.0)
    info.max_delay, info.max_step = int(d.max()), 10
    n_in = n_out + info.max_delay
    x = rng.integers(0, 256, size=(n_chan, (n_in + 3) // 4 * 4), dtype=np.uint8)
    keep = (rng.random(n_chan) > 0.15).astype(np.uint8) if zapped else np.ones(n_chan, dtype=np.uint8)
    dd = amber.dedisperse(torch.from_numpy(d).cuda(), info, torch.from_numpy(x).cuda(), n_in, n_out,
                          keep=torch.from_numpy(keep).cuda() if zapped else None)
    np.testing.assert_array_equal(dd.cpu().numpy(), oracle.dedisperse_masked(d, x, n_in, n_out, keep))
