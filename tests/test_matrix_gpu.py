"""Dedispersion on the matrix cores against the CPU oracle, bit for bit, at the
edges of its tiles, channel groups, remainder passes and of the rule that
chooses it (256 channels and a group of alike channels)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amber():
    import paper_1811_04165_amd as amber
    return amber


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


def _problem(amber, torch, n_chan, n_dm, n_out, dm0, step, order="asc", keep=None, pad=0, seed=0):
    rng = np.random.default_rng([7, n_chan, n_dm, n_out, seed])
    f = 1250.0 + np.arange(n_chan) * 300.0 / n_chan
    if order == "desc":
        f = f[::-1].copy()
    elif order == "swapped":  # neighbours 16 apart change places: several passes of remainders
        f = f[np.arange(n_chan) ^ 16] if n_chan % 32 == 0 else f
    elif order == "shuffled":  # no group's channels move alike
        f = rng.permutation(f)
    d, info = amber.delay_table(f, 81.92e-6, n_dm, dm0, step)
    n_in = n_out + info.max_delay
    x = rng.integers(0, 256, size=(n_chan, (n_in + 3) // 4 * 4 + pad), dtype=np.uint8)
    x[:, :n_out // 3] = rng.choice(np.array([0, 255], dtype=np.uint8), size=(n_chan, 1))  # the sums' extremes
    k = None
    if keep == "some":
        k = (rng.random(n_chan) > 0.2).astype(np.uint8)
        k[64:100] = 0  # a whole group and part of the next
    elif keep == "none":
        k = np.zeros(n_chan, dtype=np.uint8)
    ref = oracle.dedisperse(d, x, n_in, n_out) if k is None else oracle.dedisperse_masked(d, x, n_in, n_out, k)
    dev = dict(delays=torch.from_numpy(d).cuda(), info=info, x=torch.from_numpy(x).cuda(), n_in=n_in, n_out=n_out,
               keep=None if k is None else torch.from_numpy(k).cuda())
    return dev, ref


CASES = [
    # n_chan, n_dm, n_out, first DM, DM step, options
    (255, 33, 700, 0.0, 0.25, {}),                       # one channel below the rule's edge
    (256, 32, 640, 0.0, 0.25, {}),                       # whole tiles and groups
    (257, 33, 641, 0.0, 0.25, {"pad": 4}),               # one more of each
    (256, 1, 1, 0.0, 0.0, {"pad": 28}),                  # the smallest problem (rows are 32 bytes at least)
    (256, 31, 33, 0.0, 0.5, {"keep": "some"}),
    (387, 77, 901, 57.3, 0.35, {}),
    (1536, 96, 1300, 900.0, 0.5, {"pad": 12}),
    (1536, 65, 2049, 0.0, 0.5, {"keep": "some"}),
    (512, 64, 777, 0.0, 0.5, {"keep": "none"}),
    (500, 70, 703, 300.0, 0.25, {"order": "desc", "keep": "some"}),
    (320, 40, 600, 10.0, 0.25, {"order": "swapped"}),
    (320, 40, 600, 0.0, 1.0, {"order": "swapped"}),      # the rule's other edge: too coarse
    (288, 64, 1500, 10.0, 0.25, {"order": "shuffled", "keep": "some"}),
    (1536, 64, 515, 0.0, 4.0, {}),                       # twelve remainders a pass
]


@pytest.mark.parametrize("n_chan,n_dm,n_out,dm0,step,opt", CASES, ids=lambda v: str(v))
def test_matrix_against_oracle(amber, torch, n_chan, n_dm, n_out, dm0, step, opt):
    print("[case] matrix", n_chan, n_dm, n_out, dm0, step, opt, flush=True)
    p, ref = _problem(amber, torch, n_chan, n_dm, n_out, dm0, step, **opt)
    # automatic tiles; explicit tiles of 32 trials, which take the same kernel
    # (both row lengths), and of 8, which do not; rows of an odd stride
    sets = [None, amber.make_tiles(dms_per_block=16, dms_per_thread=2, samples_per_thread=4, channel_unroll=16),
            amber.make_tiles(dms_per_block=8, dms_per_thread=1, samples_per_thread=8, channel_unroll=16)]
    for t in sets:
        if t is not None:
            try:
                amber.validate_tiles(t, p["info"], 1)
            except amber.AmberError:
                continue
        for stride in (n_out, n_out + 5, (n_out + 3) // 4 * 4):
            out = torch.full((n_dm, stride), -7, dtype=torch.int32, device="cuda")
            amber.dedisperse(p["delays"], p["info"], p["x"], p["n_in"], n_out, tiles=t, keep=p["keep"],
                             out=out[:, :n_out] if stride != n_out else out)
            got = out.cpu().numpy()
            np.testing.assert_array_equal(got[:, :n_out], ref)
            assert (got[:, n_out:] == -7).all(), "columns past n_out"


def test_matrix_beams_in_one_batch(amber, torch):
    """Beams of the matrix kernel's different forms (remainders per pass, tile
    lengths) and one below its edge, eager and replayed."""
    widths = (1, 2, 4)
    beams, refs = [], []
    for b, (n_chan, n_dm, n_out, dm0, step, opt) in enumerate([CASES[0], CASES[2], CASES[5], CASES[6], CASES[13]]):
        p, ref = _problem(amber, torch, n_chan, n_dm, n_out, dm0, step, seed=b, **opt)
        p["dd"] = torch.full((n_dm, n_out + 3), -1, dtype=torch.int32, device="cuda")
        p["snr"] = torch.zeros((len(widths), n_dm), dtype=torch.float32, device="cuda")
        p["peak"] = torch.zeros((len(widths), n_dm), dtype=torch.int32, device="cuda")
        beams.append(p)
        refs.append(ref)
    print("[case] matrix batch", flush=True)
    batch = amber.Batch(beams, widths)
    batch.run()
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        batch.capture(stream)
    for turn in range(3):
        for p, ref in zip(beams, refs):
            np.testing.assert_array_equal(p["dd"][:, :p["n_out"]].cpu().numpy(), ref)
            p["dd"].fill_(-1)
        torch.cuda.synchronize()
        batch.launch(stream)
        torch.cuda.synchronize()
    batch.close()


@pytest.mark.parametrize("cases", [[2, 5, 6, 13], [0, 2, 5]])
def test_matrix_beams_with_one_tile_set(amber, torch, cases):
    """Beams given the same explicit tiles of 32 trials are one launch, whether
    all of them can take the matrix cores or not."""
    print("[case] matrix batch, one tile set", cases, flush=True)
    tiles = amber.make_tiles(dms_per_block=16, dms_per_thread=2, samples_per_thread=4, channel_unroll=8)
    beams, refs = [], []
    for b, c in enumerate(cases):
        n_chan, n_dm, n_out, dm0, step, opt = CASES[c]
        p, ref = _problem(amber, torch, n_chan, n_dm, n_out, dm0, min(step, 0.5), seed=b, **opt)
        p["dd"] = torch.full((n_dm, n_out), -1, dtype=torch.int32, device="cuda")
        p["snr"] = torch.zeros((1, n_dm), dtype=torch.float32, device="cuda")
        p["peak"] = torch.zeros((1, n_dm), dtype=torch.int32, device="cuda")
        beams.append(p)
        refs.append(ref)
    batch = amber.Batch(beams, (1,), tiles=[tiles] * len(beams))
    assert batch.launches() == (1, 1)
    batch.run()
    torch.cuda.synchronize()
    for p, ref in zip(beams, refs):
        np.testing.assert_array_equal(p["dd"].cpu().numpy(), ref)
    batch.close()
