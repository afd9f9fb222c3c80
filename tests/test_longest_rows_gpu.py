"""S/N of rows on both sides of 2^29 samples, where the sweeps over spans end
and the kernels of LDS chunks begin: zeros with a few pulses far apart, whose
moments and peaks follow in whole numbers.  S/N within 1e-6 relative (FP64
moments, a float32 result)."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 1 << 29
PULSES = [(70001, 900), (N // 2 + 5, 1000), (N - 70003, 1000)]  # sample, value


def _snr(n, total, squares, top):
    mean = total / n
    return (top - mean) / math.sqrt(squares / n - mean * mean)


@pytest.mark.parametrize("n_out", [N - 1, N, N + 1001])
def test_rows(n_out):
    import torch
    import paper_1811_04165_amd as amber
    print("[case] longest rows", n_out, flush=True)
    row = torch.zeros((1, n_out), dtype=torch.int32, device="cuda")
    for at, v in PULSES:
        row[0, at] = v
    total, squares = sum(v for _, v in PULSES), sum(v * v for _, v in PULSES)
    for widths in ((1, 3, 64), (5, 1024)):
        s, p = amber.integrate_snr(row, n_out, widths)
        for k, w in enumerate(widths):
            np.testing.assert_allclose(float(s[k, 0]), _snr(n_out - w + 1, w * total, w * squares, 1000), rtol=1e-6)
            assert int(p[k, 0]) == PULSES[1][0] - w + 1
    factors = (1, 10, 3200)
    s, p = amber.downsample_snr(row, n_out, factors)
    for k, f in enumerate(factors):
        np.testing.assert_allclose(float(s[k, 0]), _snr(n_out // f, total, squares, 1000), rtol=1e-6)
        assert int(p[k, 0]) == PULSES[1][0] // f
