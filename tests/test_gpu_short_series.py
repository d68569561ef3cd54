"""Short series have a kernel of their own, one row of 512 window ends per wave.
Lengths around its rows and around the last one it takes, windows of a few
cells, of a row and of more than the series, steps within and beyond a row,
missing values and constant stretches; each also on the kernel of long series
(debug bit 1), with its LDS ring and without (bits 1 and 2).  Against the
oracle: integer input bit for bit, float input within 2^-24 (float32 rounding
of the output), flags identical."""
import numpy as np
import pytest

from gpu_util import compare
from workloads import random_pair

pytestmark = pytest.mark.gpu

# rows of 512 window ends, as many as the GPU has CUs
LAST = 256 * 512


@pytest.fixture(params=[0, 2, 6])
def form(request):
    import paper_1807_06507_amd as swc
    before = swc.get_debug()
    swc.set_debug(request.param)
    yield request.param
    swc.set_debug(before)


def _pair(n, dtype, seed):
    x, y = random_pair((n,), dtype, seed=seed)
    if n > 40:
        x[n // 2:n // 2 + 20] = 3
        y[n // 3:n // 3 + 17] = 5
        if dtype == "f32":
            x[n // 5] = -999.0
            y[n - 1] = np.nan
            x[n // 2 + 30:n // 2 + 33] = np.inf
    return x, y


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("n", [1, 2, 7, 64, 511, 512, 513, 1024, 1100, 4099])
def test_lengths_and_windows(form, dtype, n):
    x, y = _pair(n, dtype, n)
    for k in (1, 2, 7, 8, 9, 100, 512, 513, n + 3):
        if dtype == "u16" and k > 1448:
            continue
        for border in ("fill", "clip", "valid"):
            if border == "valid" and k > n:
                continue
            compare(x, y, (k,), 1, border, tag=f"short series form={form}")


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("step", [2, 5, 17, 511, 600, 5000])
def test_steps(form, dtype, step):
    x, y = _pair(6007, dtype, step)
    for k, border in ((1, "clip"), (6, "fill"), (31, "clip"), (700, "valid")):
        compare(x, y, (k,), step, border, tag=f"short series form={form}")


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("n", [LAST - 1, LAST, LAST + 1, LAST + 700])
def test_last_length(form, dtype, n):
    x, y = _pair(n, dtype, 3)
    compare(x, y, (33,), 1, "clip", tag=f"short series form={form}")
    compare(x, y, (1200,), 3, "fill", tag=f"short series form={form}")
