"""The 1-D kernel's row forms against the oracle (integer input bit for bit,
float input within 2^-24, flags identical): straight-line rows inside the
series, the rolled loop at its ends and in partial rows, the masked copy for
rows holding missing values, and rows taken once more because a window is not
settled by its estimate.  Lengths around one, two and three rows of 512
positions and around the segments a wave takes; integer arrays at any byte.
"""
import numpy as np
import pytest

from gpu_util import compare, say, to_dev
from workloads import random_pair
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 512, 513, 1400])
def test_row_boundaries(dtype, k):
    for n in (511, 512, 1025, 1536, 2049, 5001):
        x, y = random_pair((n,), dtype, seed=n + k)
        for border, step in (("clip", 1), ("fill", 3), ("valid", 1)):
            if border == "valid" and n < k:
                continue
            for params in (None, (8, 2, 1)):
                compare(x, y, (k,), step, border, params=params, tag="series rows")


@pytest.mark.parametrize("dtype,offsets", [("u8", (1, 2)), ("u8", (3, 0)), ("u16", (1, 0)), ("u16", (0, 3))])
def test_series_at_any_byte(dtype, offsets):
    import torch
    import paper_1807_06507_amd as swc
    x, y = random_pair((4099,), dtype, seed=offsets[0])
    dev = []
    for a, off in zip((x, y), offsets):
        flat = torch.empty(a.size + 8, dtype=to_dev(a).dtype, device="cuda")
        view = flat[off:off + a.size]
        view.copy_(to_dev(a))
        dev.append(view)
    for k, border in ((33, "clip"), (700, "fill"), (5, "valid")):
        say(f"[series at any byte] {dtype} {offsets} k={k} {border}")
        c, fl = swc.corr(dev[0], dev[1], k, 1, border, return_flags=True)
        torch.cuda.synchronize()
        o32, _, ofl = oracle.corr(x, y, (k,), 1, border)
        assert np.array_equal(fl.cpu().numpy(), ofl)
        assert np.array_equal(c.cpu().numpy().view(np.uint32), o32.view(np.uint32))


@pytest.mark.parametrize("k", [5, 300, 1001])
def test_rows_with_many_missing_values(k):
    """Missing values throughout (masked rows follow one another), one per
    row, and a clean stretch long enough to leave the masked form again."""
    x, y = random_pair((9000,), "f32", seed=k, kind="lognormal")
    x[100::511] = np.nan
    y[3000:3300:7] = -np.inf
    x[4000], x[5000:9000] = -999.0, np.abs(x[5000:9000])
    for border, step in (("clip", 1), ("fill", 1), ("clip", 5)):
        compare(x, y, (k,), step, border, tag="series missing")


@pytest.mark.parametrize("dtype", ["u16", "f32"])
def test_rows_taken_again(dtype):
    """Every output through the exact decision (integer) or the two-pass
    recomputation (float), and constant stretches, in rows of every form."""
    import paper_1807_06507_amd as swc
    x, y = random_pair((3000,), dtype, seed=12)
    x[700:1300] = 5
    y[2000:2050] = 7
    for k in (9, 100):
        compare(x, y, (k,), 1, "clip", tag="series constant")
        swc.set_debug(1)
        try:
            compare(x, y, (k,), 1, "clip", tag="series forced")
            compare(x, y, (k,), 4, "fill", tag="series forced")
        finally:
            swc.set_debug(0)
