"""Blocks of rows (3-D) against the oracle: integer input bit for bit, float
input within 2^-24, flags identical.

Output heights around the rows a block serves, y-windows at every limit (the
flat and the tall blocks of integer input, the last height a block holds, the
first that goes to the other kernel), widths around a wave's 64 columns, steps
along every axis, x offsets that are no multiple of a word, few and many
planes, and missing values that enter a block late or everywhere.
"""
import numpy as np
import pytest

from gpu_util import compare, say, to_dev
from workloads import random_pair
import oracle

pytestmark = pytest.mark.gpu

DT = ["u8", "u16", "f32"]


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("k", [3, 5, 7, 9])
def test_cubic_windows_around_block_edges(dtype, k):
    for shape, border in (((k, 3 * k + 1, 64), "clip"), ((k + 3, 25, 63), "fill"), ((12, 31, 59), "valid"),
                          ((2, 14, 130), "clip"), ((30, 1, 5), "clip"), ((9, 20, 121), "valid")):
        if border == "valid" and any(n < k for n in shape):
            continue
        x, y = random_pair(shape, dtype, seed=sum(shape) + k)
        compare(x, y, (k, k, k), 1, border, tag="blocks")
        compare(x, y, (k, k, k), 1, border, params=(4, 3, 4, 0, 2), tag="blocks, 3 planes a tile")


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("ky", [1, 2, 5, 6, 8, 10, 12, 13, 14, 15, 20, 21])
def test_window_heights(dtype, ky):
    for shape, window, step, border in (((6, 40, 70), (2, ky, 3), 1, "clip"),
                                        ((5, 33, 100), (3, ky, 9), (1, 2, 1), "fill"),
                                        ((7, 47, 66), (1, ky, 5), (3, 4, 2), "clip"),
                                        ((4, 30, 50), (4, ky, 7), (1, 50, 3), "valid")):
        x, y = random_pair(shape, dtype, seed=ky + shape[1])
        compare(x, y, window, step, border, tag="heights")


@pytest.mark.parametrize("k", [3, 7])
def test_missing_values_in_blocks(k):
    x, y = random_pair((25, 30, 130), "f32", seed=k, kind="lognormal")
    x[13, 9, 60] = -999.0
    y[14, 28, 129] = np.nan
    x[20] = np.where(np.arange(130) % 3 == 0, np.inf, x[20])
    for window, step in (((k, k, k), 1), ((2, 4, k), (2, 1, 1)), ((k, k, k), (1, 2, 3))):
        for border in ("clip", "fill"):
            compare(x, y, window, step, border, params=(4, 25, 2, 0, 2), tag="blocks missing")
    z = x.copy()
    z[3:5, 10:12, 20:90] = 0.0
    compare(z, y, (k, k, k), 1, "clip", missing_le=0.0, tag="blocks threshold 0")


@pytest.mark.parametrize("dtype", ["u8", "u16"])
def test_volume_at_any_byte_and_forced_decisions(dtype):
    import torch
    import paper_1807_06507_amd as swc
    x, y = random_pair((9, 17, 67), dtype, seed=3)
    dev = []
    for a, off in ((x, 1), (y, 3)):
        flat = torch.empty(a.size + 8, dtype=to_dev(a).dtype, device="cuda")
        view = flat[off:off + a.size].view(a.shape)
        view.copy_(to_dev(a))
        dev.append(view)
    o32, _, ofl = oracle.corr(x, y, (3, 5, 5), 1, "clip")
    for bits in (0, 1, 2):
        say(f"[any byte] {dtype} debug={bits}")
        swc.set_debug(bits)
        try:
            c, fl = swc.corr(dev[0], dev[1], (3, 5, 5), 1, "clip", return_flags=True)
            torch.cuda.synchronize()
        finally:
            swc.set_debug(0)
        assert np.array_equal(fl.cpu().numpy(), ofl)
        assert np.array_equal(c.cpu().numpy().view(np.uint32), o32.view(np.uint32))


def test_float_windows_recomputed_and_constant():
    """The two-pass recomputation of every window, and of constant ones."""
    import paper_1807_06507_amd as swc
    x, y = random_pair((8, 20, 70), "f32", seed=9)
    x[2:7, 5:15, 10:40] = 2.5
    for bits in (0, 1):
        swc.set_debug(bits)
        try:
            compare(x, y, (3, 3, 3), 1, "clip", tag="blocks constant")
            compare(x, y, (2, 3, 5), (1, 2, 1), "fill", tag="blocks constant")
        finally:
            swc.set_debug(0)


def test_rows_too_long_for_a_block():
    """Rows whose offsets over a block pass 2^30 go to the other kernel."""
    n = 21_000_000
    x, y = random_pair((1, 1, n), "u8", seed=1)
    idx = np.unique(np.concatenate([np.arange(300), np.arange(n - 300, n),
                                    np.random.default_rng(0).integers(0, n, 3000)]))
    compare(x, y, (1, 1, 9), 1, "clip", indices=idx, tag="long rows")
