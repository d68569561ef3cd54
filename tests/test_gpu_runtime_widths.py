"""The run-time width variant of the register 2-D kernel (every window width
without a compiled variant) and the shifted loads of integer rows that start
at any byte, against the oracle: integer input bit for bit, float input within
2^-24 (float32 rounding of the output is at most 2^-25; the FP64 sums add far
less on these inputs), flags identical.

Widths: below, at and above a lane's columns and the compiled ones, wider than
a tile's halo lanes can serve (249 is the last at four columns per lane), and
wider than the array.  Heights: taller than the LDS row ring of the compiled
widths.  Rows: every remainder modulo a lane's columns, array bases at every
byte a type allows.
"""
import numpy as np
import pytest

from gpu_util import F32_TOL, compare, say, to_dev
from workloads import random_pair
import oracle

pytestmark = pytest.mark.gpu

# (shape, window, step, border)
WIDTHS = [
    ((21, 300), (3, 1), 1, "clip"), ((20, 261), (4, 2), 1, "fill"), ((19, 257), (2, 10), 1, "valid"),
    ((40, 515), (5, 16), 1, "clip"), ((33, 700), (7, 17), (1, 3), "clip"),
    ((23, 129), (1, 64), 1, "clip"), ((30, 600), (3, 129), 1, "fill"), ((12, 300), (2, 249), 1, "clip"),
    ((12, 300), (2, 250), 1, "clip"), ((9, 40), (3, 63), 1, "clip"), ((1, 5), (1, 12), 1, "clip"),
    ((60, 333), (22, 18), 4, "valid"), ((150, 90), (100, 7), 1, "clip"), ((90, 270), (80, 15), (3, 1), "fill"),
]


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("shape,window,step,border", WIDTHS)
def test_width_without_a_compiled_variant(dtype, shape, window, step, border):
    if dtype == "u16" and window[0] * window[1] > 1448:
        pytest.skip("beyond the exact 16-bit window size")
    x, y = random_pair(shape, dtype, seed=sum(shape) + sum(window))
    if dtype == "f32":
        x[shape[0] // 2, shape[1] // 3] = -999.0      # one missing value
    compare(x, y, window, step, border, tag="run-time width")
    compare(x, y, window, step, border, params=(8, 5, 2), tag="run-time width, 8 columns a lane")


def _at_offset(a, cells):
    """`a` on the device, beginning `cells` elements into its allocation."""
    import torch
    flat = torch.empty(a.size + 16, dtype=to_dev(a).dtype, device="cuda")
    view = flat[cells:cells + a.size].view(a.shape)
    view.copy_(to_dev(a))
    return view


@pytest.mark.parametrize("dtype,offsets", [("u8", (0, 1)), ("u8", (3, 2)), ("u16", (0, 1)),
                                           ("u16", (1, 3)), ("u8", (4, 0))])
@pytest.mark.parametrize("width", [1, 3, 254, 255, 256, 257])
@pytest.mark.parametrize("window", [(7, 7), (3, 12), (15, 15)])
def test_integer_rows_at_any_byte(dtype, offsets, width, window):
    import torch
    import paper_1807_06507_amd as swc
    x, y = random_pair((31, width), dtype, seed=width + offsets[0])
    xd, yd = _at_offset(x, offsets[0]), _at_offset(y, offsets[1])
    for border in ("clip", "fill"):
        say(f"[any byte] {dtype} offsets={offsets} width={width} window={window} {border}")
        c, fl = swc.corr(xd, yd, window, 1, border, return_flags=True)
        plan = swc.BatchPlan([dict(x=xd, y=yd, window=window, border=border)], return_flags=True)
        cb = plan.launch()[0]
        torch.cuda.synchronize()
        o32, _, ofl = oracle.corr(x, y, window, 1, border)
        for cc, ff in ((c, fl), (cb, plan.flags[0])):
            assert np.array_equal(ff.cpu().numpy(), ofl)
            assert np.array_equal(cc.cpu().numpy().view(np.uint32), o32.view(np.uint32))
        plan.close()


def test_run_time_width_certifies_its_prefix_sums():
    """Prefix sums carry the rounding of every column of the wave: one large
    value left of a constant patch, outside every window of the patch."""
    import paper_1807_06507_amd as swc
    rng = np.random.default_rng(4)
    x = rng.normal(0, 1, (40, 250)).astype(np.float32)
    y = rng.normal(0, 1, (40, 250)).astype(np.float32)
    x[:, 120:200] = 3.0
    x[5, 4] = 1e6
    c, fl = swc.corr(to_dev(x), to_dev(y), (6, 12), border="clip", return_flags=True)
    _, o64, ofl = oracle.corr(x, y, (6, 12), 1, "clip")
    assert np.array_equal(fl.cpu().numpy(), ofl) and np.count_nonzero(ofl & 4) > 0
    ok = ofl == 0
    assert np.max(np.abs(c.cpu().numpy().astype(np.float64)[ok] - o64[ok])) <= F32_TOL
