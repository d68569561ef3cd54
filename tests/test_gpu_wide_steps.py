"""Column steps wider than half the window (2-D): most of a lane's columns are
no window's centre, and windows at the array's edges are clipped next to them.
Against the oracle: integer input bit for bit, float input within the float32
rounding of the output, flags identical."""
import pytest

from gpu_util import compare
from workloads import random_pair

pytestmark = pytest.mark.gpu

CASES = [((50, 300), 3, 3, "clip"), ((50, 300), 3, 3, "fill"), ((30, 257), 3, 4, "clip"),
         ((40, 300), 7, 5, "clip"), ((40, 300), (3, 1), 2, "clip"), ((40, 301), (4, 2), (1, 4), "fill"),
         ((40, 301), (5, 3), (1, 7), "clip"), ((40, 301), (5, 15), (1, 20), "valid")]


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("params", [None, (8, 8, 1)])
@pytest.mark.parametrize("shape,window,step,border", CASES)
def test_steps_wider_than_half_the_window(dtype, params, shape, window, step, border):
    x, y = random_pair(shape, dtype, seed=3)
    if dtype == "f32":
        x[20, 150] = x[0, 0] = x[3, -1] = -999.0
    compare(x, y, window, step, border, tag="wide step", params=params)
