"""Images small enough for tiles of one to three output rows (2-D, the launch's
own tile height): against the oracle, integer input bit for bit, float input
within the float32 rounding of the output, flags identical.  Shapes: one row,
fewer rows than the window, heights that leave a short last tile, and one large
enough for two or three rows a tile."""
import pytest

from gpu_util import compare
from workloads import random_pair

pytestmark = pytest.mark.gpu

CASES = [((1, 40), 7, 1, "clip"), ((4, 300), (9, 5), 1, "fill"), ((96, 128), 7, 1, "fill"),
         ((97, 513), (5, 11), 2, "clip"), ((130, 700), 15, (3, 1), "valid"), ((643, 1201), 5, 1, "clip"),
         ((1500, 61), 3, 1, "clip")]


@pytest.mark.parametrize("dtype", ["u8", "u16", "f32"])
@pytest.mark.parametrize("shape,window,step,border", CASES)
def test_low_tiles(dtype, shape, window, step, border):
    x, y = random_pair(shape, dtype, seed=sum(shape))
    if dtype == "f32":
        x[shape[0] // 2, shape[1] // 3] = -999.0
    compare(x, y, window, step, border, tag="low tiles")
