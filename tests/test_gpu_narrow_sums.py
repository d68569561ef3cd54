"""Float windows of every width at which the sums along the row change form
(2-D): the first ones inside one lane, sums of parts of two lanes with none, one
and more whole lanes between them, the prefix form from 31 columns on.  A large
mean (x ~ N(1000, 1)) makes rounding that comes from outside the window visible;
missing values and constant patches need the counts and the recomputation.
Against the oracle: flags identical, correlations within 2^-24."""
import numpy as np
import pytest

from gpu_util import compare
from workloads import random_pair

pytestmark = pytest.mark.gpu

WIDTHS = list(range(1, 18)) + [20, 23, 24, 25, 28, 29, 30, 31, 32, 33]


@pytest.mark.parametrize("kw", WIDTHS)
def test_large_mean(kw):
    for kh in (1, 2, 5):
        if kh * kw < 4:      # two or three cells: c is +-1 or close to it, the variance anything
            continue
        x, y = random_pair((90, 700), "f32", seed=10 * kw + kh, kind="offset", rho=0.7)
        compare(x, y, (kh, kw), 1, "clip", tag="large mean")
        compare(x, y, (kh, kw), 1, "clip", tag="large mean", params=(4, 40, 2))


@pytest.mark.parametrize("kw", WIDTHS)
@pytest.mark.parametrize("border", ["fill", "clip", "valid"])
def test_missing_and_constant(kw, border):
    rng = np.random.default_rng(kw)
    x, y = (rng.integers(1, 200, (75, 523)).astype(np.float32) for _ in range(2))
    x[20, 100] = y[20, 101] = x[21, 260] = y[50, 0] = x[50, -1] = -999.0
    x[52:55, 300:330] = np.nan
    x[25:40, 90:140] = 5.0
    y[5:16, 240:300] = 7.0
    for kh, step in ((3, 1), (4, (1, 2)), (2, (2, 3)), (1, 1)):
        for params in (None, (4, 64, 1)):
            compare(x, y, (kh, kw), step, border, tag="narrow sums", params=params)


@pytest.mark.parametrize("shape,window,step", [((150, 300), (33, 3), 1), ((150, 300), (40, 3), 2),
                                               ((90, 130), (100, 3), 1), ((1460, 1450), (14, 3), 1)])
def test_tall_windows_three_wide(shape, window, step):
    """Too tall for the LDS row ring, as a window or for the launch's size."""
    x, y = random_pair(shape, "f32", seed=shape[1], kind="offset", rho=0.7)
    x[70, 100] = y[60, 40] = np.nan
    x[75:89, 10:90] = 1000.0
    compare(x, y, window, step, "clip", tag="tall, three wide")
