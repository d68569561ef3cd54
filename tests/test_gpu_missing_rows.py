"""The float 2-D kernel screens whole rows for missing values: values that only
the screen's sum of products catches (NaN, infinities), finite values whose
products overflow it, thresholds above the zeros read outside the array, and
rows that enter and leave the window with one, several and no missing value.
Against the oracle: flags identical, correlations within the float32 rounding
of the output (integer-valued input)."""
import numpy as np
import pytest

from gpu_util import compare

pytestmark = pytest.mark.gpu


def _pair(shape, seed):
    rng = np.random.default_rng(seed)
    return [rng.integers(1, 200, shape).astype(np.float32) for _ in range(2)]


@pytest.mark.parametrize("window,step", [(3, 1), (7, 1), (15, 1), ((5, 11), 1), ((9, 4), 2), ((40, 7), 1)])
@pytest.mark.parametrize("border", ["fill", "clip", "valid"])
@pytest.mark.parametrize("value", [-999.0, -np.inf, np.inf, np.nan])
def test_missing_values_by_row(window, step, border, value):
    x, y = _pair((130, 530), 5)
    x[0, 0] = x[41, 200] = y[41, 203] = y[42, 200] = x[-1, -1] = value
    x[70, ::37] = value
    compare(x, y, window, step, border, tag="missing rows")


@pytest.mark.parametrize("window", [7, 15, 11])
@pytest.mark.parametrize("missing_le", [0.0, 3.0, -np.inf, 1e38])
def test_thresholds(window, missing_le):
    x, y = _pair((60, 300), 6)
    compare(x, y, window, 1, "clip", tag="threshold", missing_le=missing_le)


@pytest.mark.parametrize("window", [7, 15, 11])
def test_products_that_overflow_the_screen(window):
    x, y = _pair((60, 300), 7)
    x[20:24, 100:104] *= 2.0 ** 65                 # finite; x*y overflows float32
    y[20:24, 100:104] *= 2.0 ** 65
    x[40, 50] = -999.0
    compare(x, y, window, 1, "clip", tag="overflow")
