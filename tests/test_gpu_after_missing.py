"""Rows after a missing value has left the window (float 2-D): windows the
estimate does not settle there, constant ones and ones of small variance at a
large mean, in the columns that held the missing value, above and below it and
in the same tile.  Tiles of many rows, marched both ways, single launches with
and without a flag map, forced recomputation and batches.  Against the oracle:
flags identical, correlations within the float32 rounding of the output (such
windows are recomputed by the two-pass formula)."""
import numpy as np
import pytest

import oracle
from gpu_util import F32_TOL, say, to_dev

pytestmark = pytest.mark.gpu

SHAPE = (200, 300)


def _pair(k, seed):
    rng = np.random.default_rng(seed)
    x = rng.lognormal(size=SHAPE).astype(np.float32)
    y = (rng.normal(size=SHAPE) - 0.6 * x).astype(np.float32)
    for r in (60, 150):                                   # one per tile of 100 rows
        x[r, 40] = y[r, 150] = x[r, 151] = y[r + 1, 290] = -999.0
        for sign in (-1, 1):
            # rows from the first whose windows are free of row r on
            rows = slice(*sorted((r + sign * (k + 2), r + sign * (k + 22))))
            x[rows, 30:60] = 3.25
            y[rows, 140:170] = -7.5
            x[rows, 270:] = 1e6 + rng.normal(size=(20, 30))
    return x, y


def _check(c, fl, x, y, k, border):
    _, o64, ofl = oracle.corr(x, y, (k, k), 1, border)
    if fl is not None:
        assert np.array_equal(fl, ofl)
    bad = ofl != 0
    assert (ofl & 2).any() and (ofl & 4).any() and (ofl & 8).any()
    assert np.all(c[bad] == np.float32(-2.0))
    assert float(np.max(np.abs(c[~bad].astype(np.float64) - o64[~bad]))) <= F32_TOL


@pytest.mark.parametrize("k", [3, 5, 7, 9, 15, 11])
@pytest.mark.parametrize("params", [(4, 256, 1), (4, 100, 2)])
@pytest.mark.parametrize("border", ["fill", "clip", "valid"])
@pytest.mark.parametrize("force", [0, 1])
def test_windows_after_a_missing_value(k, params, border, force):
    import paper_1807_06507_amd as swc
    x, y = _pair(k, k)
    say(f"[after missing] k={k} params={params} {border} force={force}")
    xd, yd = to_dev(x), to_dev(y)
    before = swc.get_debug()
    swc.set_debug(force)
    try:
        c, fl = swc.corr(xd, yd, (k, k), 1, border, return_flags=True, params=params)
        bare = swc.corr(xd, yd, (k, k), 1, border, params=params)
        c, fl, bare = c.cpu().numpy(), fl.cpu().numpy(), bare.cpu().numpy()
    finally:
        swc.set_debug(before)
    _check(c, fl, x, y, k, border)
    _check(bare, None, x, y, k, border)


@pytest.mark.parametrize("flags", [False, True])
def test_windows_after_a_missing_value_in_a_batch(flags):
    import paper_1807_06507_amd as swc
    cases = [(k, *_pair(k, 20 + k)) for k in (3, 5, 7, 9, 15)]
    say(f"[after missing] batch flags={flags}")
    plan = swc.BatchPlan([dict(x=to_dev(x), y=to_dev(y), window=(k, k)) for k, x, y in cases],
                         return_flags=flags, params=(4, 100, 1))
    out = [c.cpu().numpy() for c in plan.launch()]
    for (k, x, y), c, fl in zip(cases, out, plan.flags):
        _check(c, fl.cpu().numpy() if flags else None, x, y, k, "clip")
    plan.close()
