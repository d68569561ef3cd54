"""make_problem packs the descriptor in one copy: every field against the same
descriptor filled field by field, also where a value does not fit its field."""
import itertools

import pytest

import paper_1807_06507_amd as swc


def _by_fields(shape, dtype, window, step, border, accum, invalid, missing_le):
    p = swc.Problem()
    p.ndim = len(shape)
    p.dtype = {"uint8": 0, "uint16": 1, "float32": 2}[dtype]
    p.border, p.accum = swc.BORDERS[border], swc.ACCUMS[accum]
    for d in range(3):
        inside = d < len(shape)
        p.shape[d] = shape[d] if inside else 1
        p.window[d] = (window if isinstance(window, int) else window[d]) if inside else 1
        p.step[d] = (step if isinstance(step, int) else step[d]) if inside else 1
    p.invalid_value, p.missing_le = invalid, missing_le
    return p


@pytest.mark.parametrize("shape", [(5,), (3, 2 ** 40), (2, 3, 4)])
def test_packed_descriptor_equals_the_fields(shape):
    for dtype, border, accum, inv, miss in itertools.product(
            ("uint8", "uint16", "float32"), ("fill", "clip", "valid"), ("default", "naive", "comp"),
            (-2.0, 0.1, 1e39, float("nan")), (-999.0, float("-inf"))):
        for window, step in ((7, 1), (tuple(range(3, 3 + len(shape))), [2] * len(shape)),
                             (2 ** 32 + 7, -1), (True, 2 ** 31)):
            got = swc.make_problem(shape, dtype, window, step, border, accum, inv, miss)
            want = _by_fields(shape, dtype, window, step, border, accum, inv, miss)
            assert bytes(got) == bytes(want)


@pytest.mark.parametrize("bad", [dict(shape=()), dict(shape=(1, 2, 3, 4)), dict(window=(3, 3, 3)),
                                 dict(step=[1]), dict(border="wrap"), dict(accum="half"),
                                 dict(dtype="int32")])
def test_refused_descriptors(bad):
    args = dict(shape=(5, 6), dtype="uint8", window=3, step=1, border="fill", accum="default")
    args.update(bad)
    with pytest.raises(ValueError):
        swc.make_problem(**args)
