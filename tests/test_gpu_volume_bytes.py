"""Volumes whose cells lie at any byte (callers of the C entry point may pass such
pointers): two output rows per wave, no blocks of rows.  Against the oracle:
integer input bit for bit, float input within 2^-24, flags identical."""
import ctypes

import numpy as np
import pytest

import oracle
from gpu_util import F32_TOL, say, to_dev
from workloads import random_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,offsets", [("u16", (1, 0)), ("u16", (1, 3)), ("f32", (2, 0)),
                                           ("f32", (1, 3)), ("f32", (4, 2))])
@pytest.mark.parametrize("border", ["clip", "fill"])
def test_cells_at_any_byte(dtype, offsets, border):
    import torch
    import paper_1807_06507_amd as swc
    shape, window = (9, 21, 75), (3, 5, 7)
    x, y = random_pair(shape, dtype, seed=sum(offsets))
    say(f"[volume bytes] {dtype} offsets={offsets} {border}")
    at = []
    for a, off in zip((x, y), offsets):
        raw = to_dev(np.ascontiguousarray(a).view(np.uint8).ravel())
        room = torch.zeros(raw.numel() + 16, dtype=torch.uint8, device="cuda")
        room[off:off + raw.numel()] = raw
        at.append(room)
    p = swc.make_problem(shape, {"u16": "uint16", "f32": "float32"}[dtype], window, 1, border)
    c = torch.full(shape, 9.0, device="cuda")
    fl = torch.full(shape, 77, dtype=torch.uint8, device="cuda")
    code = swc._load().swc_corr_ex(ctypes.byref(p), None, at[0].data_ptr() + offsets[0],
                                   at[1].data_ptr() + offsets[1], c.data_ptr(), fl.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream)
    assert code == 0
    c, fl = c.cpu().numpy(), fl.cpu().numpy()
    o32, o64, ofl = oracle.corr(x, y, window, 1, border)
    assert np.array_equal(fl, ofl)
    ok = ofl == 0
    assert np.all(c[~ok] == np.float32(-2.0))
    if dtype == "u16":
        assert np.array_equal(c[ok], o32[ok])
    else:
        assert float(np.max(np.abs(c[ok].astype(np.float64) - o64[ok]))) <= F32_TOL
