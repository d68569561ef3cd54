"""The host rules that choose tile sizes (csrc/swc_dispatch.hpp), compiled by
themselves with the host compiler."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1807_06507_amd", "csrc")

SOURCE = r"""
#include "swc_dispatch.hpp"
extern "C" {
int64_t low_tile_rows(int64_t OH, int64_t tx, int kh, int sh, int64_t first, int64_t simds)
{ return swc::low_tile_rows(OH, tx, kh, sh, first, simds); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC,
                    str(d / "rules.cpp"), "-o", str(d / "rules.so")], check=True)
    lib = ctypes.CDLL(str(d / "rules.so"))
    lib.low_tile_rows.restype = ctypes.c_int64
    lib.low_tile_rows.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int,
                                  ctypes.c_int64, ctypes.c_int64]
    return lib


@pytest.mark.parametrize("OH,tiles_x,kh,sh,first,rows", [
    (670, 4, 31, 1, 1, 3),       # 700x900 at 31x31, VALID: three waves a SIMD at one row
    (994, 5, 31, 1, 2, 3),       # 1024x1024 at 31x31, VALID: 29.4, 23.8, 26.3 us at two, three, four
    (96, 1, 7, 1, 1, 1),         # few tiles: every row a tile
    (200, 3, 7, 2, 1, 1),        # 399x574 in steps of 2
    (768, 5, 3, 1, 1, 2),        # 768x1024 at 3x3: more than three waves at one row
    (4, 1, 200, 1, 1, 1), (1, 1, 3, 1, 1, 1), (3000, 17, 7, 1, 3, 4),
])
def test_low_tiles(rules, OH, tiles_x, kh, sh, first, rows):
    assert rules.low_tile_rows(OH, tiles_x, kh, sh, first, 1024) == rows
