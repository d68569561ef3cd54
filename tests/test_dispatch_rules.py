"""The host rules that choose tile sizes (csrc/swc_dispatch.hpp), compiled by
themselves with the host compiler."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1807_06507_amd", "csrc")

SOURCE = r"""
#include <chrono>
#include "swc_dispatch.hpp"
extern "C" {
int64_t low_tile_rows(int64_t OH, int64_t tx, int kh, int sh, int64_t first, int64_t simds,
                      double third, bool f)
{ return swc::low_tile_rows(OH, tx, kh, sh, first, simds, third, f); }
int tile_planes(int64_t txy, int OD, int kz, int sz, int64_t slots, double warm)
{ return swc::tile_planes(txy, OD, kz, sz, slots, warm); }
int batch_tile_rows(int n, const int64_t* v, int cus, bool f)
{
    std::vector<swc::BatchShape> b;
    for (int i = 0; i < n; i++)
        b.push_back(swc::BatchShape{v[4 * i], v[4 * i + 1], (int)v[4 * i + 2], (int)v[4 * i + 3]});
    return swc::batch_tile_rows(b, cus, f);
}
int series_waves(int per_simd, int64_t ring, int wpb) { return swc::series_waves(per_simd, ring, wpb); }
double tile_planes_us(int OD)
{
    double best = 1e9;
    long long sum = 0;
    for (int i = 0; i < 20; i++) {
        const auto t0 = std::chrono::steady_clock::now();
        for (int j = 0; j < 50; j++) sum += swc::tile_planes(3 + j, OD, 7, 1, 2048, 0.35);
        const std::chrono::duration<double, std::micro> t = std::chrono::steady_clock::now() - t0;
        if (t.count() / 50 < best) best = t.count() / 50;
    }
    return sum > 0 ? best : 1e9;
}
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
                                  ctypes.c_int64, ctypes.c_int64, ctypes.c_double, ctypes.c_bool]
    lib.tile_planes.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int,
                                ctypes.c_int64, ctypes.c_double]
    lib.series_waves.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int]
    lib.batch_tile_rows.argtypes = [ctypes.c_int, ctypes.POINTER(ctypes.c_int64), ctypes.c_int,
                                    ctypes.c_bool]
    lib.tile_planes_us.restype = ctypes.c_double
    return lib


@pytest.mark.parametrize("OH,tiles_x,kh,sh,first,rows", [
    (670, 4, 31, 1, 1, 3),       # 700x900 at 31x31, VALID: three waves a SIMD at one row
    (994, 5, 31, 1, 2, 3),       # 1024x1024 at 31x31, VALID: 29.4, 23.8, 26.3 us at two, three, four
    (1804, 5, 31, 1, 3, 5),      # 1804x1115 at 31x31: 35.1, 36.6, 34.0, 35.8 us at three to six
    (96, 1, 7, 1, 1, 1),         # few tiles: every row a tile
    (200, 3, 7, 2, 1, 1),        # 399x574 in steps of 2
    (768, 5, 3, 1, 1, 2),        # 768x1024 at 3x3: more than three waves at one row
    (4, 1, 200, 1, 1, 1), (1, 1, 3, 1, 1, 1), (3000, 17, 7, 1, 3, 4),
])
def test_low_tiles(rules, OH, tiles_x, kh, sh, first, rows):
    assert rules.low_tile_rows(OH, tiles_x, kh, sh, first, 1024, 1.5, False) == rows


@pytest.mark.parametrize("OH,tiles_x,kh,first,rows", [
    (407, 10, 100, 2, 2),        # 407x2412 at 100x7: a tenth is not worth half the waves
    (96, 1, 7, 1, 1), (768, 5, 31, 2, 2), (670, 4, 31, 2, 2), (1000, 4, 31, 2, 2),
])
def test_low_tiles_of_float_input(rules, OH, tiles_x, kh, first, rows):
    assert rules.low_tile_rows(OH, tiles_x, kh, 1, first, 1024, 1.5, True) == rows


def _every_tile_count(tiles_xy, OD, kz, sz, slots, warm):
    best, best_cost = OD, 1e300
    for tiles_z in range(1, min(OD, 4096) + 1):
        TZ = -(-OD // tiles_z)
        rounds = -(-tiles_xy * -(-OD // TZ) // slots)
        cost = float(rounds) * (TZ + warm * ((TZ - 1.0) * sz + kz - TZ) + 1.0)
        if cost < best_cost * 0.999:
            best, best_cost = TZ, cost
    return best


def test_planes_per_tile_as_from_every_tile_count(rules):
    rng = random.Random(1)
    for i in range(300):
        OD = int(10 ** rng.uniform(0, 3.9))
        args = (int(10 ** rng.uniform(0, 5)), OD, rng.randint(1, 40), rng.choice([1, 1, 2, 5]),
                rng.choice([2048, 3072]), rng.choice([0.35, 1.0]))
        assert rules.tile_planes(*args) == _every_tile_count(*args), args


def test_planes_per_tile_cost_little_in_deep_volumes(rules):
    """A launch takes a few microseconds of host time in all; looking at 4096
    tile counts one by one took 25 of its own."""
    assert rules.tile_planes_us(4096) < 8.0


def test_which_windows_the_register_kernel_takes(tmp_path):
    """Windows of 2^31 cells (float input alone allows them) pass the 32-bit cell
    counts of the register kernel and stay on the generic one."""
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("no hipcc")
    (tmp_path / "taken.hip").write_text("""
#include "swc_corr2d_fast.hpp"
using namespace swc;
constexpr bool taken(int mode, int kh, int kw)
{
    return fast2d_supported(mode, 4, kh, kw, fast2d_variant(mode, 4, kh, kw, 1));
}
static_assert(taken(MODE_F64, 7, 7) && taken(MODE_F64, 13, 21) && taken(MODE_F64, 1, 1), "");
static_assert(taken(MODE_F64, 1 << 24, 127) && !taken(MODE_F64, 1 << 24, 128), "");
static_assert(!taken(MODE_F64, 10737419, 200) && taken(MODE_F64, 10737418, 200), "");
static_assert(taken(MODE_U8, 150, 220) && taken(MODE_U16, 6, 240) && !taken(MODE_F64, 2, 250), "");
""")
    inc = os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include")
    subprocess.run([hipcc, "-std=c++17", "-x", "hip", "--cuda-host-only", "-fsyntax-only", "-I" + CSRC,
                    "-I" + inc, str(tmp_path / "taken.hip")], check=True)


def test_rings_of_tall_windows_by_outputs(tmp_path):
    """Compiled widths keep rings past 24 KB per wave up to 2^22 outputs of
    integer input and 2^21 of float (then 0: the run-time variant), 64 KB at most."""
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("no hipcc")
    (tmp_path / "rings.hip").write_text("""
#include "swc_corr2d_fast.hpp"
using namespace swc;
constexpr int64_t M = 1 << 20;
constexpr int width(int mode, int kh, int kw, int64_t outputs) { return fast2d_variant(mode, 4, kh, kw, outputs); }
static_assert(width(MODE_U8, 100, 7, 2 * M + 1) == 7 && width(MODE_U16, 60, 3, 2 * M + 1) == 3, "");
static_assert(width(MODE_U8, 100, 7, 4 * M) == 7 && width(MODE_U16, 60, 3, 4 * M) == 3, "");
static_assert(width(MODE_U8, 100, 7, 4 * M + 1) == 0 && width(MODE_U16, 60, 3, 4 * M + 1) == 0, "");
static_assert(width(MODE_U8, 40, 7, 16 * M) == 7 && width(MODE_U16, 20, 3, 16 * M) == 3, "");
static_assert(width(MODE_F64, 30, 5, 2 * M) == 5 && width(MODE_F64, 30, 5, 2 * M + 1) == 0, "");
static_assert(width(MODE_U8, 140, 3, 1) == 0 && width(MODE_U16, 70, 3, 1) == 0, "");
""")
    inc = os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include")
    subprocess.run([hipcc, "-std=c++17", "-x", "hip", "--cuda-host-only", "-fsyntax-only", "-I" + CSRC,
                    "-I" + inc, str(tmp_path / "rings.hip")], check=True)


@pytest.mark.parametrize("per_simd,ring,wpb,waves", [
    (3, 0, 4, 12), (2, 0, 2, 8), (3, 12160, 4, 12), (3, 13632, 4, 12), (3, 13696, 4, 8),
    (3, 28160, 2, 4), (3, 28160, 1, 5), (2, 8128, 4, 8), (3, 32768, 2, 4),
])
def test_resident_waves_of_a_series(rules, per_simd, ring, wpb, waves):
    """By registers (12 or 8 a CU) and by the LDS rings of whole workgroups."""
    assert rules.series_waves(per_simd, ring, wpb) == waves


# batches as measured (sides, window, step) and their times in us by tile height:
# three of integer input, where the heights for float input take 22% to 43% more
# than the best one, and a float one
BATCHES = [
    (False, [((599, 142), (9, 9), 1), ((357, 42), (9, 9), 2), ((99, 1572), (4, 5), 1),
             ((170, 44), (5, 9), 2), ((36, 47), (17, 3), 1), ((261, 100), (5, 5), 2),
             ((573, 960), (3, 3), 1), ((1294, 1274), (6, 5), 1), ((36, 1235), (5, 5), 1)],
     {2: 125.0, 3: 104.0, 4: 92.6, 6: 80.8, 8: 66.4, 12: 51.3, 16: 46.4, 24: 48.0, 32: 58.6,
      48: 78.5, 64: 99.8}),
    (False, [((707, 1841), (5, 5), 1), ((437, 590), (7, 7), 2), ((1693, 62), (7, 7), 1),
             ((717, 174), (7, 7), 1), ((1710, 479), (7, 7), 2), ((341, 741), (5, 5), 1),
             ((118, 238), (7, 7), 1), ((159, 438), (7, 7), 1), ((1333, 29), (5, 5), 1)],
     {2: 129.5, 3: 106.8, 4: 93.2, 6: 83.5, 8: 67.6, 12: 51.9, 16: 48.7, 24: 49.9, 32: 61.1,
      48: 81.8, 64: 102.7}),
    (False, [((1225, 1709), (9, 9), 1), ((744, 1693), (5, 5), 1), ((1960, 1488), (5, 5), 1)],
     {2: 201.3, 3: 153.7, 4: 130.4, 6: 108.2, 8: 96.0, 12: 89.1, 16: 73.8, 24: 69.0, 32: 59.1,
      48: 71.6, 64: 88.3, 96: 123.6, 128: 159.8}),
    (True, [((806, 2587), (5, 5), 1), ((1300, 738), (15, 15), 1), ((2097, 2190), (15, 15), 1),
            ((1115, 640), (15, 15), 1), ((372, 3915), (15, 15), 1), ((2028, 2744), (5, 5), 1),
            ((2080, 1346), (7, 7), 1), ((2677, 674), (9, 9), 1), ((381, 347), (5, 5), 1),
            ((2916, 2473), (5, 5), 1), ((1817, 3067), (7, 7), 1), ((1984, 3229), (5, 5), 1),
            ((2417, 1164), (15, 15), 1), ((2286, 2520), (7, 7), 1), ((1671, 1201), (7, 7), 1),
            ((2138, 1442), (5, 5), 1)],
     {2: 1414.5, 4: 759.4, 8: 434.5, 12: 341.9, 16: 292.6, 24: 264.5, 32: 247.7, 48: 238.2,
      64: 238.4, 96: 261.6, 128: 312.7}),
]


@pytest.mark.parametrize("recomputes,pairs,times", BATCHES)
def test_batch_tile_height(rules, recomputes, pairs, times):
    """Within a fifth of the best height measured."""
    flat = []
    for (h, w), (kh, kw), s in pairs:
        lanes = -(-max(kw // 2, kw - 1 - kw // 2) // 4)
        wq = (64 - 2 * lanes) * 4 if s == 1 else (253 - kw) // s + 1
        flat += [-(-h // s), -(-(-(-w // s)) // wq), kh, s]
    rows = rules.batch_tile_rows(len(pairs), (ctypes.c_int64 * len(flat))(*flat), 256, recomputes)
    assert times[rows] <= 1.2 * min(times.values()), rows
    if not recomputes:
        other = rules.batch_tile_rows(len(pairs), (ctypes.c_int64 * len(flat))(*flat), 256, True)
        assert times[other] > 1.2 * min(times.values()), other
