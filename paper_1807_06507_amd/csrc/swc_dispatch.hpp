// Rules of the host side that choose tile sizes: plain arithmetic, no GPU call.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace swc {

// Output rows per tile of the register 2-D kernel when filling the resident
// wave slots once would take fewer than four.  Such a tile is mostly its
// window's first k_h rows.  That still pays while a SIMD has few waves: a lone
// wave takes about 1.2 us an output row and 0.6 us a halo row (float, 7x7), so
// 96x128 takes 7.6 us at one row and 11.5 at four, 399x574 in steps of 2 8.4 and
// 16.0.  With more waves a SIMD the halo rows' own work shows: 768x1024 8-bit at
// 3x3 takes 8.8 us at one row (more than three waves), 7.1 at two, 8.7 at four;
// 700x900 16-bit at 31x31, VALID, 27.5 us at one row (three waves), 22.7 at two
// (two waves), 20.2 at three (one), 21.5 at four.  So of the heights from the
// first at which three waves a SIMD hold all tiles up to eight it takes the one
// with the least product of rows marched (an output row counts for three) and
// what two and three waves on a SIMD cost each other (the SIMDs with one wave
// more than the others end the launch: 1804x1115 16-bit at 31x31 35.1 us at three
// rows, 2.9 waves a SIMD, 36.6 at four, 2.2 waves, 34.0 at five, 1.8 waves).  The
// weights were fitted to 600 launches of 3x3 to 31x31 windows on images up to
// 1255x2793; over 260 others of random sides, windows and steps the height taken
// is within 1.0% of the best on average, 20% at most.
// Float input takes the lowest height within a tenth of that: windows its
// estimate does not settle (flat areas) are recomputed cell by cell, which more
// waves share (407x2412 at 100x7, a quarter flat: 0.80 ms at two rows, 1.55 at
// four, where the product says 4% less).
// `first`: the lowest height whose tiles the wave slots hold; `third`: the cost
// of three waves on a SIMD (8-bit input 1.3, whose rows leave the vector units
// more idle, else 1.5).
inline int64_t low_tile_rows(int64_t OH, int64_t tiles_x, int kh, int sh, int64_t first, int64_t simds,
                             double third, bool recomputes)
{
    const int64_t ty3 = std::max<int64_t>(1, 3 * simds / std::max<int64_t>(1, tiles_x));
    const int64_t lo = std::min<int64_t>(4, std::max(first, (OH + ty3 - 1) / ty3));
    int64_t rows = lo;
    double best = 1e300;
    for (int64_t th = lo; th <= 8; th++) {
        const int64_t waves = (tiles_x * ((OH + th - 1) / th) + simds - 1) / simds;
        const double cost = ((double)(th - 1) * sh + kh + 2.0 * th) *
                            (waves <= 1 ? 1.0 : (waves <= 2 ? 1.1 : third));
        if (cost < best * (recomputes ? 1.0 / 1.1 : 1.0)) {
            best = cost;
            rows = th;
        }
    }
    return rows;
}

// Output planes per tile (3-D): rounds of `slots` concurrent tiles, each as long
// as its planes plus the planes that only warm its sums up (those cost `warm` of
// a finished one).  Tile counts that give the same planes are looked at once:
// two square roots of OD of them instead of OD (4096 planes: 1.8 us of host time
// a call instead of 25).
inline int tile_planes(int64_t tiles_xy, int OD, int kz, int sz, int64_t slots, double warm)
{
    int best = OD;
    double best_cost = 1e300;
    for (int tiles_z = 1; tiles_z <= OD && tiles_z <= 4096;) {
        const int TZ = (OD + tiles_z - 1) / tiles_z;
        const int64_t n = tiles_xy * ((OD + TZ - 1) / TZ);
        const double rounds = (double)((n + slots - 1) / slots);
        const double steps = (double)(TZ - 1) * sz + kz;
        const double cost = rounds * (TZ + warm * (steps - TZ) + 1.0);
        if (cost < best_cost * 0.999) {
            best_cost = cost;
            best = TZ;
        }
        if (TZ == 1) break;
        tiles_z = (OD + TZ - 2) / (TZ - 1);      // the first count with fewer planes
    }
    return best;
}

// One pair of a batch: output rows, tiles across, window height and row step.
struct BatchShape {
    int64_t OH, tiles_x;
    int kh, sh;
};

// Output rows per tile of a batch: one height for all pairs, by the rows marched.
// All tiles' rows are shared by the SIMDs, and a part of the largest tile's is
// for the waves that finish last.  Integer input: an output row counts for
// three, a tile's setup for twelve and the part is 0.3, fitted to 90 batches of 2
// to 60 pairs of sides 20 to 3000 at up to thirteen heights (the choice is
// within 3.1% of the best height on average and 17% at most; with the weights of
// float input 11% and 43%: nine 16-bit images up to 2000 px 66.5 us at 8 rows,
// 46.4 at 16; three up to 1960 px 73.8 at 16, 59.1 at 32).  Float input: an output
// row counts for one, the setup for three and the part is 0.75, which gives lower
// tiles: 6% from the best on average without flat areas, but windows in flat
// areas are recomputed cell by cell by the wave that owns them, and more tiles
// share them better (eleven images up to 2000 px, a quarter of half of them flat:
// 171 us, with the weights of integer input 268).
inline int batch_tile_rows(const std::vector<BatchShape>& pairs, int cus, bool recomputes)
{
    const double tail = recomputes ? 0.75 : 0.3;
    int rows = 32;
    double best = 1e300;
    for (int th : {2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128}) {
        if (recomputes && th < 4) continue;
        double all = 0.0, largest = 0.0;
        for (const BatchShape& b : pairs) {
            const double out = (double)std::min<int64_t>(th, b.OH);
            const double each = recomputes ? out * b.sh + b.kh + 3.0
                                           : (out - 1.0) * b.sh + b.kh + 2.0 * out + 12.0;
            all += (double)(b.tiles_x * ((b.OH + th - 1) / th)) * each;
            largest = std::max(largest, each);
        }
        const double cost = all / (cus * 4.0) + tail * largest;
        if (cost < best) {
            best = cost;
            rows = th;
        }
    }
    return rows;
}

// Waves of the 1-D kernel resident on a CU: `per_simd` by their registers, and
// as many workgroups of `wpb` waves as the CU's 160 KB of LDS holds rings for
// (k = 1001: twelve waves of 12.2 KB; k = 3000: four of 28.1 KB by twos).  Segments
// sized for more waves than that would run in a second round: 2^22 floats, k =
// 1448 35.1 -> 27.5 us, k = 3000 62.2 -> 37.4; k = 5000 (no ring, two waves a SIMD)
// 53.8 -> 42.1.
inline int series_waves(int per_simd, int64_t ring_bytes, int wpb)
{
    const int64_t by_lds = ring_bytes > 0 ? 160 * 1024 / (ring_bytes * wpb) * wpb : 4 * per_simd;
    return (int)std::max<int64_t>(1, std::min<int64_t>(4 * per_simd, by_lds));
}

}  // namespace swc
