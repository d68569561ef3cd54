// Host side of the fused 3-D kernels (swc_corr3d.hpp): geometry, launch
// configuration checks and dispatch to the per-mode instantiations.
#include <algorithm>

#include "swc_corr3d.hpp"
#include "swc_dispatch.hpp"
#include "swc_internal.h"

namespace swc {

// Output columns of a wave of `cols` input columns, `skip` of them lost to
// alignment.
static int wq3_of(int cols, int skip, int kw, int sx)
{
    const int span = cols - skip;
    return span < kw ? 0 : (span - kw) / sx + 1;
}

bool cfg_ok_3d(const swc_problem& p, const LaunchCfg& L)
{
    const int mode = mode_of(p.dtype, p.accum);
    if (!fast3d_supported(mode, p.window[2])) return false;
    if (L.R != 4) return false;
    if (!(L.wpb == 1 || L.wpb == 2 || L.wpb == 4)) return false;
    if (L.TH < 0 || L.TH > 4096) return false;   // 0: chosen per launch
    if (!(L.TY == 2 || L.TY == 4)) return false;
    for (int d = 0; d < 3; d++)
        if (p.shape[d] >= ((int64_t)1 << 30)) return false;
    // rows are addressed as raw buffers of at most 2^31 - 1 bytes
    if (p.shape[2] * 4 >= ((int64_t)1 << 31) - 64) return false;
    return wq3_of(kWave * 4, 3, p.window[2], p.step[2]) >= 1;
}

hipError_t launch_corr3d(const swc_problem& p, const int64_t* oshape, const LaunchCfg& L,
                         const void* x, const void* y, float* c, uint8_t* flags,
                         hipStream_t s, int force)
{
    const int mode = mode_of(p.dtype, p.accum);
    P3D g;
    g.x = x;
    g.y = y;
    g.c = c;
    g.flags = flags;
    g.D = (int)p.shape[0];
    g.H = (int)p.shape[1];
    g.W = (int)p.shape[2];
    g.OD = (int)oshape[0];
    g.OH = (int)oshape[1];
    g.OW = (int)oshape[2];
    g.kz = p.window[0];
    g.ky = p.window[1];
    g.sz = p.step[0];
    g.sy = p.step[1];
    g.sx = p.step[2];
    g.oz = window_offset(p.border, p.window[0]);
    g.oy = window_offset(p.border, p.window[1]);
    g.ox = window_offset(p.border, p.window[2]);
    g.border = p.border;
    g.invalid = p.invalid_value;
    g.miss_thr = missing_threshold(p.missing_le);
    g.force = force;
    const int kw = p.window[2];
    const size_t esz = p.dtype == SWC_U8 ? 1 : (p.dtype == SWC_U16 ? 2 : 4);
    const double n = (double)g.kz * g.ky * kw;
    const double nterms = (double)(g.kz + 1) * (g.ky + 1) * (kw + 1);
    // blocks of rows, when the y-window fits one, its rows can be addressed with
    // 30-bit offsets and cells lie at multiples of their size (the buffer loads
    // of the block kernel; the other one takes any byte)
    const int NR = block3_rows(mode, g.ky);
    const bool whole = (uintptr_t)x % esz == 0 && (uintptr_t)y % esz == 0 && (uintptr_t)c % 4 == 0;
    if (whole && g.ky <= NR && (int64_t)(NR + 1) * g.W * 4 < ((int64_t)1 << 30)) {
        g.NO = (NR - g.ky) / g.sy + 1;
        g.Wq = wq3_of(kWave, 0, kw, g.sx);
        g.tiles_x = (g.OW + g.Wq - 1) / g.Wq;
        g.tiles_y = (g.OH + g.NO - 1) / g.NO;
        const int64_t tiles_xy = (int64_t)g.tiles_x * g.tiles_y;
        // a plane that only warms the sums up costs about a third of a
        // finished one
        g.TZ = L.TH > 0 ? L.TH : tile_planes(tiles_xy, g.OD, g.kz, g.sz,
                                             (int64_t)device_cus() * 4 * block3_waves(mode, NR), 0.35);
        g.tiles_z = (g.OD + g.TZ - 1) / g.TZ;
        const int64_t nt = tiles_xy * g.tiles_z;
        if (nt >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
        g.n_tiles = (int)nt;
        // certification: chain = z-march steps (two operations each), then the
        // walk down the rows and the sums along x
        const double nzs = (double)(g.TZ - 1) * g.sz + g.kz;
        g.cert_g = cert_factor(mode, n, 2.0 * nzs + 2.0 * NR + kw + 16.0, nterms);
        const int wpb = L.wpb;
        const int grid = (int)((nt + wpb - 1) / wpb);
        if (mode == MODE_U8) return launch_fast3d_modeu8(g, kw, true, false, grid, wpb, s);
        if (mode == MODE_U16) return launch_fast3d_modeu16(g, kw, true, false, grid, wpb, s);
        return launch_fast3d_modef64(g, kw, true, false, grid, wpb, s);
    }

    // one wave per tile of two output rows
    constexpr int kTY = 2;
    g.NO = kTY;
    g.Wq = wq3_of(kWave * 4, 3, kw, g.sx);
    g.tiles_x = (g.OW + g.Wq - 1) / g.Wq;
    g.tiles_y = (g.OH + kTY - 1) / kTY;
    g.TZ = L.TH > 0 ? L.TH
                    : tile_planes((int64_t)g.tiles_x * g.tiles_y, g.OD, g.kz, g.sz,
                                  (int64_t)device_cus() * 4 * 2, 1.0);
    g.tiles_z = (g.OD + g.TZ - 1) / g.TZ;
    const int64_t nt = (int64_t)g.tiles_x * g.tiles_y * g.tiles_z;
    if (nt >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    g.n_tiles = (int)nt;
    // certification: chain = z-march steps plus the per-step y and x sums
    const double nzs = (double)(g.TZ - 1) * g.sz + g.kz;
    const double chain = 2.0 * nzs + 2.0 * ((kTY - 1) * g.sy + g.ky) + kw + 16.0;
    g.cert_g = cert_factor(mode, n, chain, nterms);
    const bool vec = ((uintptr_t)x % (esz * 4) == 0) && ((uintptr_t)y % (esz * 4) == 0) &&
                     (g.W % 4 == 0);
    // waves per workgroup: halved while the LDS running sums would exceed 64 KB
    const int lds_wave = tile3d_lds_bytes(mode, kTY, 4);
    int wpb = L.wpb;
    while (wpb > 1 && (int64_t)wpb * lds_wave > 64 * 1024) wpb /= 2;
    const int grid = (int)(((int64_t)g.n_tiles + wpb - 1) / wpb);
    if (mode == MODE_U8) return launch_fast3d_modeu8(g, kw, false, vec, grid, wpb, s);
    if (mode == MODE_U16) return launch_fast3d_modeu16(g, kw, false, vec, grid, wpb, s);
    return launch_fast3d_modef64(g, kw, false, vec, grid, wpb, s);
}

}  // namespace swc
