// Fused 3-D sliding-window correlation (Poyda & Zhizhin, arXiv 1807.06507:
// Section 1 steps 1-4 with the summation repeated once per dimension, as the
// n-dimensional remark of Section 1 describes).
//
// Two kernels.  corr3d_block_kernel keeps a block of rows per wave (below);
// corr3d_kernel, two output rows per wave, serves what that
// one does not hold: windows taller than a block's rows and rows too long for
// 32-bit offsets over a block.  In the latter one wave owns a tile of TZ output
// planes x TY output rows x Wq output columns (lanes own R adjacent columns,
// as in the 2-D kernel) and marches along z: per step it forms, for the TY
// rows' window rows, the element difference of the five channel contributions
// between the plane entering the z-window and the plane leaving it; sums
// those differences over each output row's y-window in registers; takes the
// x-window through the DPP halo exchange of the 2-D kernel; and adds the
// result to running 3-D sums kept in LDS.  Output planes are finished
// (epilogue + store) as soon as their z-window is complete.  Tiles are
// numbered with y fastest, so the tiles that share a y-halo run at the same
// time and march z in step (their shared rows hit the same L2).
#pragma once

#include <stddef.h>
#include <type_traits>

#include "swc_corr2d_fast.hpp"

namespace swc {

struct P3D {
    const void* x;
    const void* y;
    float* c;
    uint8_t* flags;
    int D, H, W, OD, OH, OW;
    int kz, ky, sz, sy, sx, oz, oy, ox;
    int border;
    float invalid;
    float miss_thr;
    int force;
    double cert_g;
    int TZ, Wq, tiles_x, tiles_y, tiles_z, n_tiles;
    int NO;                    // output rows per block of rows
};

__host__ __device__ inline bool fast3d_supported(int mode, int KW)
{
    if (mode != MODE_U8 && mode != MODE_U16 && mode != MODE_F64) return false;
    return KW == 3 || KW == 5 || KW == 7 || KW == 9;
}

// Blocks of rows (corr3d_block_kernel), or `block` false: two output rows per
// wave (corr3d_kernel, `vec` loads of whole aligned runs).
hipError_t launch_fast3d_modeu8(const P3D& g, int KW, bool block, bool vec, int grid, int wpb,
                                hipStream_t s);
hipError_t launch_fast3d_modeu16(const P3D& g, int KW, bool block, bool vec, int grid, int wpb,
                                 hipStream_t s);
hipError_t launch_fast3d_modef64(const P3D& g, int KW, bool block, bool vec, int grid, int wpb,
                                 hipStream_t s);

// Contribution difference (entering minus leaving) of one element pair, in
// the running-sum representation of Col<M> (integer modes keep 2*Sxy).
template <int M, class T>
__device__ __forceinline__ Col<M> col_delta(T a, T b, T ao, T bo, int m, int mo)
{
    Col<M> d;
    if constexpr (col_is_f64(M)) {
        const double x = (double)a, y = (double)b, xo = (double)ao, yo = (double)bo;
        d.x = x - xo;
        d.y = y - yo;
        d.xx = __builtin_fma(x, x, -(xo * xo));
        d.yy = __builtin_fma(y, y, -(yo * yo));
        d.xy = __builtin_fma(x, y, -(xo * yo));
        d.miss = m - mo;
    } else {
        col_zero<M>(d);
        col_update_int<M>(d, (int)a, (int)b, (int)ao, (int)bo);
    }
    return d;
}

// a += col_delta(a, b, ao, bo) without forming the difference first: the
// product channels take the entering and leaving products as two FMAs into
// the sum (two roundings, as the difference and its addition have).
template <int M, class T>
__device__ __forceinline__ void col_accum_delta(Col<M>& s, T a, T b, T ao, T bo)
{
    if constexpr (M == MODE_F64) {
        const double x = (double)a, y = (double)b, xo = (double)ao, yo = (double)bo;
        s.x += x - xo;
        s.y += y - yo;
        s.xx = __builtin_fma(x, x, __builtin_fma(-xo, xo, s.xx));
        s.yy = __builtin_fma(y, y, __builtin_fma(-yo, yo, s.yy));
        s.xy = __builtin_fma(x, y, __builtin_fma(-xo, yo, s.xy));
    } else {
        col_update_int<M>(s, (int)a, (int)b, (int)ao, (int)bo);
    }
}

// The sums the general kernel keeps: float input with its missing counts.
__host__ __device__ constexpr int col3d_mode(int M) { return M == MODE_F64 ? kF64Miss : M; }

// LDS bytes per wave for the running 3-D sums (TY rows x R columns).
template <int M, int TY> __host__ __device__ constexpr int tile3d_lds_per_wave(int R)
{
    return TY * R * (int)sizeof(Col<col3d_mode(M)>) * kWave;
}
__host__ __device__ inline int tile3d_lds_bytes(int mode, int TY, int R)
{
    const int cb = mode == MODE_U8 ? (int)sizeof(Col<MODE_U8>)
                                   : (mode == MODE_U16 ? (int)sizeof(Col<MODE_U16>)
                                                       : (int)sizeof(Col<kF64Miss>));
    return TY * R * cb * kWave;
}

// Running 3-D sums of one (row, column) slot in LDS, one 32-bit word per
// lane per component, components strided by 64 lanes (conflict-free).
template <int M> struct S3Slot {
    uint32_t* base;   // word 0 of this slot for lane 0
    static constexpr int NDW = (int)(sizeof(Col<M>) / 4);
    __device__ __forceinline__ void add(int lane, const Col<M>& v) const
    {
        uint32_t w[NDW], a[NDW];
        __builtin_memcpy(a, &v, sizeof(Col<M>));
#pragma unroll
        for (int i = 0; i < NDW; i++) w[i] = base[i * kWave + lane];
        Col<M> cur;
        __builtin_memcpy(&cur, w, sizeof(Col<M>));
        col_add<M>(cur, v);
        __builtin_memcpy(w, &cur, sizeof(Col<M>));
#pragma unroll
        for (int i = 0; i < NDW; i++) base[i * kWave + lane] = w[i];
        (void)a;
    }
    __device__ __forceinline__ Col<M> get(int lane) const
    {
        uint32_t w[NDW];
#pragma unroll
        for (int i = 0; i < NDW; i++) w[i] = base[i * kWave + lane];
        Col<M> cur;
        __builtin_memcpy(&cur, w, sizeof(Col<M>));
        return cur;
    }
    __device__ __forceinline__ void zero(int lane) const
    {
#pragma unroll
        for (int i = 0; i < NDW; i++) base[i * kWave + lane] = 0u;
    }
};

// One row of entering and leaving raw values per lane.
template <class T, int R> struct Row3 {
    static constexpr int NW = Run<T, R>::NW;
    uint32_t xi[NW], yi[NW], xo[NW], yo[NW];
};

template <int M, int R, int KW, int TY, bool VEC>
__device__ __forceinline__ void tile3d(const P3D& g, const int tile, char* smem)
{
    using T = typename Tr<M>::T;
    constexpr int LH = KW / 2;
    constexpr int NW = Run<T, R>::NW;
    constexpr bool kFloat = (M == MODE_F64);
    const int lane = threadIdx.x & (kWave - 1);

    // ---- tile geometry (wave-uniform): y fastest, then x, then z ----
    const int ty = tile % g.tiles_y;
    const int rest = tile / g.tiles_y;
    const int tx = rest % g.tiles_x;
    const int tz = rest / g.tiles_x;
    const int pz0 = tz * g.TZ;
    const int pzn = min(g.TZ, g.OD - pz0);
    const int py0 = ty * TY;
    const int pyn = min(TY, g.OH - py0);
    const int q0 = tx * g.Wq;
    const int qw = min(g.Wq, g.OW - q0);
    const int D = g.D, H = g.H, W = g.W;
    const int E = q0 * g.sx + g.ox;
    const int Eal = (E >= 0) ? (E / R) * R : -((-E + R - 1) / R) * R;
    const bool fill = g.border == BORDER_FILL;
    const bool has_flags = g.flags != nullptr;

    // ---- per-lane column metadata ----
    const int c0 = Eal + lane * R;
    const bool edge = (Eal < 0) || (Eal + kWave * R > W);
    int cidx[R];
    uint32_t colok = 0;
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int c = c0 + j;
        const bool ok = c >= 0 && c < W;
        colok |= ok ? (1u << j) : 0u;
        cidx[j] = ok ? c : (c < 0 ? 0 : W - 1);
    }
    // VEC (W a multiple of R): a lane's run is entirely inside or outside [0, W)
    const uint32_t lane_vo = (colok & 1u) ? (uint32_t)c0 * (uint32_t)sizeof(T) : kOffNone;
    uint32_t omask = 0, fillb = 0;
    int qj[R];
    int ncol[R];
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int qs = c0 + j - g.ox - LH;
        int q = -1;
        if (qs >= 0) {
            q = (g.sx == 1) ? qs : qs / g.sx;
            if (q * g.sx != qs) q = -1;
        }
        omask |= (q >= q0 && q < q0 + qw) ? (1u << j) : 0u;
        qj[j] = q;
        const int clo = q * g.sx + g.ox, chi = clo + KW - 1;
        fillb |= (fill && (clo < 0 || chi >= W)) ? (1u << j) : 0u;
        ncol[j] = min(chi, W - 1) - max(clo, 0) + 1;
    }

    // ---- rows of the y-windows of this tile's output rows ----
    const int ys = py0 * g.sy + g.oy;               // first window row
    const int nyr = (pyn - 1) * g.sy + g.ky;        // window rows in the tile
    // ---- planes ----
    const int zs = pz0 * g.sz + g.oz;               // first window plane
    const int nz = (pzn - 1) * g.sz + g.kz;

    const char* __restrict__ Xb = (const char*)g.x;
    const char* __restrict__ Yb = (const char*)g.y;
    const int64_t rowbytes = (int64_t)W * (int64_t)sizeof(T);
    const int64_t planebytes = (int64_t)H * rowbytes;

    // raw buffer over row r of plane z (zero records outside the volume)
    auto rsrc = [&](const char* A, int z, int r) {
        const bool ok = (unsigned)z < (unsigned)D && (unsigned)r < (unsigned)H;
        const int64_t o = ok ? (int64_t)z * planebytes + (int64_t)r * rowbytes : 0;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(A + o), (short)0, ok ? (int)rowbytes : 0,
                                                 kBufWord3);
    };
    auto load_row = [&](int zin, int zout, int r, Row3<T, R>& out) __attribute__((always_inline)) {
        if constexpr (VEC) {
            buf_load_words<NW>(rsrc(Xb, zin, r), lane_vo, out.xi);
            buf_load_words<NW>(rsrc(Yb, zin, r), lane_vo, out.yi);
            buf_load_words<NW>(rsrc(Xb, zout, r), lane_vo, out.xo);
            buf_load_words<NW>(rsrc(Yb, zout, r), lane_vo, out.yo);
        } else {
            auto one = [&](int z, int rr, uint32_t (&wx)[NW], uint32_t (&wy)[NW]) {
                const bool ok = (unsigned)z < (unsigned)D && (unsigned)rr < (unsigned)H;
                const size_t rb = ok ? ((size_t)z * (size_t)H + (size_t)rr) * (size_t)W : 0;
                const T* xr = (const T*)g.x + rb;
                const T* yr = (const T*)g.y + rb;
                T vx[R], vy[R];
#pragma unroll
                for (int j = 0; j < R; j++) {
                    const bool v = ok && ((colok >> j) & 1u);
                    vx[j] = v ? xr[cidx[j]] : (T)0;
                    vy[j] = v ? yr[cidx[j]] : (T)0;
                }
                uint32_t tx_[NW] = {}, ty_[NW] = {};
                __builtin_memcpy(tx_, vx, sizeof(T) * R);
                __builtin_memcpy(ty_, vy, sizeof(T) * R);
#pragma unroll
                for (int i = 0; i < NW; i++) { wx[i] = tx_[i]; wy[i] = ty_[i]; }
            };
            one(zin, r, out.xi, out.yi);
            one(zout, r, out.xo, out.yo);
        }
    };

    // running 3-D sums in LDS: slot (t, j) at word offset (t*R + j) * NDW * 64
    constexpr int MC = col3d_mode(M);
    constexpr int NDW = S3Slot<MC>::NDW;
    uint32_t* s3w = (uint32_t*)smem;
    auto slot = [&](int t, int j) { return S3Slot<MC>{s3w + (t * R + j) * NDW * kWave}; };
#pragma unroll
    for (int t = 0; t < TY; t++)
#pragma unroll
        for (int j = 0; j < R; j++) slot(t, j).zero(lane);
    float hmx = 0.f, hmy = 0.f;

    int next_ready = g.kz - 1;
    int pz = pz0;
    for (int li = 0; li < nz; li++) {
        const int zin = zs + li;
        const int zout = li >= g.kz ? zin - g.kz : -1;     // -1: nothing leaves yet
        // ---- y-window sums of the z-difference field (registers) ----
        Col<MC> VY[TY][R];
#pragma unroll
        for (int t = 0; t < TY; t++)
#pragma unroll
            for (int j = 0; j < R; j++) col_zero<MC>(VY[t][j]);
        auto consume = [&](int r, Row3<T, R>& rw) __attribute__((always_inline)) {
            T ax[R], ay[R], bx[R], by[R];
            __builtin_memcpy(ax, rw.xi, sizeof(T) * R);
            __builtin_memcpy(ay, rw.yi, sizeof(T) * R);
            __builtin_memcpy(bx, rw.xo, sizeof(T) * R);
            __builtin_memcpy(by, rw.yo, sizeof(T) * R);
            int m[R], mo[R];
#pragma unroll
            for (int j = 0; j < R; j++) { m[j] = 0; mo[j] = 0; }
            if constexpr (kFloat) {
                // missing values are rare: test the row's extremes first
                float lo = ax[0], hi = ax[0];
                bool nan = false;
#pragma unroll
                for (int j = 0; j < R; j++) {
                    lo = fminf(lo, fminf(fminf(ax[j], ay[j]), fminf(bx[j], by[j])));
                    hi = fmaxf(hi, fmaxf(fmaxf(ax[j], ay[j]), fmaxf(bx[j], by[j])));
                    nan = nan | (ax[j] != ax[j]) | (ay[j] != ay[j]) | (bx[j] != bx[j]) |
                          (by[j] != by[j]);
                }
                const bool clean = (lo > g.miss_thr) & (hi < __builtin_inff()) & !nan;
                if (__builtin_amdgcn_ballot_w64(!clean)) {
                    // positions outside the volume read zero and are never missing
                    const bool row_in = (unsigned)(ys + r) < (unsigned)H;
                    const bool in_i = row_in && (unsigned)zin < (unsigned)D;
                    const bool in_o = row_in && (unsigned)zout < (unsigned)D;
#pragma unroll
                    for (int j = 0; j < R; j++) {
                        const bool col_in = (colok >> j) & 1u;
                        m[j] = (in_i && col_in &&
                                (is_missing(ax[j], g.miss_thr) | is_missing(ay[j], g.miss_thr))) ? 1 : 0;
                        mo[j] = (in_o && col_in &&
                                 (is_missing(bx[j], g.miss_thr) | is_missing(by[j], g.miss_thr))) ? 1 : 0;
                        ax[j] = m[j] ? 0.f : ax[j];
                        ay[j] = m[j] ? 0.f : ay[j];
                        bx[j] = mo[j] ? 0.f : bx[j];
                        by[j] = mo[j] ? 0.f : by[j];
                    }
                }
#pragma unroll
                for (int j = 0; j < R; j++) {
                    hmx = fmaxf(hmx, __builtin_fabsf(ax[j]));
                    hmy = fmaxf(hmy, __builtin_fabsf(ay[j]));
                }
            }
#pragma unroll
            for (int j = 0; j < R; j++) {
                const Col<MC> d = col_delta<MC, T>(ax[j], ay[j], bx[j], by[j], m[j], mo[j]);
#pragma unroll
                for (int t = 0; t < TY; t++) {
                    const int lo = t * g.sy;
                    if (t < pyn && r >= lo && r < lo + g.ky) col_add<MC>(VY[t][j], d);
                }
            }
        };
        // rows in pairs: the next row's loads are in flight while one is used
        Row3<T, R> A, B;
        load_row(zin, zout, ys, A);
        for (int r = 0; r < nyr; r += 2) {
            if (r + 1 < nyr) load_row(zin, zout, ys + r + 1, B);
            consume(r, A);
            if (r + 1 >= nyr) break;
            if (r + 2 < nyr) load_row(zin, zout, ys + r + 2, A);
            consume(r + 1, B);
        }
        // ---- x-window sums, added to the running 3-D sums ----
#pragma unroll
        for (int t = 0; t < TY; t++) {
            if (t >= pyn) continue;
            hsum_row<MC, R, KW, false>(VY[t], [&](int j, const Col<MC>& S) __attribute__((always_inline)) {
                slot(t, j).add(lane, S);
            });
        }
        if (li != next_ready) continue;
        next_ready += g.sz;

        // ---- epilogue for output plane pz ----
        const int zlo = pz * g.sz + g.oz, zhi = zlo + g.kz - 1;
        const bool zb = fill && (zlo < 0 || zhi >= D);
        const double nzp = (double)(min(zhi, D - 1) - max(zlo, 0) + 1);
        double gx = 0.0, gy = 0.0;
        if constexpr (kFloat) {
            // bound on |x|, |y| over every value in the running sums: wave max
            float mx = hmx, my = hmy;
            for (int sft = 1; sft < kWave; sft <<= 1) {
                mx = fmaxf(mx, __shfl_xor(mx, sft));
                my = fmaxf(my, __shfl_xor(my, sft));
            }
            gx = g.cert_g * (double)mx * (double)mx;
            gy = g.cert_g * (double)my * (double)my;
        }
#pragma unroll
        for (int t = 0; t < TY; t++) {
            if (t >= pyn) continue;
            const int ylo = (py0 + t) * g.sy + g.oy, yhi = ylo + g.ky - 1;
            const bool rowb = fill && (ylo < 0 || yhi >= H);
            const double nrow = (double)(min(yhi, H - 1) - max(ylo, 0) + 1);
            const size_t orow = ((size_t)pz * g.OH + (size_t)(py0 + t)) * (size_t)g.OW;
#pragma unroll
            for (int j = 0; j < R; j++) {
                if (!((omask >> j) & 1u)) continue;
                const Col<MC> A3 = slot(t, j).get(lane);
                const bool fb = zb || rowb || ((fillb >> j) & 1u);
                const double dn = nzp * nrow * (double)ncol[j];
                uint8_t fl = 0;
                float cv = 0.f;
                if (fb) {
                    fl = FL_BORDER;
                } else if constexpr (kFloat) {
                    if (A3.miss > 0) {
                        fl = FL_MISSING;
                    } else {
                        const int64_t clo = (int64_t)qj[j] * g.sx + g.ox;
                        WinBox wb{(int64_t)H * W, (int64_t)W, max(zlo, 0), min(zhi, D - 1),
                                  max(ylo, 0), min(yhi, H - 1),
                                  max(clo, (int64_t)0), min(clo + KW - 1, (int64_t)W - 1)};
                        // certification against the per-plane thresholds
                        const double N = __builtin_fma(dn, A3.xy, -(A3.x * A3.y));
                        const double Vx = __builtin_fma(dn, A3.xx, -(A3.x * A3.x));
                        const double Vy = __builtin_fma(dn, A3.yy, -(A3.y * A3.y));
                        const bool cert = (Vx > gx) && (Vy > gy) && !(g.force & 1);
                        if (cert) {
                            cv = clamp_unit(newton_ratio(N, Vx * Vy));
                        } else {
                            fl = twopass_window((const float*)g.x, (const float*)g.y, wb.s0, wb.s1,
                                                wb.lo0, wb.hi0, wb.lo1, wb.hi1, wb.lo2, wb.hi2, &cv);
                        }
                    }
                } else {
                    const double sxv = (double)A3.x, syv = (double)A3.y;
                    const double N = __builtin_fma(0.5 * dn, (double)A3.xy2, -(sxv * syv));
                    const double Vx = __builtin_fma(dn, (double)A3.xx, -(sxv * sxv));
                    const double Vy = __builtin_fma(dn, (double)A3.yy, -(syv * syv));
                    fl = (Vx == 0.0 ? FL_ZVAR_X : 0) | (Vy == 0.0 ? FL_ZVAR_Y : 0);
                    if (!fl) cv = rn32_certified(N, Vx, Vy, (g.force & 1) != 0);
                }
                if (fl) cv = g.invalid;
                g.c[orow + (uint32_t)qj[j]] = cv;
                if (has_flags) g.flags[orow + (uint32_t)qj[j]] = fl;
            }
        }
        ++pz;
    }
}

// ---------------------------------------------------------------------------
// Blocks of rows.
//
// One wave owns a block of NR input rows by 64 input columns, one column per
// lane, and marches along z.  A lane keeps the z-window sums Z of its NR cells
// (5 channels) in registers: a step adds the cells of the plane entering the
// z-window and takes those of the leaving one away, once per cell of the
// block.  A step that finishes an output plane also walks down the rows: the
// y-window sum gains row r and loses row r - k_y, the x-window sum comes from
// the neighbour lanes (DPP for distance one, the LDS crossbar beyond), and the
// epilogue and the store of that output row follow.  No cell is ever formed
// twice in a block, no sum passes through LDS, and waves do not wait for each
// other.
//
// What bounds it: vector issue.  A cell costs 14 FP64 operations and a few to
// screen it, NR / NO times per output (12 rows serve 6 output rows at k_y = 7;
// integer input 14 or 20 rows serve 8 or 14); the sums along y two additions per channel, along x (k_x = 7) six
// instructions and four crossbar moves per channel.  A wave that sums the rows
// of its own y-windows step by step (corr3d_kernel) forms each cell (k_y + 1)
// / 2 times and needs the x sums of every plane that only warms its sums up.
// Measured against such a kernel with straight-line steps, 256x512x512: float
// k = 7 725 -> 480 us (216 -> 147 vector instructions per output; 4.6 TB/s from
// and to memory beyond L2: each cell is read again when it leaves and for the
// rows that neighbouring blocks share), k = 3 558
// -> 337; u16 k = 7 654 -> 400, k = 3 486 -> 261; u8 k = 7 345 -> 337, k = 3
// 295 -> 236.  Sharing the rows of a block among the waves of a workgroup
// through LDS instead (units of two rows, R = 4 columns) took 866 us (float k
// = 7): its phases between barriers leave the vector units idle.
// ---------------------------------------------------------------------------
// Input rows per block.  Integer input: blocks that leave registers for three
// waves per SIMD for flat windows, taller ones (two waves) where the rows lost
// to the window weigh more (256x512x512 u8: k = 3 237 us at 12 rows, 287 at 20;
// k = 7 356 and 335; u16 k = 3 275 at 10, 298 at 14; 128x300x301 k = 9 148 and
// 102).  Float input has registers for 12 at two waves: with flat windows they
// gain little in large volumes and lose in small ones (k = 3 at 12 rows and at
// 10: 256x512x512 328 and 336 us, 40x130x200 15.9 and 14.4).
__host__ __device__ constexpr int block3_rows(int mode, int ky)
{
    if (mode == MODE_F64) return ky <= 5 ? 10 : 12;
    if (mode == MODE_U16) return ky <= 5 ? 10 : 14;
    return ky <= 5 ? 12 : 20;
}
__host__ __device__ constexpr int block3_waves(int mode, int NR)
{
    return mode != MODE_F64 && NR <= 12 ? 3 : 2;
}

// x-window sum of one channel with one column per lane, window columns
// [lane - LH, lane + LH]; lanes whose window passes the wave's ends get
// garbage (they store no output).
template <class V, int KW> __device__ __forceinline__ V xsum_lanes(V v)
{
    static_assert(KW == 3 || KW == 5 || KW == 7 || KW == 9, "compiled widths");
    if constexpr (KW == 3) {
        return (dpp_move<true>(v) + v) + dpp_move<false>(v);
    } else {
        const V t2 = v + dpp_move<false>(v);                   // columns c, c + 1
        if constexpr (KW == 5) {
            return (lane_from<2>(t2) + v) + dpp_move<false>(t2);
        } else {
            const V t4 = t2 + lane_from<-2>(t2);               // columns c .. c + 3
            if constexpr (KW == 7) return (lane_from<3>(t4) - v) + t4;   // column c is in both
            else return (lane_from<4>(t4) + v) + dpp_move<false>(t4);
        }
    }
}

// CUBE: k_y = k_x, unit y and z step (the y sums slide); otherwise any k_y <= NR
// and y step, each output row's sum taken from its rows.
template <int M, int KW, int NR, bool CUBE>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(block3_waves(M, NR), 8))) corr3d_block_kernel(P3D g)
{
    using T = typename Tr<M>::T;
    constexpr int LH = KW / 2;
    constexpr bool kFloat = (M == MODE_F64);
    // missing values in the z-window of every cell (float input; touched only
    // once one has entered the block)
    __shared__ int zmiss_all[kFloat ? 4 * NR * kWave : 1];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int tile = xcd_remap(blockIdx.x, gridDim.x) * (int)(blockDim.x / kWave) + wv;
    if (tile >= g.n_tiles) return;
    int* const zmiss = zmiss_all + (kFloat ? wv * NR * kWave : 0);

    // ---- block geometry (wave-uniform): y fastest, then x, then z ----
    const int ty = tile % g.tiles_y;
    const int rest = tile / g.tiles_y;
    const int tx = rest % g.tiles_x;
    const int tz = rest / g.tiles_x;
    const int pz0 = tz * g.TZ;
    const int pzn = min(g.TZ, g.OD - pz0);
    const int py0 = ty * g.NO;
    const int pyn = min(g.NO, g.OH - py0);
    const int q0 = tx * g.Wq;
    const int qw = min(g.Wq, g.OW - q0);
    const int D = g.D, H = g.H, W = g.W, kz = g.kz;
    const int ky = CUBE ? KW : g.ky, sy = CUBE ? 1 : g.sy;
    const bool fill = g.border == BORDER_FILL;
    const bool has_flags = g.flags != nullptr;
    const bool force = (g.force & 1) != 0;

    // ---- this lane's column: the centre of output q when q*sx + ox + LH ----
    const int col = q0 * g.sx + g.ox + lane;
    const bool cin = col >= 0 && col < W;
    const uint32_t lane_vo = cin ? (uint32_t)col * (uint32_t)sizeof(T) : kOffNone;
    const int qs = lane - LH;                           // = (q - q0) * sx
    const int ql = g.sx == 1 ? qs : qs / g.sx;
    const bool out = qs >= 0 && ql * g.sx == qs && ql < qw;
    const uint32_t qoff = out ? (uint32_t)ql * 4u : kOffNone;
    const int ncol = min(col + LH, W - 1) - max(col - LH, 0) + 1;
    const double dncol = (double)ncol;
    const bool fillb = fill && (col - LH < 0 || col + LH >= W);

    // ---- rows ----
    const int ys = py0 * sy + g.oy;                     // first input row of the block
    const int rb = min(max(ys, 0), H - 1);
    const int64_t rowbytes = (int64_t)W * (int64_t)sizeof(T);
    const int64_t planebytes = (int64_t)H * rowbytes;
    // Offsets count from row rb on and the records end with the block's rows or
    // the plane: rows outside the array fall outside the records (those above
    // it wrap to large offsets), and lanes outside the row start 2^31 beyond
    // (all row offsets are below 2^30, the host checks)
    const uint32_t nrec = (uint32_t)min(H - rb, NR) * (uint32_t)rowbytes;
    const uint32_t voff0 = lane_vo + (uint32_t)(ys - rb) * (uint32_t)rowbytes;
    const int zs = pz0 * g.sz + g.oz;                   // first input plane
    const int nz = (pzn - 1) * g.sz + kz;
    auto plane = [&](const void* A, int z) __attribute__((always_inline)) {
        const bool in = (unsigned)z < (unsigned)D;
        const char* at = (const char*)A + (in ? (int64_t)z * planebytes + (int64_t)rb * rowbytes : 0);
        return __builtin_amdgcn_make_buffer_rsrc((void*)at, (short)0, in ? (int)nrec : 0, kBufWord3);
    };
    struct Cell { T x, y, xo, yo; };
    auto load1 = [&](__amdgpu_buffer_rsrc_t rs, uint32_t off) __attribute__((always_inline)) -> T {
        if constexpr (sizeof(T) == 4) return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
        else if constexpr (sizeof(T) == 2) return (T)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
        else return (T)__builtin_amdgcn_raw_buffer_load_b8(rs, off, 0, 0);
    };
    // the block's cells of step li: entering and leaving planes
    auto load_step = [&](int li, Cell (&c)[NR]) __attribute__((always_inline)) {
        const int zi = zs + li, zo = li >= kz ? zi - kz : -1;
        const __amdgpu_buffer_rsrc_t xi = plane(g.x, zi), yi = plane(g.y, zi);
        const __amdgpu_buffer_rsrc_t xo = plane(g.x, zo), yo = plane(g.y, zo);
        // (one add per row instead of a register each)
        const uint32_t v0 = opaque(voff0), step = (uint32_t)opaque_s((int)rowbytes);
#pragma unroll
        for (int r = 0; r < NR; r++) {
            const uint32_t o = v0 + (uint32_t)r * step;
            c[r].x = load1(xi, o);
            c[r].y = load1(yi, o);
            c[r].xo = load1(xo, o);
            c[r].yo = load1(yo, o);
        }
    };

    Col<M> Z[NR];                   // z-window sums
#pragma unroll
    for (int r = 0; r < NR; r++) col_zero<M>(Z[r]);
    if constexpr (kFloat) {
        for (int r = 0; r < NR; r++) zmiss[r * kWave + lane] = 0;
    }
    bool dirty = false;             // wave-uniform: a missing value has entered the block
    float MX = 0.f, MY = 0.f;       // largest |x|, |y| so far (wave-uniform)
    double gx = 0.0, gy = 0.0;      // certification thresholds
    const float thr = g.miss_thr;

    Cell c[NR];                     // the step's cells, loaded during the one before
    load_step(0, c);
    // ---- one step: entering cells in, leaving cells out, the next step's
    //      cells on their way ----
    auto step = [&](int li) __attribute__((always_inline)) {
        if constexpr (kFloat) {
            const int zin = zs + li, zout = li >= kz ? zin - kz : -1;
            auto lost = [&](int r, int z, float a, float b) __attribute__((always_inline)) {
                return (unsigned)(opaque_s(ys) + r) < (unsigned)H && (unsigned)z < (unsigned)D && cin &&
                       (is_missing(a, thr) | is_missing(b, thr));
            };
            auto largest = [&](float& mx, float& my) __attribute__((always_inline)) {
                mx = my = 0.f;
#pragma unroll
                for (int r = 0; r < NR; r += 2) {
                    mx = fmax3_abs(mx, c[r].x, c[r + 1].x);
                    my = fmax3_abs(my, c[r].y, c[r + 1].y);
                }
            };
            // Entering values above the threshold, finite?  (the leaving ones
            // entered earlier.)  While all magnitudes are below a negative
            // threshold's, only NaN is left to look for, which spoils the sum
            // of products.
            float mx, my, t = 0.f;
            largest(mx, my);
#pragma unroll
            for (int r = 0; r < NR; r++) t = __builtin_fmaf(c[r].x, c[r].y, t);
            bool sus = !(__builtin_fabsf(t) < __builtin_inff());
            if (__builtin_amdgcn_ballot_w64(!(fmaxf(mx, my) < -thr))) {
                float lo = c[0].x;
#pragma unroll
                for (int r = 0; r < NR; r++) lo = fmin3(lo, c[r].x, c[r].y);
                sus = sus | !(lo > thr);
            }
            if (dirty || __builtin_amdgcn_ballot_w64(sus)) {
                // some value may be missing, or the threshold takes the zeros
                // read outside the array for missing ones
                bool any = false;
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    const bool m = lost(r, zin, c[r].x, c[r].y), mo = lost(r, zout, c[r].xo, c[r].yo);
                    any |= m;
                    c[r].x = m ? 0.f : c[r].x;
                    c[r].y = m ? 0.f : c[r].y;
                    c[r].xo = mo ? 0.f : c[r].xo;
                    c[r].yo = mo ? 0.f : c[r].yo;
                    if (m != mo) zmiss[r * kWave + lane] += m ? 1 : -1;
                }
                dirty = dirty || __builtin_amdgcn_ballot_w64(any) != 0;
                largest(mx, my);
            }
            if (__builtin_amdgcn_ballot_w64((mx > MX) | (my > MY))) {
                MX = fmaxf(MX, wave_max(mx));
                MY = fmaxf(MY, wave_max(my));
                gx = g.cert_g * (double)MX * (double)MX;
                gy = g.cert_g * (double)MY * (double)MY;
            }
        }
#pragma unroll
        for (int r = 0; r < NR; r++) col_accum_delta<M, T>(Z[r], c[r].x, c[r].y, c[r].xo, c[r].yo);
        // (formed before the next loads are issued: the next cells take these
        // cells' registers)
#pragma unroll
        for (int r = 0; r < NR; r++)
            col_each<M>(Z[r], Z[r], [](auto& d, const auto&) __attribute__((always_inline)) { d = opaque(d); });
        // (past the last step: planes that are not used)
        load_step(li + 1, c);
    };
    // ---- output plane pz from the sums as they are ----
    auto finish = [&](int pz) __attribute__((always_inline)) {
        const int zlo = pz * g.sz + g.oz, zhi = zlo + kz - 1;
        const bool zb = fill && (zlo < 0 || zhi >= D);
        const int nzp = min(zhi, D - 1) - max(zlo, 0) + 1;
        const int64_t obase = ((int64_t)pz * g.OH + py0) * (int64_t)g.OW + q0;
        const int orec = (pyn - 1) * g.OW + qw;
        const __amdgpu_buffer_rsrc_t rc =
            __builtin_amdgcn_make_buffer_rsrc(g.c + obase, (short)0, orec * 4, kBufWord3);
        const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc(
            has_flags ? (void*)(g.flags + obase) : (void*)g.c, (short)0, has_flags ? orec : 0, kBufWord3);
        uint32_t missm = 0, pm = 0; // output rows: a missing value in the window; not settled
        Col<M> V;                   // running y-window sum (CUBE)
        col_zero<M>(V);

        // output row o (rows o*sy .. o*sy + ky - 1 of the block) from its y sums
        auto emit = [&](int o, const Col<M>& Y) __attribute__((always_inline)) {
            Col<M> S;
            S.x = xsum_lanes<decltype(S.x), KW>(Y.x);
            S.y = xsum_lanes<decltype(S.y), KW>(Y.y);
            S.xx = xsum_lanes<decltype(S.xx), KW>(Y.xx);
            S.yy = xsum_lanes<decltype(S.yy), KW>(Y.yy);
            if constexpr (kFloat) S.xy = xsum_lanes<double, KW>(Y.xy);
            else S.xy2 = xsum_lanes<decltype(S.xy2), KW>(Y.xy2);
            const int ylo = opaque_s(ys) + o * sy, yhi = ylo + ky - 1;
            const bool fb = zb || (fill && (ylo < 0 || yhi >= H));
            const double dn = (double)(nzp * (min(yhi, H - 1) - max(ylo, 0) + 1)) * dncol;
            const bool bord = fb | fillb;
            float cv;
            uint32_t fl;
            if constexpr (kFloat) {
                const double N = __builtin_fma(dn, S.xy, -(S.x * S.y));
                const double Vx = __builtin_fma(dn, S.xx, -(S.x * S.x));
                const double Vy = __builtin_fma(dn, S.yy, -(S.y * S.y));
                const bool miss = (missm >> o) & 1u;
                const bool bad = bord | miss;
                pm |= (!((Vx > gx) & (Vy > gy)) | force) & !bad & out & (o < pyn) ? 1u << o : 0u;
                const float v = opaque(clamp_unit(newton_ratio(N, Vx * Vy)));
                cv = bad ? g.invalid : v;
                fl = bord ? FL_BORDER : (miss ? FL_MISSING : 0u);
            } else {
                const double sx = (double)S.x, syv = (double)S.y;
                const double N = __builtin_fma(0.5 * dn, (double)S.xy2, -(sx * syv));
                const double Vx = __builtin_fma(dn, (double)S.xx, -(sx * sx));
                const double Vy = __builtin_fma(dn, (double)S.yy, -(syv * syv));
                const double q = Vx * Vy;
                bool amb;
                cv = opaque(rn32_fast(N, q, amb));
                const bool bad = bord | (q == 0.0);
                if (__builtin_amdgcn_ballot_w64((amb | force) & !bad & out)) {
                    if ((amb | force) && !bad) {
                        // any estimate far inside half an ulp selects the right bucket
                        const double aN = __builtin_fabs(N);
                        const float f = rn32_exact_decide(aN, Vx, Vy, aN / __builtin_sqrt(q));
                        cv = N < 0.0 ? -f : f;
                    }
                }
                cv = bad ? g.invalid : cv;
                fl = bord ? (uint32_t)FL_BORDER
                          : ((Vx == 0.0 ? FL_ZVAR_X : 0u) | (Vy == 0.0 ? FL_ZVAR_Y : 0u));
            }
            // (output rows past the block's last are formed; their offsets lie
            // beyond the records)
            const uint32_t orow = (uint32_t)(o * opaque_s(g.OW));
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(cv), rc, opaque(qoff) + orow * 4u, 0, 0);
            if (has_flags)
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)fl, rf, out ? (opaque(qoff) >> 2) + orow : kOffNone, 0, 0);
        };

        if (kFloat && dirty) {
            // window sums of the missing counts, output row by output row
            for (int o = 0; o < pyn; o++) {
                int m = 0;
                for (int r = o * sy; r < o * sy + ky; r++) m += zmiss[r * kWave + lane];
                missm |= xsum_lanes<int, KW>(m) > 0 ? 1u << o : 0u;
            }
        }
        if constexpr (CUBE) {
#pragma unroll
            for (int r = 0; r < NR; r++) {
                col_add<M>(V, Z[r]);
                if (r >= KW) col_sub<M>(V, Z[r >= KW ? r - KW : 0]);
                if (r >= KW - 1) emit(r - (KW - 1), V);
                // (one output row at a time: more would not leave registers)
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            int o = 0;
#pragma unroll
            for (int r = 0; r < NR; r++) {
                // (uniform: is row r the first of an output row's window?)
                if (o < pyn && r == o * sy) {
                    Col<M> Y = Z[r];
#pragma unroll
                    for (int i = 1; i < NR - r; i++)
                        if (i < ky) col_add<M>(Y, Z[r + i]);
                    emit(o, Y);
                    o++;
                }
            }
        }
        if constexpr (kFloat) {
            // rare path: the two-pass formula, stored over the estimate
            if (__builtin_amdgcn_ballot_w64(pm != 0u)) {
                __builtin_amdgcn_s_waitcnt(0);
                while (pm) {
                    const int o = __builtin_ctz(pm);
                    pm &= pm - 1;
                    const int ylo = (py0 + o) * sy + g.oy;
                    float cv = 0.f;
                    const uint8_t fl = twopass_window(
                        (const float*)g.x, (const float*)g.y, (int64_t)H * W, (int64_t)W, max(zlo, 0),
                        min(zhi, D - 1), max(ylo, 0), min(ylo + ky - 1, H - 1), max(col - LH, 0),
                        min(col + LH, W - 1), &cv);
                    const int64_t oi = obase + (int64_t)o * g.OW + ql;
                    g.c[oi] = fl ? g.invalid : cv;
                    if (has_flags) g.flags[oi] = fl;
                }
            }
        }
    };
    int next_ready = kz - 1;        // the step that completes output plane pz
    int pz = pz0;
    for (int li = 0; li < nz; li++) {
        step(li);
        if (li != next_ready) continue;
        next_ready += CUBE ? 1 : g.sz;
        finish(pz++);
    }
}

template <int M, int R, int KW, int TY, bool VEC>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(2, 8))) corr3d_kernel(P3D g)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);   // wave-uniform
    const int wpb = blockDim.x / kWave;
    const int tile = xcd_remap(blockIdx.x, gridDim.x) * wpb + wv;
    if (tile >= g.n_tiles) return;
    tile3d<M, R, KW, TY, VEC>(g, tile, smem + (size_t)wv * tile3d_lds_per_wave<M, TY>(R));
}

}  // namespace swc
