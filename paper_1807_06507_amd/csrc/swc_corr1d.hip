// 1-D sliding-window correlation (Poyda & Zhizhin, arXiv 1807.06507: the
// one-dimensional moving sum of Section 1, applied to x, y, xy, x^2, y^2,
// then the one-pass formula per position).
//
// Work decomposition: one wavefront owns a contiguous segment of outputs and
// walks the window-end positions e of that segment in rows of 64*R
// consecutive positions (lane t owns positions row + t*R .. row + t*R + R-1).
// With S_e the sum over [e-k+1, e]:
//     S_e = S_{e-1} + v_e - v_{e-k}
// so a row of S values is  carry + (prefix over the row of d_e = v_e - v_{e-k}):
// an in-lane prefix over R positions, a wavefront scan of the lane totals
// (DPP row shifts + row broadcasts) and the carry from the previous row.
// The carry starts from a direct sum of the k positions before the segment.
//
// What bounds it is vector issue and, at the end, memory (2^28 floats,
// k = 1001: 2.1 GB in, 1.1 GB out, 0.63 ms at the rate of a copy; 1.085 ms
// before the points below, 0.71 ms now, u16 2.00 -> 0.65 ms).  Rows of the
// inside of a series (every window inside it) run straight-line code, 78
// vector instructions per output where 129 were: products enter and leave
// the prefix as two FMAs without forming their difference; the values
// entering are screened by their minimum and by one sum that a NaN or Inf
// spoils; the largest |x|, |y| of the wave is looked at again only when a lane
// passes it; rows holding missing values (entering, or leaving until k
// positions later) take a masked copy of the same code; windows the estimate
// does not settle send the row through the rolled loop below once more.  (R =
// 16 positions per lane would halve the scan's share of 17, but the float
// kernel then spills: 1.3 ms.)  Rows at the ends of the series, and a
// segment's last, partial row, take that rolled loop alone (edge_sums,
// one_by_one).
#include <algorithm>
#include <type_traits>

#include "swc_device.hpp"
#include "swc_dispatch.hpp"
#include "swc_internal.h"

namespace swc {

struct P1D {
    const void* x;
    const void* y;
    float* c;
    uint8_t* flags;
    int64_t N, ON;
    int k, s, off;        // window, step, window start offset (-k/2 or 0)
    int border;
    float invalid;
    float miss_thr;
    int force;
    double cert_g;
    int64_t seg;          // outputs per wave
    int64_t n_waves;
    int vst;              // bit 0: c 16-byte aligned, bit 1: flags 4-byte aligned (vector stores)
    int ring_g;           // RING kernel: groups of R positions in the per-wave LDS ring
    int edge;             // EDGE kernel (host only)
};

constexpr int kR1 = 8;               // positions per lane per row
constexpr int kRow1 = kWave * kR1;   // positions per row
constexpr int kBufWord3_1d = 0x00020000;   // raw buffer access (gfx9 family)

// The five sums, all in FP64 (exact integers for integer input).
struct Ch {
    double x, y, xx, yy, xy;
};
__device__ __forceinline__ Ch operator+(const Ch& a, const Ch& b)
{
    return Ch{a.x + b.x, a.y + b.y, a.xx + b.xx, a.yy + b.yy, a.xy + b.xy};
}
__device__ __forceinline__ Ch operator-(const Ch& a, const Ch& b)
{
    return Ch{a.x - b.x, a.y - b.y, a.xx - b.xx, a.yy - b.yy, a.xy - b.xy};
}
__device__ __forceinline__ Ch ch_scan(const Ch& a)
{
    return Ch{wave_incl_scan(a.x), wave_incl_scan(a.y), wave_incl_scan(a.xx),
              wave_incl_scan(a.yy), wave_incl_scan(a.xy)};
}
__device__ __forceinline__ Ch ch_lane63(const Ch& a)
{
    return Ch{lane63(a.x), lane63(a.y), lane63(a.xx), lane63(a.yy), lane63(a.xy)};
}
// S + v - v' for one position: the products enter and leave as two FMAs (two
// roundings, as the difference and its addition would have).
__device__ __forceinline__ Ch ch_step(const Ch& S, float x, float y, float xo, float yo)
{
    const double a = (double)x, b = (double)y, ao = (double)xo, bo = (double)yo;
    return Ch{S.x + (a - ao), S.y + (b - bo), __builtin_fma(a, a, __builtin_fma(-ao, ao, S.xx)),
              __builtin_fma(b, b, __builtin_fma(-bo, bo, S.yy)),
              __builtin_fma(a, b, __builtin_fma(-ao, bo, S.xy))};
}

// Raw buffer over one wave's span of an input array: span position d (array
// index e_base + d) is read at byte offset d * sizeof(T) + delta + mis, where
// mis is the misalignment of span position 0 to a word (integer input; float
// input is read at any word).
struct SpanBuf {
    __amdgpu_buffer_rsrc_t rs;
    int delta;
    uint32_t mis;
};

template <class T>
__device__ __forceinline__ SpanBuf span_buf(const T* A, int64_t N, int64_t e_base)
{
    constexpr uintptr_t kMask = sizeof(T) == 4 ? 0 : 3;
    const int64_t eb0 = e_base > 0 ? e_base : 0;
    const uintptr_t first = (uintptr_t)(A + eb0);
    const uintptr_t base = first & ~kMask;
    const int64_t avail = N - eb0 > 0 ? N - eb0 : 0;
    const int64_t bytes = ((int64_t)(avail * (int64_t)sizeof(T) + (int64_t)(first - base)) + (int64_t)kMask) &
                          ~(int64_t)kMask;
    const int nrec = (int)(bytes < 0x7FFFFFF0ll ? bytes : 0x7FFFFFF0ll);
    const uintptr_t at0 = (uintptr_t)A + (uintptr_t)(e_base * (int64_t)sizeof(T));
    SpanBuf b;
    b.mis = (uint32_t)(at0 & kMask);
    b.rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, avail ? nrec : 0, kBufWord3_1d);
    b.delta = (int)(int64_t)(at0 - b.mis - base);
    return b;
}

// The value at span position d; zero outside the series (`in` false).
template <class T>
__device__ __forceinline__ float span_load(const SpanBuf& b, int d, bool in)
{
    const uint32_t off = in ? (uint32_t)(d * (int)sizeof(T) + b.delta) + b.mis : 0x80000000u;
    if constexpr (sizeof(T) == 4)
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b.rs, off, 0, 0));
    else if constexpr (sizeof(T) == 2)
        return (float)__builtin_amdgcn_raw_buffer_load_b16(b.rs, off, 0, 0);
    else
        return (float)__builtin_amdgcn_raw_buffer_load_b8(b.rs, off, 0, 0);
}

// A lane's R consecutive cells as words (integer input: one word more, the
// run may begin inside one).  Every cell lies in the series.
template <class T> struct Cells {
    static constexpr int NW = kR1 * (int)sizeof(T) / 4;
    static constexpr int NL = sizeof(T) == 4 ? NW : NW + 1;
    uint32_t w[NL];
    __device__ __forceinline__ void load(const SpanBuf& b, int d0)
    {
        const uint32_t off = (uint32_t)(d0 * (int)sizeof(T) + b.delta);
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int i = 0; i + 4 <= NL; i += 4) {
            const u4 v = __builtin_amdgcn_raw_buffer_load_b128(b.rs, off + 4u * i, 0, 0);
            w[i] = v.x; w[i + 1] = v.y; w[i + 2] = v.z; w[i + 3] = v.w;
        }
        constexpr int kRest = NL & ~3;
        if constexpr (NL % 4 == 3) {
            typedef uint32_t u3 __attribute__((ext_vector_type(3)));
            const u3 v = __builtin_amdgcn_raw_buffer_load_b96(b.rs, off + 4u * kRest, 0, 0);
            w[kRest] = v.x; w[kRest + 1] = v.y; w[kRest + 2] = v.z;
        } else if constexpr (NL % 4 == 1) {
            w[kRest] = __builtin_amdgcn_raw_buffer_load_b32(b.rs, off + 4u * kRest, 0, 0);
        }
        static_assert(NL % 4 != 2, "words of a run");
    }
    __device__ __forceinline__ float at(int j, uint32_t mis) const
    {
        if constexpr (sizeof(T) == 4) {
            return __uint_as_float(w[j]);
        } else {
            constexpr int kPer = 4 / (int)sizeof(T), kBits = 8 * (int)sizeof(T);
            const uint32_t v = __builtin_amdgcn_alignbyte(w[j / kPer + 1], w[j / kPer], mis);
            return (float)((v >> (kBits * (j % kPer))) & ((1u << kBits) - 1u));
        }
    }
};

// Waves per SIMD the register allocation allows: three (2^28 floats, k = 1001:
// 769 us with two; u16 730 us with two, 657 with three), but two for the float
// kernels that would spill.
template <int M, bool RING, bool STEP1> constexpr int corr1d_min_waves()
{
    return M == MODE_F64 && !(RING && STEP1) ? 2 : 3;
}

// RING: the values leaving the window come from a per-wave LDS ring of the
// last ring_g*R positions instead of a second read from memory.  Position p
// lives at pair (p mod R) * ring_g + (p / R mod ring_g), x and y together
// (ring_g exactly k + one row, so that a CU holds the rings of twelve waves up to
// k = 1185): a lane owns R consecutive positions starting at a multiple of R, so for each
// of them the 64 lanes write, and (k back) read, 64 consecutive pairs.  The
// ring holds the raw values; missing values are masked on use.
// STEP1: unit step (every position is an output, stored as vectors).
// EDGE: one row per wave, settled position by position but with every cell of the
// row read before (series of no more rows than CUs, whose time is that of the
// rows at the ends; 411 cells, k = 5: u8 and u16 7.0 -> 5.0 us, float 10.6 -> 5.9;
// 100000, k = 1001: u16 9.2 -> 7.1, float 13.0 -> 8.4).
template <int M, bool RING, bool STEP1, bool EDGE = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(EDGE ? 2 : corr1d_min_waves<M, RING, STEP1>(), 8)))
corr1d_kernel(P1D g)
{
    static_assert(!(EDGE && RING), "one row needs no ring");
    using T = typename Tr<M>::T;
    constexpr int R = kR1;
    constexpr bool kFloat = !Tr<M>::kInt;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);   // wave-uniform
    const int wpb = blockDim.x / kWave;
    const int64_t w = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * wpb + wv;
    if (w >= g.n_waves) return;

    const int64_t N = g.N;
    const int k = g.k;
    const int64_t p_first = w * g.seg;
    const int64_t p_last = min(p_first + g.seg, g.ON) - 1;
    const int64_t e_first = p_first * g.s + g.off + k - 1;   // window end of p_first
    const int64_t e_last = p_last * g.s + g.off + k - 1;
    const int kal = ((k + R - 1) / R) * R;
    // span positions are relative to e_base; everything below is 32-bit
    const int64_t e_base = e_first - kal;
    const int d_end = (int)(e_last - e_base);                // last window end
    const int64_t nlim64 = N - e_base;                       // positions d < nlim are < N
    const int nlim = (int)(nlim64 > 0x3FFFFFFF ? 0x3FFFFFFF : (nlim64 < -0x3FFFFFFF ? -0x3FFFFFFF : nlim64));
    const int dmin = (int)(e_base < 0 ? -e_base : 0);        // positions d >= dmin are >= 0
    const SpanBuf bx = span_buf<T>((const T*)g.x, N, e_base);
    const SpanBuf by = span_buf<T>((const T*)g.y, N, e_base);
    const int pstep = g.s;
    const float thr = g.miss_thr;
    auto inside = [&](int d) __attribute__((always_inline)) { return d >= dmin && d < nlim; };
    auto missing = [&](float a, float b) __attribute__((always_inline)) {
        return is_missing(a, thr) | is_missing(b, thr);
    };

    // ---- per-wave LDS ring (RING) ----
    extern __shared__ __attribute__((aligned(16))) float2 ring_smem[];
    const int rg = g.ring_g;
    float2* ring = ring_smem + (size_t)wv * R * rg;
    // (the span's first ring_g groups hold the positions before the first row;
    // a group index only ever lies in [0, 2 ring_g) before it is wrapped)
    auto wrap = [&](int q) __attribute__((always_inline)) { return q >= rg ? q - rg : q; };
    int rbase = kal / R;                   // ring group of the row's first position

    // ---- carry = sums over span positions [kal - k, kal - 1] ----
    Ch carry;
    int cmiss = 0;                   // missing values in the window before the row
    float MX = 0.f, MY = 0.f;        // largest |x|, |y| so far (wave-uniform)
    int dirty_end = 0;               // rows beginning before it may hold missing values
    {
        Ch part = Ch{0, 0, 0, 0, 0};
        int pm = 0;
        float mx = 0.f, my = 0.f;
        constexpr int B = 8;         // loads in flight per lane and array
        for (int i0 = kal - k + lane; i0 < kal; i0 += B * kWave) {
            float a[B], b[B];
#pragma unroll
            for (int u = 0; u < B; u++) {
                const int i = i0 + u * kWave;
                const bool in = i < kal && inside(i);
                a[u] = span_load<T>(bx, i, in);
                b[u] = span_load<T>(by, i, in);
            }
#pragma unroll
            for (int u = 0; u < B; u++) {
                const int i = i0 + u * kWave;
                if (i >= kal) break;
                if constexpr (RING) ring[(i & (R - 1)) * rg + i / R] = make_float2(a[u], b[u]);
                if constexpr (kFloat) {
                    // positions outside the series read zero and are never missing
                    if (inside(i) && missing(a[u], b[u])) { a[u] = 0.f; b[u] = 0.f; pm++; }
                    mx = fmaxf(mx, __builtin_fabsf(a[u]));
                    my = fmaxf(my, __builtin_fabsf(b[u]));
                }
                part = ch_step(part, a[u], b[u], 0.f, 0.f);
            }
        }
        carry = ch_lane63(ch_scan(part));
        if constexpr (kFloat) {
            MX = wave_max(mx);
            MY = wave_max(my);
            cmiss = lane63(wave_incl_scan(pm));
            if (cmiss) dirty_end = kal + k;
        }
    }
    const double gcert = g.cert_g;
    double gx = gcert * (double)MX * (double)MX, gy = gcert * (double)MY * (double)MY;
    auto grow = [&](float lmx, float lmy) __attribute__((always_inline)) {
        if (__builtin_amdgcn_ballot_w64((lmx > MX) | (lmy > MY))) {
            MX = fmaxf(MX, wave_max(lmx));
            MY = fmaxf(MY, wave_max(lmy));
            gx = gcert * (double)MX * (double)MX;
            gy = gcert * (double)MY * (double)MY;
        }
    };
    const bool has_flags = g.flags != nullptr;
    const bool fill = g.border == BORDER_FILL;
    const bool force = (g.force & 1) != 0;
    const double dk = (double)k;

    // outputs of this wave as raw buffers (out-of-range offsets drop stores)
    const int nout = (int)(p_last - p_first + 1);
    const __amdgpu_buffer_rsrc_t rc =
        __builtin_amdgcn_make_buffer_rsrc(g.c + p_first, (short)0, nout * 4, kBufWord3_1d);
    const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc(
        has_flags ? (void*)(g.flags + p_first) : (void*)g.c, (short)0, has_flags ? nout : 0,
        kBufWord3_1d);
    const bool vec_c = (g.vst & 1) && (p_first & 3) == 0;
    const bool vec_f = (g.vst & 2) && (p_first & 3) == 0;

    // N, Vx, Vy of window sums S over n cells
    auto nvv = [](const Ch& S, double n, double& Nn, double& Vx, double& Vy)
        __attribute__((always_inline)) {
        Nn = __builtin_fma(n, S.xy, -(S.x * S.y));
        Vx = __builtin_fma(n, S.xx, -(S.x * S.x));
        Vy = __builtin_fma(n, S.yy, -(S.y * S.y));
    };
    // ---- a row whose windows all lie inside the series ----
    Cells<T> cx, cy;                 // its cells, loaded while the previous row was worked on
    auto row_ok = [&](int rrel) __attribute__((always_inline)) {
        return rrel + kRow1 - 1 <= d_end && rrel + kRow1 - 1 < nlim && rrel - k + 1 >= dmin &&
               rrel - k >= dmin;
    };
    // Returns whether a float window of the row is not settled by its estimate;
    // integer windows are settled here.
    auto fast_row = [&](const int rrel, auto dirty_tag) __attribute__((always_inline)) -> bool {
        constexpr bool dirty = decltype(dirty_tag)::value;   // it may hold missing values
        const int d0 = rrel + lane * R;
        Ch P[R];                     // in-lane prefix of the differences
        uint32_t me = 0, ml = 0;     // entering / leaving positions that are missing
        // the ring slots of the leaving positions: d0 + j - k = (d0 - kal) + (kk + j),
        // group (d0 - kal) / R or the one after it, slot (kk + j) mod R
        const int kk = kal - k;
        const float2* rd[2] = {ring, ring};       // of the leaving positions' two groups
        if constexpr (RING) {
            const int from = rbase - kal / R + (rbase < kal / R ? rg : 0) + lane;
            rd[0] = ring + wrap(from);
            rd[1] = ring + wrap(from + 1);
            float2* wr = ring + wrap(rbase + lane);
#pragma unroll
            for (int j = 0; j < R; j++) wr[j * rg] = make_float2(cx.at(j, bx.mis), cy.at(j, by.mis));
            wave_lds_sync();         // other lanes read them
        }
        Cells<T> ox, oy;
        if constexpr (!RING) {
            // (k back is any alignment: integer input re-reads cell by cell)
            if constexpr (kFloat) {
                ox.load(bx, d0 - k);
                oy.load(by, d0 - k);
            }
        }
        auto leaving = [&](int j, float& xo, float& yo) __attribute__((always_inline)) {
            if constexpr (RING) {
                const int q = kk + j;
                const float2 v = (q < R ? rd[0] : rd[1])[(q & (R - 1)) * rg];
                xo = v.x;
                yo = v.y;
            } else if constexpr (kFloat) {
                xo = ox.at(j, 0);
                yo = oy.at(j, 0);
            } else {
                xo = span_load<T>(bx, d0 + j - k, true);
                yo = span_load<T>(by, d0 + j - k, true);
            }
        };
        // differences and their prefix; MISS: missing values masked
        auto prefix = [&](auto miss_tag) __attribute__((always_inline)) {
            constexpr bool MISS = decltype(miss_tag)::value;
#pragma unroll
            for (int j = 0; j < R; j++) {
                float a = cx.at(j, bx.mis), b = cy.at(j, by.mis), ao, bo;
                leaving(j, ao, bo);
                if constexpr (MISS) {
                    const bool m = missing(a, b), mo = missing(ao, bo);
                    a = m ? 0.f : a;
                    b = m ? 0.f : b;
                    ao = mo ? 0.f : ao;
                    bo = mo ? 0.f : bo;
                    me |= m ? 1u << j : 0u;
                    ml |= mo ? 1u << j : 0u;
                }
                P[j] = ch_step(j ? P[j - 1] : Ch{0, 0, 0, 0, 0}, a, b, ao, bo);
                // (in groups: the ring reads of a whole row at once would
                // not leave registers for the prefix)
                if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
        };
        prefix(dirty_tag);
        if constexpr (kFloat && dirty) {
            float lmx = 0.f, lmy = 0.f;
#pragma unroll
            for (int j = 0; j < R; j++) {
                lmx = fmaxf(lmx, ((me >> j) & 1u) ? 0.f : __builtin_fabsf(cx.at(j, 0)));
                lmy = fmaxf(lmy, ((me >> j) & 1u) ? 0.f : __builtin_fabsf(cy.at(j, 0)));
            }
            if (__builtin_amdgcn_ballot_w64(me != 0)) dirty_end = rrel + kRow1 + k;
            grow(lmx, lmy);
        }
        // the next row's cells, in flight during the scan and the outputs
        if (row_ok(rrel + kRow1)) {
            cx.load(bx, d0 + kRow1);
            cy.load(by, d0 + kRow1);
        }
        // wavefront scan of the lane totals -> sums before each lane's positions
        const Ch tot = P[R - 1];
        const Ch inc = ch_scan(tot);
        const Ch base = carry + (inc - tot);
        carry = carry + ch_lane63(inc);
        int bmiss = 0;
        if constexpr (kFloat && dirty) {
            const int tm = __popc(me) - __popc(ml);
            const int im = wave_incl_scan(tm);
            bmiss = cmiss + im - tm;
            cmiss += lane63(im);
        }
        uint64_t pend_row = 0;
        // ---- outputs ending at span positions d0 + j ----
        int o0 = d0 - kal, orem = 0;          // output of position d0 (STEP1), or the last one
        if constexpr (!STEP1) {               // at or before it and the positions since
            const int qs = d0 - kal;
            o0 = qs / pstep;
            orem = qs - o0 * pstep;
        }
        auto miss_at = [&](int j) __attribute__((always_inline)) {
            const uint32_t low = (2u << j) - 1u;
            return bmiss + __popc(me & low) - __popc(ml & low) > 0;
        };
#pragma unroll
        for (int j0 = 0; j0 < R; j0 += 4) {
            float cv[4];
            uint32_t fl = 0, outm = 15u;
            uint64_t pend = 0;
            int oidx[STEP1 ? 1 : 4];
            if constexpr (!STEP1) {
                outm = 0;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    oidx[i] = o0;
                    outm |= orem == 0 ? 1u << i : 0u;
                    orem++;
                    if (orem == pstep) { orem = 0; o0++; }
                    // (position d0 + j with a remainder r belongs between outputs)
                }
                if (!__builtin_amdgcn_ballot_w64(outm != 0)) continue;
            }
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int j = j0 + i;
                const Ch S = base + P[j];
                double Nn, Vx, Vy;
                nvv(S, dk, Nn, Vx, Vy);
                const double q = Vx * Vy;
                if constexpr (kFloat) {
                    cv[i] = clamp_unit(newton_ratio(Nn, q));
                    bool pd = !((Vx > gx) & (Vy > gy));
                    if constexpr (dirty) {
                        const bool ms = miss_at(j);
                        cv[i] = ms ? g.invalid : cv[i];
                        fl |= ms ? (uint32_t)FL_MISSING << (8 * i) : 0u;
                        pd = pd & !ms;
                    }
                    pend |= __builtin_amdgcn_ballot_w64(pd);
                } else {
                    const double a = newton_ratio(Nn, q);
                    const uint32_t lo29 = (uint32_t)__double_as_longlong(a) & 0x1FFFFFFFu;
                    const bool amb = (lo29 - (0x10000000u - (1u << 15))) <= (2u << 15);
                    const bool zero = q == 0.0;
                    cv[i] = zero ? g.invalid : (float)a;
                    if (has_flags)
                        fl |= ((Vx == 0.0 ? FL_ZVAR_X : 0u) | (Vy == 0.0 ? FL_ZVAR_Y : 0u)) << (8 * i);
                    pend |= __builtin_amdgcn_ballot_w64(amb & !zero);
                }
            }
            if constexpr (kFloat) {
                pend_row |= pend;
            } else if (pend || force) {
                // rare path: the exact rounding decision
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const Ch S = base + P[j0 + i];
                    double Nn, Vx, Vy;
                    nvv(S, dk, Nn, Vx, Vy);
                    if (((outm >> i) & 1u) && Vx != 0.0 && Vy != 0.0)
                        cv[i] = rn32_certified(Nn, Vx, Vy, force);
                }
            }
            if constexpr (STEP1) {
                const uint32_t o = (uint32_t)(o0 + j0);
                if (vec_c) {
                    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
                    const u4 v = {__float_as_uint(cv[0]), __float_as_uint(cv[1]),
                                  __float_as_uint(cv[2]), __float_as_uint(cv[3])};
                    __builtin_amdgcn_raw_buffer_store_b128(v, rc, o * 4u, 0, 0);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; i++)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(cv[i]), rc, (o + i) * 4u, 0, 0);
                }
                if (has_flags) {
                    if (vec_f) {
                        __builtin_amdgcn_raw_buffer_store_b32(fl, rf, o, 0, 0);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; i++)
                            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(fl >> (8 * i)), rf, o + i, 0, 0);
                    }
                }
            } else {
                // positions that are not outputs get an offset beyond any
                // record count (after the scaling, so that it cannot wrap)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const bool is_o = (outm >> i) & 1u;
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(cv[i]), rc,
                                                          is_o ? (uint32_t)oidx[i] * 4u : 0x80000000u, 0, 0);
                    if (has_flags)
                        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(fl >> (8 * i)), rf,
                                                             is_o ? (uint32_t)oidx[i] : 0x80000000u, 0, 0);
                }
            }
        }
        return kFloat && (pend_row || force);
    };

    // Whether the row just loaded may hold missing values, entering or (up to
    // k positions after one entered) leaving: the entering values are screened
    // by their minimum and by a sum of products that a NaN or Inf spoils (a
    // finite overflow merely sends the row through the masked code).
    auto screen = [&](const int rrel) __attribute__((always_inline)) -> bool {
        if constexpr (!kFloat) return false;
        if (rrel < dirty_end) return true;
        float lo = fmin3(cx.at(0, 0), cy.at(0, 0), cx.at(1, 0)), t = 0.f, lmx = 0.f, lmy = 0.f;
        lo = fmin3(lo, cy.at(1, 0), cy.at(1, 0));
#pragma unroll
        for (int j = 2; j < R; j++) lo = fmin3(lo, cx.at(j, 0), cy.at(j, 0));
#pragma unroll
        for (int j = 0; j < R; j++) t = __builtin_fmaf(cx.at(j, 0), cy.at(j, 0), t);
        if (__builtin_amdgcn_ballot_w64(!(lo > thr) | !(__builtin_fabsf(t) < __builtin_inff()))) return true;
#pragma unroll
        for (int j = 0; j < R; j += 2) {
            lmx = fmax3_abs(lmx, cx.at(j, 0), cx.at(j + 1, 0));
            lmy = fmax3_abs(lmy, cy.at(j, 0), cy.at(j + 1, 0));
        }
        grow(lmx, lmy);
        return false;
    };

    // ---- rows one position at a time ----
    // value of span position d (zero outside the series or when missing)
    auto cell = [&](int d, float& a, float& b) __attribute__((always_inline)) {
        const bool in = inside(d);
        a = span_load<T>(bx, d, in);
        b = span_load<T>(by, d, in);
        const bool m = kFloat && in && missing(a, b);
        a = m ? 0.f : a;
        b = m ? 0.f : b;
        return m ? 1 : 0;
    };
    // The sums before each lane's positions, for a row that is not row_ok; or
    // (`done`) once more for one that fast_row has been through, whose carry
    // is the next row's already (taken back here rather than kept: it would
    // cost the registers of the common case).
    auto edge_sums = [&](const int rrel, bool done, Ch& S, int& miss) __attribute__((always_inline)) {
        const int d0 = rrel + lane * R;
        if (RING && !done) {
            // later rows read their leaving values from the ring
#pragma unroll 4
            for (int j = 0; j < R; j++) {
                const bool in = inside(d0 + j);
                ring[j * rg + wrap(rbase + lane)] = make_float2(span_load<T>(bx, d0 + j, in), span_load<T>(by, d0 + j, in));
            }
        }
        Ch tot = Ch{0, 0, 0, 0, 0};
        int tm = 0;
        bool seen = false;
        float lmx = 0.f, lmy = 0.f;
#pragma unroll 4
        for (int j = 0; j < R; j++) {
            float a, b, ao, bo;
            const int m = cell(d0 + j, a, b), mo = cell(d0 + j - k, ao, bo);
            tm += m - mo;
            seen |= m != 0;
            lmx = fmaxf(lmx, __builtin_fabsf(a));
            lmy = fmaxf(lmy, __builtin_fabsf(b));
            tot = ch_step(tot, a, b, ao, bo);
        }
        if constexpr (kFloat) {
            grow(lmx, lmy);
            if (__builtin_amdgcn_ballot_w64(seen)) dirty_end = rrel + kRow1 + k;
        }
        const Ch inc = ch_scan(tot), row = ch_lane63(inc);
        const int im = wave_incl_scan(tm), rowm = lane63(im);
        if (done) {
            S = (carry - row) + (inc - tot);
            miss = cmiss - rowm + (im - tm);
        } else {
            S = carry + (inc - tot);
            miss = cmiss + (im - tm);
            carry = carry + row;
            cmiss += rowm;
        }
    };
    // The output, if any, whose window ends at span position d: sums S, `miss`
    // missing values.
    auto settle = [&](const int d, const Ch& S, int miss) __attribute__((always_inline)) {
        const int qs = d - kal;                                 // = (p - p_first) * s
        if (d > d_end || (!STEP1 && qs % pstep != 0)) return;
        const int lo = d - k + 1;
        const int clo = max(lo, dmin), chi = min(d, nlim - 1);
        uint32_t fl = 0;
        float cv = g.invalid;
        if (fill && (lo < dmin || d >= nlim)) {
            fl = FL_BORDER;
        } else if (kFloat && miss > 0) {
            fl = FL_MISSING;
        } else {
            double Nn, Vx, Vy;
            nvv(S, (double)(chi - clo + 1), Nn, Vx, Vy);
            if constexpr (kFloat) {
                if ((Vx > gx) & (Vy > gy) & !force) {
                    cv = clamp_unit(newton_ratio(Nn, Vx * Vy));
                } else {
                    float c2 = 0.f;
                    fl = twopass_window((const float*)g.x, (const float*)g.y, 0, 0, 0, 0, 0, 0,
                                        e_base + clo, e_base + chi, &c2);
                    cv = fl ? g.invalid : c2;
                }
            } else {
                fl = (Vx == 0.0 ? FL_ZVAR_X : 0u) | (Vy == 0.0 ? FL_ZVAR_Y : 0u);
                if (!fl) cv = rn32_certified(Nn, Vx, Vy, force);
            }
        }
        const uint32_t o = (uint32_t)(STEP1 ? qs : qs / pstep);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(cv), rc, o * 4u, 0, 0);
        if (has_flags) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)fl, rf, o, 0, 0);
    };
    auto one_by_one = [&](const int rrel, Ch S, int miss) __attribute__((always_inline)) {
#pragma unroll 1
        for (int j = 0; j < R; j++) {
            const int d = rrel + lane * R + j;
            float a, b, ao, bo;
            const int m = cell(d, a, b), mo = cell(d - k, ao, bo);
            miss += m - mo;
            S = ch_step(S, a, b, ao, bo);
            settle(d, S, miss);
        }
    };
    if constexpr (EDGE) {
        const int d0 = kal + lane * R;
        float a[R], b[R], ao[R], bo[R];
        int dm[R];
#pragma unroll
        for (int j = 0; j < R; j++) {
            const bool in = inside(d0 + j), ino = inside(d0 + j - k);
            a[j] = span_load<T>(bx, d0 + j, in);
            b[j] = span_load<T>(by, d0 + j, in);
            ao[j] = span_load<T>(bx, d0 + j - k, ino);
            bo[j] = span_load<T>(by, d0 + j - k, ino);
        }
        Ch tot = Ch{0, 0, 0, 0, 0};
        int tm = 0;
        float lmx = 0.f, lmy = 0.f;
#pragma unroll
        for (int j = 0; j < R; j++) {
            dm[j] = 0;
            if constexpr (kFloat) {
                const bool m = inside(d0 + j) && missing(a[j], b[j]);
                const bool mo = inside(d0 + j - k) && missing(ao[j], bo[j]);
                a[j] = m ? 0.f : a[j];
                b[j] = m ? 0.f : b[j];
                ao[j] = mo ? 0.f : ao[j];
                bo[j] = mo ? 0.f : bo[j];
                dm[j] = (m ? 1 : 0) - (mo ? 1 : 0);
                tm += dm[j];
                lmx = fmaxf(lmx, __builtin_fabsf(a[j]));
                lmy = fmaxf(lmy, __builtin_fabsf(b[j]));
            }
            tot = ch_step(tot, a[j], b[j], ao[j], bo[j]);
        }
        if constexpr (kFloat) grow(lmx, lmy);
        Ch S = carry + (ch_scan(tot) - tot);
        int miss = cmiss + (wave_incl_scan(tm) - tm);
#pragma unroll
        for (int j = 0; j < R; j++) {
            S = ch_step(S, a[j], b[j], ao[j], bo[j]);
            miss += dm[j];
            settle(d0 + j, S, miss);
        }
        return;
    }

    bool loaded = false;             // cx, cy hold the row's cells
    for (int rrel = kal; rrel <= d_end; rrel += kRow1) {
        const bool ok = row_ok(rrel);
        bool redo = true;
        if (ok) {
            if (!loaded) {
                cx.load(bx, rrel + lane * R);
                cy.load(by, rrel + lane * R);
            }
            redo = screen(rrel) ? fast_row(rrel, std::true_type{}) : fast_row(rrel, std::false_type{});
        }
        loaded = ok && row_ok(rrel + kRow1);
        if (redo) {
            // (a row stored by fast_row is stored again, after those stores)
            if (ok) __builtin_amdgcn_s_waitcnt(0);
            Ch S;
            int miss;
            edge_sums(rrel, ok, S, miss);
            one_by_one(rrel, S, miss);
        }
        if constexpr (RING) {
            wave_lds_sync();         // the next row's writes must not pass this row's reads
            rbase = wrap(rbase + kWave);
        }
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

bool cfg_ok_1d(const swc_problem& p, const LaunchCfg& L)
{
    const int mode = mode_of(p.dtype, p.accum);
    if (mode != MODE_U8 && mode != MODE_U16 && mode != MODE_F64) return false;
    if (!(L.wpb == 1 || L.wpb == 2 || L.wpb == 4)) return false;
    if (L.TH < 1 || L.TH > (1 << 16)) return false;
    return L.R == 8;       // rows of the launch parameters are 512 positions
}

template <int M, bool STEP1>
static hipError_t go1d(const P1D& g, int grid, int wpb, hipStream_t s)
{
    if (g.ring_g > 0) {
        const size_t smem = (size_t)wpb * kR1 * g.ring_g * sizeof(float2);
        return launch_kernel(&corr1d_kernel<M, true, STEP1>, dim3(grid), dim3(wpb * kWave), smem, s, g);
    }
    if (g.edge)
        return launch_kernel(&corr1d_kernel<M, false, STEP1, true>, dim3(grid), dim3(wpb * kWave), 0, s, g);
    return launch_kernel(&corr1d_kernel<M, false, STEP1>, dim3(grid), dim3(wpb * kWave), 0, s, g);
}
template <int M> static hipError_t go1d(const P1D& g, int grid, int wpb, hipStream_t s)
{
    return g.s == 1 ? go1d<M, true>(g, grid, wpb, s) : go1d<M, false>(g, grid, wpb, s);
}

hipError_t launch_corr1d(const swc_problem& p, const int64_t* oshape, const LaunchCfg& L,
                         const void* x, const void* y, float* c, uint8_t* flags,
                         hipStream_t s, int force)
{
    const int mode = mode_of(p.dtype, p.accum);
    P1D g;
    g.x = x;
    g.y = y;
    g.c = c;
    g.flags = flags;
    g.N = p.shape[0];
    g.ON = oshape[0];
    g.k = p.window[0];
    g.s = p.step[0];
    g.off = window_offset(p.border, g.k);
    g.border = p.border;
    g.invalid = p.invalid_value;
    g.miss_thr = missing_threshold(p.missing_le);
    g.force = force;
    // A series of no more rows than CUs: one row per wave, one wave per CU (debug
    // bits 1 and 2: the other forms).  Up to there the row-wise loads of a wave,
    // R cells apart between lanes, cost less than the loads one after another of
    // the rows at the ends (float, k = 301, 63 rows 11.7 -> 6.9 us; four waves to a
    // CU 13.6).
    const int64_t rows = (g.ON * g.s + kRow1 - 1) / kRow1;
    g.edge = rows <= (int64_t)device_cus() && !(force & 6);
    // LDS ring of the leaving values: groups of R positions covering k + one
    // row, at most 32 KB per wave (else re-read)
    g.ring_g = 0;
    if (!g.edge) {
        const int64_t rg = ((int64_t)g.k + kRow1 + kR1 - 1) / kR1;
        if (rg * kR1 * (int64_t)sizeof(float2) <= 32 * 1024 && !(force & 4)) g.ring_g = (int)rg;
    }
    const int64_t ring_bytes = (int64_t)kR1 * g.ring_g * (int64_t)sizeof(float2);
    int wpb = g.edge ? 1 : L.wpb;
    while (wpb > 1 && wpb * ring_bytes > 64 * 1024) wpb /= 2;
    // outputs per wave: whole rows, at most TH rows of 512 window ends, fewer
    // when the series is short, so that its waves fill the GPU before any of
    // them takes a second row, and so that the last round of waves is a full
    // one (2^28 floats, k = 5: 1000 -> 883 us)
    const int min_waves = mode != MODE_F64 ? corr1d_min_waves<MODE_U16, true, true>()
                          : (g.ring_g && g.s == 1 ? corr1d_min_waves<MODE_F64, true, true>()
                                                  : corr1d_min_waves<MODE_F64, true, false>());
    const int64_t slots = (int64_t)device_cus() * series_waves(min_waves, ring_bytes, wpb);
    const int64_t rounds = std::max<int64_t>(1, (rows + slots * L.TH - 1) / (slots * L.TH));
    const int64_t per_wave = std::max<int64_t>(1, (rows + slots * rounds - 1) / (slots * rounds));
    g.seg = std::max<int64_t>(1, per_wave * kRow1 / g.s);
    g.n_waves = (g.ON + g.seg - 1) / g.seg;
    g.vst = ((uintptr_t)c % 16 == 0 ? 1 : 0) | ((uintptr_t)flags % 4 == 0 ? 2 : 0);
    const double nrows = (double)(g.seg * g.s) / kRow1 + 1.0;
    const double chain = 2.0 * (double)(g.seg * g.s + g.k) + 16.0 * nrows + 64.0;
    g.cert_g = cert_factor(mode, (double)g.k, chain, (double)g.k + 3.0);
    const int64_t grid64 = (g.n_waves + wpb - 1) / wpb;
    if (grid64 >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    switch (mode) {
    case MODE_U8: return go1d<MODE_U8>(g, (int)grid64, wpb, s);
    case MODE_U16: return go1d<MODE_U16>(g, (int)grid64, wpb, s);
    default: return go1d<MODE_F64>(g, (int)grid64, wpb, s);
    }
}

}  // namespace swc
