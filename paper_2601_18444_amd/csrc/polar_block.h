// Device building block of the polar-detector sums (Sec. 3.2 (q, theta) grid) on the
// FP64 matrix cores.
//
// S_c(q_i, theta_m) = sum_j w_{j,c} exp(-i q_i u_m(j)),  u_m = Y sin(theta_m) + Z cos(theta_m).
// The phase does not separate over the detector, but at one theta the q rows do: with
// blocks of 32 rows, row 32 a + 15.5 +- (b + 1/2) of block a has the phasor
// exp(-i c_a u) exp(-+ i (b + 1/2) dq u), so the sums of a column are the same four
// real contractions over points as a Cartesian cell's (cartesian_block.h) with the block
// centres c_a in the place of |q_M| and the 16 offsets in that of |q_N|: two real
// multiply-adds per term and channel (one where theta + pi is a column too and is
// filled in as the conjugate), against the ten vector FP64 operations of a walk along q.
//
// A wave owns one theta column and one group of `na` row blocks (at most 16, all
// channels), and works alone: tables of a chunk of 32 points go through its own LDS,
// without workgroup barriers.  What bounds it is the FP64 pipe, which matrix and vector
// instructions share; the tables cost one sincos per (point, column), products and
// two-term recurrences x_{k+1} = 2 cos(step) x_k - x_{k-1} of at most 8 (offsets) and 16
// (centres) steps:
//   the first half of the lanes (one lane per point) starts from exp(-i dq u / 2) and
//   walks up 8 offsets, the second from exp(-i 15.5 dq u), which is also the centre of
//   block 0, and walks down 8; the centre step is 32 dq u = 2 (15.5 dq u) + dq u.
// Every start is a sincos of its own phase, so a phasor carries the rounding of that
// phase, at most 16 times that of the centre step, and the recurrence's.
#pragma once

#include "cartesian_block.h"

namespace numag {
namespace pblk {

using cblk::v4d;
using cblk::Point;

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kChunk = 32;    // points per chunk of a wave
constexpr int kRows = 32;     // q rows per block
constexpr int kMaxNA = 16;    // row blocks per wave

// Accumulators of a wave: MT tiles of 16 x 16 (eight slots, that is row blocks and channels,
// each), or with MT <= 0 1 - MT tiles of 4 x 16 (two slots each), for detectors of so few rows
// that the larger one would hold zeros: 16 x 16 takes 69 cycles of the SIMD's FP64 pipe, 4 x 16
// 20.  (50,000 points, 8 x 181, one channel: 268 -> 169 us; four: 244 -> 210.)
// MT = -2 and -3 are the one and two tiles of a detector of up to 16 rows, a block of 8 offsets:
// the four products of 4 x 4 x 4 of an instruction take these for eight points instead of 16
// offsets for four, half of the products and tables (100,000 points, 16 x 361, four channels:
// 741 -> 509 us, 611 by walking the rows).
template <int MT>
struct Tiles {
    using T = v4d;
    static constexpr int N = MT, kSlots = 8, kOffsets = 16;
};
template <>
struct Tiles<0> {
    using T = double;
    static constexpr int N = 1, kSlots = 2, kOffsets = 16;
};
template <>
struct Tiles<-1> {
    using T = double;
    static constexpr int N = 2, kSlots = 2, kOffsets = 16;
};
template <>
struct Tiles<-2> {
    using T = double;
    static constexpr int N = 1, kSlots = 2, kOffsets = 8;
};
template <>
struct Tiles<-3> {
    using T = double;
    static constexpr int N = 2, kSlots = 2, kOffsets = 8;
};
// Tiles of 4 x 16 of a wave.
__host__ __device__ constexpr int few_tiles(int mt) { return mt == 0 || mt == -2 ? 1 : 2; }
__device__ __forceinline__ v4d mfma(double a, double b, v4d c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ double mfma(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Row blocks a wave holds.
template <int MT, int CH>
constexpr int max_na()
{
    constexpr int n = Tiles<MT>::kOffsets == 8 ? 1 : Tiles<MT>::kSlots * Tiles<MT>::N / CH;
    return n < kMaxNA ? n : kMaxNA;
}

// NW weights per point: CH, or 2 CH for pairs of points at u and -u (accumulate below).
template <int MT, int CH, int NW = CH>
struct WaveSmem {
    double2 off[kChunk][Tiles<MT>::kOffsets + 1];
    static constexpr int kCtr = max_na<MT, CH>() == 1 ? 1 : max_na<MT, CH>() + 1;
    double2 ctr[kChunk][kCtr];
    double w[kChunk][NW + 1];
};

// Value of v in the other half of the wave (lane ^ 32).
__device__ __forceinline__ double other_half(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __shfl_xor((int)b, 32), hi = __shfl_xor((int)(b >> 32), 32);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// x_{k+1} = k2 x_k - x_{k-1} for both parts.
__device__ __forceinline__ double2 next_term(double k2, double2 x, double2 before)
{
    return make_double2(fma(k2, x.x, -before.x), fma(k2, x.y, -before.y));
}

// Offset phasors of point gp = lane % 32 at u, M = 16 or 8 of them, written to off[gp]; returns,
// in the second half of the lanes, the centre of block 0 (exp(-i (M - 1/2) dq u)) and the
// centre step.
template <int M>
__device__ __forceinline__ void offsets(double2 (*off)[M + 1], double dq, double u, double2 &centre, double2 &step)
{
    const int lane = threadIdx.x & 63, half = lane >> 5, gp = lane & 31;
    double2 x = phasor(half_turns((half == 0 ? 0.5 : M - 0.5) * dq), u, fabs(u) < phasor_range(M * dq));
    centre = x;
    double2 st = cmul(x, x);  // dq u in the first half
    const double2 so = make_double2(other_half(st.x), other_half(st.y));
    if (half != 0) st = make_double2(so.x, -so.y);  // the second half walks down
    const double k2 = st.x + st.x;
    const int at = half == 0 ? 0 : M - 1, by = half == 0 ? 1 : -1;
    double2 y = cmul(x, st);
    off[gp][at] = x;
    off[gp][at + by] = y;
#pragma unroll
    for (int k = 2; k < M / 2; ++k) {
        const double2 z = next_term(k2, y, x);
        off[gp][at + by * k] = z;
        x = y;
        y = z;
    }
    step = cmul(cmul(centre, centre), so);
}

// N centres from a on, written to ctr[gp] by the second half of the lanes.  Every one the
// tiles have room for: those beyond the row blocks are never used, and the unrolled
// walk takes three instructions an entry.
template <int N>
__device__ __forceinline__ void centres(double2 *ctr, double2 a, double2 step)
{
    const double k2 = step.x + step.x;
    double2 b = cmul(a, step);
    ctr[0] = a;
    if (N > 1) ctr[1] = b;
#pragma unroll
    for (int k = 2; k < N; ++k) {
        const double2 c = next_term(k2, b, a);
        ctr[k] = c;
        a = b;
        b = c;
    }
}

// Tables of a chunk: point gp = lane % 32 of the wave at u, weights p.w, centres of the
// row blocks from a0 on.
template <int MT, int CH, int NW>
__device__ __forceinline__ void generate(WaveSmem<MT, CH, NW> &sm, int a0, double dq, double u, const Point<NW> &p)
{
    const int lane = threadIdx.x & 63, half = lane >> 5, gp = lane & 31;
    double2 centre, step, first = make_double2(1.0, 0.0);
    offsets<Tiles<MT>::kOffsets>(sm.off, dq, u, centre, step);
    if (a0 != 0) {  // wave-uniform
        const double q = (double)(kRows * a0) * dq;
        first = phasor(half_turns(q), u, fabs(u) < phasor_range(q));
    }
    if (half != 0) {
        if (a0 != 0) centre = cmul(centre, first);
        centres<max_na<MT, CH>()>(sm.ctr[gp], centre, step);
    } else {
#pragma unroll
        for (int c = 0; c < NW; ++c) sm.w[gp][c] = p.w[c];
    }
}

// Adds the points [jbeg, jend) of `ld` (the loader concept of cartesian_block.h with
// m = Y, n = Z) to the wave's tiles: theta direction (sth, cth), row blocks from a0 on.
//
// With 2 CH weights a point stands for a pair at u and -u with weights f+ and f-: given
// f+ + f- (even entries) and f+ - f- (odd ones),
//   f+ exp(-i q u) + f- exp(i q u) = (f+ + f-) cos(q u) - i (f+ - f-) sin(q u),
// so RR and II, which make up the real parts, take the first, RI and IR the second.
template <int MT, int CH, int NW, class Loader>
__device__ __forceinline__ void accumulate(const Loader &ld, int64_t jbeg, int64_t jend, double sth, double cth,
                                           double dq, int a0, WaveSmem<MT, CH, NW> &sm,
                                           typename Tiles<MT>::T (&accC)[Tiles<MT>::N],
                                           typename Tiles<MT>::T (&accS)[Tiles<MT>::N])
{
    const int lane = threadIdx.x & 63, gp = lane & 31;
    const int r16 = lane & 15, kq = lane >> 4;
    constexpr bool kPairs = NW != CH;
    static_assert(NW == CH || NW == 2 * CH, "one weight per channel, or two of a pair");
    constexpr int N = Tiles<MT>::N, kOff = Tiles<MT>::kOffsets;
    constexpr int kLog = kOff == 8 ? 3 : 2, kPoints = 1 << kLog;  // points of a matrix step
    const int pt = kOff == 8 ? kq + 4 * (r16 >> 3) : kq;
    // this lane's matrix row: slot 8 t + 4 (r16 / 8) + r16 % 4, part (r16 / 4) % 2 of 16 rows;
    // slot 2 t + r16 % 2, part (r16 / 2) % 2 of four
    const int part = (r16 >> (MT > 0 ? 2 : 1)) & 1;
    // weight of tile t: the same in every tile unless the slots of a tile are no multiple of CH
    constexpr bool kEach = CH == 3 || (MT <= 0 && CH > 2);
    int ea[N], wc[N];
#pragma unroll
    for (int t = 0; t < N; ++t) {
        const int s = MT > 0 ? 8 * t + 4 * (r16 >> 3) + (r16 & 3) : 2 * t + (r16 & 1);
        ea[t] = min(s / CH, max_na<MT, CH>() - 1);
        wc[t] = s % CH;
    }
    auto fetch = [&](int64_t j0) {
        typename Loader::Raw r{};
        if (j0 + gp < jend) r = ld.raw(j0 + gp);
        return r;
    };
    typename Loader::Raw raw = fetch(jbeg);
#pragma unroll 1
    for (int64_t j0 = jbeg; j0 < jend; j0 += kChunk) {
        const Point<NW> p = ld.point(raw);
        const double u = p.m * sth + p.n * cth;
        // A wave that builds tables goes first: its short instructions otherwise wait for a
        // matrix instruction of the SIMD's other wave each, and both end up building at the
        // same time (100,003 points, 256 x 360: 1.39 -> 1.33 ms).
        __builtin_amdgcn_s_setprio(2);
        generate<MT, CH, NW>(sm, a0, dq, u, p);
        wave_fence();
        __builtin_amdgcn_s_setprio(0);
        raw = fetch(j0 + kChunk);
        const int steps = __builtin_amdgcn_readfirstlane((int)((min((int64_t)kChunk, jend - j0) + kPoints - 1) >> kLog));
        const double2 *op = &sm.off[pt][r16 & (kOff - 1)], *cp = &sm.ctr[pt][0];
        const double *wp = &sm.w[pt][0];
        auto step = [&](int s) {
            const double2 z = op[s * kPoints * (kOff + 1)];
            const double *c = (const double *)(cp + s * kPoints * WaveSmem<MT, CH, NW>::kCtr) + part;
            const double *w = wp + s * kPoints * (NW + 1);
            double a[N], b[kPairs ? N : 1];
            if (kPairs) {
#pragma unroll
                for (int t = 0; t < N; ++t) {
                    const double y = c[2 * ea[t]];
                    a[t] = y * w[2 * wc[kEach ? t : 0] + part];
                    b[t] = y * w[2 * wc[kEach ? t : 0] + 1 - part];
                }
            } else if (kEach) {
#pragma unroll
                for (int t = 0; t < N; ++t) a[t] = c[2 * ea[t]] * w[wc[t]];
            } else {
                const double w0 = w[wc[0]];
#pragma unroll
                for (int t = 0; t < N; ++t) a[t] = c[2 * ea[t]] * w0;
            }
#pragma unroll
            for (int t = 0; t < N; ++t) {
                accC[t] = mfma(a[t], z.x, accC[t]);
                accS[t] = mfma(kPairs ? b[t] : a[t], z.y, accS[t]);
            }
        };
        int s = 0;
        for (; s + 4 <= steps; s += 4) {
            step(s);
            step(s + 1);
            step(s + 2);
            step(s + 3);
        }
        for (; s < steps; ++s) step(s);
        wave_fence();
    }
    if constexpr (kOff == 8) {  // the two sets of points
#pragma unroll
        for (int t = 0; t < N; ++t) {
            accC[t] += __shfl_xor(accC[t], 8);
            accS[t] += __shfl_xor(accS[t], 8);
        }
    }
}

// The sums of tile t of 4 x 16 in this lane: slot 2 t + (lane / 16) % 2, offset lane % 16, the
// first row (lane < 32, which hold RR and RI) or the second (IR and II).
__device__ __forceinline__ double2 few_rows(double c, double s)
{
    const double oc = other_half(c), os = other_half(s);
    return (threadIdx.x & 32) == 0 ? make_double2(c - os, s + oc) : make_double2(oc + s, c - os);
}

// Offset of a lane's sums; of 8 offsets the second half of the lanes of 16 repeat the first,
// and have no row.
__device__ __forceinline__ int lane_offset(const PolGeom &g)
{
    const int b = threadIdx.x & 15;
    return b < g.mid ? b : (1 << 29);
}

// Rows of block a, offset b: 32 a + mid + b (k = 0) and 32 a + mid - 1 - b (k = 1).  Negative or
// beyond the detector: none.
__device__ __forceinline__ int slot_row(const PolGeom &g, int rg, int e, int b, int k)
{
    const int a = kRows * (rg * g.na + e);
    return k == 0 ? a + g.mid + b : a + g.mid - 1 - b;
}

// Writes (add: adds) the two rows of slot s, offset b, at the mirrored column too (nh > 0:
// column m + nh holds the conjugates).  which: 1 for the first row, 2 for the second.
__device__ __forceinline__ void put_slot(double *__restrict__ amp, const PolGeom &g, int CH, int rg, int col, int s,
                                         int b, double2 vp, double2 vm, bool add, int which = 3)
{
    const int e = s / CH, c = s - e * CH;
    if (e >= g.na) return;
    const int first = CH == 3 ? 1 : 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int row = slot_row(g, rg, e, b, k);
        if ((unsigned)row >= (unsigned)g.n0 || !(which >> k & 1)) continue;
        const double2 v = k == 0 ? vp : vm;
        const int64_t p = (int64_t)row * g.n_out + col;
        auto put = [&](int ch, double2 x) {
            cblk::put_pixel(amp, p, ch, x.x, x.y, add);
            if (g.nh > 0) cblk::put_pixel(amp, p + g.nh, ch, x.x, -x.y, add);
        };
        put(first + c, v);
        if (c == 0 && !add) {  // channels outside the set
            if (CH == 3) put(0, make_double2(0.0, 0.0));
            if (CH <= 2)
                for (int ch = CH; ch < 4; ++ch) put(ch, make_double2(0.0, 0.0));
        }
    }
}

// Which of a slot's sums are NaN on the detector (1, 2).
__device__ __forceinline__ int which_nan(const PolGeom &g, int CH, int rg, int s, int b, double2 vp, double2 vm)
{
    const int e = s / CH;
    if (e >= g.na) return 0;
    return (is_nan(vp) && (unsigned)slot_row(g, rg, e, b, 0) < (unsigned)g.n0 ? 1 : 0) |
           (is_nan(vm) && (unsigned)slot_row(g, rg, e, b, 1) < (unsigned)g.n0 ? 2 : 0);
}

// A slot's sums vp, vm over the points [j0, j1) of src (nonfinite.h), which of them (1, 2)
// being NaN, at the direction (sth, cth).
__device__ __forceinline__ void repair(const PolGeom &g, const PointSource &src, int64_t j0, int64_t j1, int CH, int rg,
                                       int s, int b, double sth, double cth, int which, double2 &vp, double2 &vm)
{
    const int e = s / CH, ch = s - e * CH + (CH == 3 ? 1 : 0);
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
        if (!(which >> k & 1)) continue;
        const double q = (double)slot_row(g, rg, e, b, k) * g.dq;
        const double2 v = nonfinite_sum(src, j0, j1, ch, q * sth, q * cth, k == 0 ? vp : vm);
        (k == 0 ? vp : vm) = v;
    }
}

}  // namespace pblk
}  // namespace numag
