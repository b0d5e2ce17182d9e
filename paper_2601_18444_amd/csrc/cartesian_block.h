// Device building block of the Cartesian direct sums on the FP64 matrix cores.
//
// The phase separates, exp(-i (q_M m + q_N n)) = exp(-i q_M m) exp(-i q_N n) with m, n
// a point's lab-frame coordinates along the two detector axes (M: the axis whose
// blocks are packed into matrix rows, N: the other), and the detector is symmetric
// about q = 0 on both axes.  So the sums of the four pixels (+-q_M, +-q_N) of one
// cell |q_M|, |q_N| and one channel follow from four real contractions over points,
//   RR = sum w yr zr,  RI = sum w yr zi,  IR = sum w yi zr,  II = sum w yi zi,
// with (yr, yi) = exp(-i |q_M| m) and (zr, zi) = exp(-i |q_N| n):
//   S(+,+) = (RR - II) + i (RI + IR),  S(+,-) = (RR + II) + i (IR - RI),
// and S(-q) = conj S(q) for the other two (real weights).  That is one multiply-add
// per term and channel, four instead of the ten and a half vector FP64 operations a
// pixel-by-pixel walk with a two-term phasor recurrence takes, and it runs on
// v_mfma_f64_16x16x4f64.
//
// The FP64 vector and matrix instructions share one pipe (measured: 74.7 TFLOP/s of
// matrix products alone, 65.3 of vector FMAs alone, and their sum stays at 74.7 when
// a wave issues both), so what is not a matrix product is kept small:
//  - a workgroup of 8 waves owns one block of `na` |q_M| values (all channels; 64 row
//    slots at most) and `nz` blocks of 16 |q_N| values, one per wave; waves beyond the
//    nz blocks take other points of the same chunk (8 / nz groups);
//  - the row operand w_c exp(-i |q_M| m) is formed once per chunk of 32 points for all
//    waves and read from LDS; the column operand is the product of a block's centre
//    phasor and one of 16 offsets exp(-i (b + 1/2) dq n), b = -8 .. 7 (8 sincos, the
//    others are conjugates): one complex product per wave and four points.
// A lane generates for one point (two entries of a 32-point chunk per wave
// instruction), so every sincos lane does useful work; every phasor is a sincos or a
// product of two, which keeps the error at the rounding of the phase itself.
// Chunks are double-buffered: the next chunk is generated while this one is summed, one
// barrier per chunk, its points loaded one chunk ahead of their use.
#pragma once

#include "nonfinite.h"
#include "numag_internal.h"
#include "phasor.h"

namespace numag {
namespace cblk {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kChunk = 32;   // points per LDS chunk
constexpr int kOff = 16;     // |q_N| values per column block
constexpr int kMaxMT = 8;    // 16-row matrix tiles per wave

// First channel of a CH-channel set: 4 (N, Mx, My, Mz), 3 (the magnetic channels, a
// sample without nuclear weights) or 1 (N only).
template <int CH>
__host__ __device__ constexpr int ch_first()
{
    static_assert(CH == 4 || CH == 3 || CH == 1, "channel set");
    return CH == 3 ? 1 : 0;
}

// What a lane needs of its point: coordinates along the two axes and the weights.
template <int CH>
struct Point {
    double m, n;
    double w[CH];
};

// Row slots: slot s = e CH + c is |q_M| value e of the block, channel c.  Its real
// part sits in matrix row 16 (s / 8) + 8 ((s / 4) % 2) + s % 4 and its imaginary part
// four rows further, so that after the contraction one lane holds RR, IR, RI and II
// of a slot (accumulator register r of lane l is row 4 r + l / 16, column l % 16).
__device__ __forceinline__ int slot_row(int s) { return 16 * (s >> 3) + 8 * ((s >> 2) & 1) + (s & 3); }

// The wave's index in its workgroup, known to be uniform (scalar branches and loops:
// a divergent loop around the matrix instructions costs a copy of the accumulators).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

template <int MT>
struct Smem {
    double y[2][kChunk][16 * MT + 1];   // odd row stride: the point-major stores are free of conflicts
    double2 off[2][kChunk][kOff + 1];
    double2 ctr[2][kChunk][kWaves + 1];
    static constexpr int kRed = 8 * 64 * kWaves;  // doubles the epilogue's reduction uses at a time
};
static_assert(sizeof(Smem<1>) >= Smem<1>::kRed * sizeof(double), "the epilogue reduces over the whole buffer");

// Copies the n double2 (a multiple of 64) at src to LDS at dst, 64 of them per wave
// instruction, straight from memory without passing through registers; done for this
// wave's share by wait_copies().
__device__ __forceinline__ void copy_to_lds(const double2 *src, double2 *dst, int n, int waves)
{
    const int lane = threadIdx.x & 63;
    for (int k = 64 * wave_id(); k < n; k += 64 * waves)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + k + lane),
                                         (__attribute__((address_space(3))) void *)(dst + k), 16, 0, 0);
}
__device__ __forceinline__ void wait_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int MT>
__device__ __forceinline__ void zero(v4d (&accC)[MT], v4d (&accS)[MT])
{
#pragma unroll
    for (int t = 0; t < MT; ++t) accC[t] = accS[t] = v4d{0.0, 0.0, 0.0, 0.0};
}

// Loader concept: `Raw raw(int64_t j) const` loads what point j needs from memory, and
// `Point<CH> point(const Raw &) const` makes the point of it, one chunk later.
//
// Adds the points [jbeg, jend) of `ld` to this wave's tiles: row block rb, column block
// zb0 + wave % nz.  accC holds the contractions with zr, accS those with zi.  p and q
// hold the raw points of the first two chunks (first_points).  Ends with a barrier.
template <class Loader>
__device__ __forceinline__ void first_points(const Loader &ld, int64_t jbeg, int64_t jend, typename Loader::Raw &p,
                                             typename Loader::Raw &q)
{
    const int gp = threadIdx.x & 31;
    p = q = typename Loader::Raw{};
    if (jbeg + gp < jend) p = ld.raw(jbeg + gp);
    if (jbeg + kChunk + gp < jend) q = ld.raw(jbeg + kChunk + gp);
}

template <int MT, int CH, class Loader>
__device__ __forceinline__ void accumulate(const Loader &ld, int64_t jbeg, int64_t jend, const CartGeom &g, int rb,
                                           int zb0, Smem<MT> &sm, typename Loader::Raw p, typename Loader::Raw q,
                                           v4d (&accC)[MT], v4d (&accS)[MT])
{
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int half = lane >> 5, gp = lane & 31;  // generation: entry of a pair, point
    const int zi = wave % g.nz, kg = wave / g.nz, nk = kWaves / g.nz;
    const bool active = zb0 + zi < g.nzb;
    const int r16 = lane & 15, kq = lane >> 4;
    // coefficient of this lane's column entry: an offset (first half) or a block centre
    const HalfTurns qn = half_turns(half == 0 ? ((double)wave + 0.5) * g.stepN
                                              : ((double)(kOff * (zb0 + wave)) + g.firstN + 7.5) * g.stepN);
    // (block centres and rows may lie up to a block beyond the detector)
    const double range = phasor_range(fmax((g.A + 16.0 * kMaxMT) * g.stepM, (g.B + 256.0) * g.stepN));

    auto put_row = [&](int b, const Point<CH> &p, int e, double2 y) {
        if (e < g.na) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int row = slot_row(e * CH + c);
                sm.y[b][gp][row] = p.w[c] * y.x;
                sm.y[b][gp][row + 4] = p.w[c] * y.y;
            }
        }
    };
    const HalfTurns qm0 = half_turns(((double)(rb * g.na + 2 * wave + half) + g.firstM) * g.stepM);
    auto generate = [&](int b, const typename Loader::Raw &raw) {
        const Point<CH> p = ld.point(raw);
        const bool fast = fmax(fabs(p.m), fabs(p.n)) < range && p.m == p.m && p.n == p.n;
        double2 z, y;
        phasor2(qn, p.n, qm0, p.m, fast, z, y);
        if (half == 0) {
            sm.off[b][gp][8 + wave] = z;
            sm.off[b][gp][7 - wave] = make_double2(z.x, -z.y);
        } else {
            sm.ctr[b][gp][wave] = z;
        }
        put_row(b, p, 2 * wave + half, y);
#pragma unroll 1
        for (int e0 = 2 * (wave + kWaves); e0 < g.na; e0 += 2 * kWaves) {
            const HalfTurns q = half_turns(((double)(rb * g.na + e0 + half) + g.firstM) * g.stepM);
            put_row(b, p, e0 + half, phasor(q, p.m, fast));
        }
    };
    // point group kg takes 8 / nk consecutive steps of a chunk
    auto sum = [&](int b, int np) {
        const int s0 = kg * (kChunk / 4) / nk;
        const int steps = active ? min((kChunk / 4) / nk, ((np + 3) >> 2) - s0) : 0;
        const double *yp = &sm.y[b][4 * s0 + kq][r16];
        const double2 *cp = &sm.ctr[b][4 * s0 + kq][zi], *op = &sm.off[b][4 * s0 + kq][r16];
        auto step = [&](int s) {
            double a[MT];
#pragma unroll
            for (int t = 0; t < MT; ++t) a[t] = yp[s * 4 * (16 * MT + 1) + 16 * t];
            const double2 z = cmul(cp[s * 4 * (kWaves + 1)], op[s * 4 * (kOff + 1)]);
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                accC[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], z.x, accC[t], 0, 0, 0);
                accS[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], z.y, accS[t], 0, 0, 0);
            }
        };
        // four at a time: the LDS addresses are then offsets of one register
        int s = 0;
        for (; s + 4 <= steps; s += 4) {
            step(s);
            step(s + 1);
            step(s + 2);
            step(s + 3);
        }
        for (; s < steps; ++s) step(s);
    };

    generate(0, p);
    __syncthreads();
    int b = 0;
#pragma unroll 1
    for (int64_t j0 = jbeg; j0 < jend; j0 += kChunk, b ^= 1) {
        if (j0 + kChunk < jend) {
            // q holds the next chunk's points, and takes those of the one after as soon as
            // they are used (handing a second set on by a copy would wait for its load here)
            generate(b ^ 1, q);
            if (j0 + 2 * kChunk + gp < jend) q = ld.raw(j0 + 2 * kChunk + gp);
            else q = typename Loader::Raw{};
        }
        sum(b, (int)min((int64_t)kChunk, jend - j0));
        __syncthreads();
    }
}

// Hands the finished sums to put(t, h, S(+,+), S(+,-)): slot 8 t + 4 h + lane / 16, column
// lane % 16 of the block.
template <int MT, class Put>
__device__ __forceinline__ void finish_whole(const v4d (&accC)[MT], const v4d (&accS)[MT], const Put &put)
{
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double RR = accC[t][2 * h], IR = accC[t][2 * h + 1], RI = accS[t][2 * h], II = accS[t][2 * h + 1];
            put(t, h, make_double2(RR - II, RI + IR), make_double2(RR + II, IR - RI));
        }
}

// The same with several point groups, which are first added, in a fixed order, through LDS
// (one tile at a time; group k < 2 then puts half k): every wave of the workgroup has to
// call this.
template <int MT, class Put>
__device__ __forceinline__ void finish_groups(const CartGeom &g, int zb0, Smem<MT> &sm, const v4d (&accC)[MT],
                                              const v4d (&accS)[MT], const Put &put)
{
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int zi = wave % g.nz, kg = wave / g.nz, nk = kWaves / g.nz;
    const bool active = zb0 + zi < g.nzb;
    double *red = (double *)&sm;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            red[(wave * 8 + r) * 64 + lane] = accC[t][r];
            red[(wave * 8 + 4 + r) * 64 + lane] = accS[t][r];
        }
        __syncthreads();
        if (active && kg < 2) {
            double v[4] = {0.0, 0.0, 0.0, 0.0};
            for (int k = 0; k < nk; ++k) {
                const double *p = red + (k * g.nz + zi) * 512 + lane;
                v[0] += p[(2 * kg) * 64];
                v[1] += p[(2 * kg + 1) * 64];
                v[2] += p[(4 + 2 * kg) * 64];
                v[3] += p[(5 + 2 * kg) * 64];
            }
            put(t, kg, make_double2(v[0] - v[3], v[2] + v[1]), make_double2(v[0] + v[3], v[1] - v[2]));
        }
        __syncthreads();
    }
}

// Whichever of the two the launch shape needs.
template <int MT, class Put>
__device__ __forceinline__ void finish(const CartGeom &g, int zb0, Smem<MT> &sm, const v4d (&accC)[MT],
                                       const v4d (&accS)[MT], const Put &put)
{
    if (g.nz != kWaves)
        finish_groups<MT>(g, zb0, sm, accC, accS, put);
    else if (zb0 + wave_id() < g.nzb)
        finish_whole<MT>(accC, accS, put);
}

// The pixels +-|q| of a cell's slot on the two axes.
struct CellPixels {
    bool ok, twoM, twoN;      // slot on the detector; distinct mirrors on each axis
    int c;                    // channel within the set
    int64_t pp, pm, mp, mm;   // pixel (+,+), (+,-), (-,+), (-,-)
};

__device__ __forceinline__ CellPixels cell_pixels(const CartGeom &g, int CH, int rb, int zb, int s, int col)
{
    CellPixels x;
    const int e = s / CH;
    x.c = s - e * CH;
    const int a = rb * g.na + e, b = kOff * zb + col;
    x.ok = e < g.na && a < g.A && b < g.B;
    const int ip = g.nM - g.A + a, im = g.A - 1 - a, jp = g.nN - g.B + b, jm = g.B - 1 - b;
    x.twoM = ip != im;
    x.twoN = jp != jm;
    x.pp = ip * g.strideM + jp * g.strideN;
    x.pm = ip * g.strideM + jm * g.strideN;
    x.mp = im * g.strideM + jp * g.strideN;
    x.mm = im * g.strideM + jm * g.strideN;
    return x;
}

// Writes (add: adds) one channel of the four pixels of a cell; v = S(+,+), S(+,-).
__device__ __forceinline__ void put_pixel(double *__restrict__ amp, int64_t p, int ch, double re, double im, bool add)
{
    double *o = amp + p * 8 + 2 * ch;
    o[0] = add ? o[0] + re : re;
    o[1] = add ? o[1] + im : im;
}

// which: 1 for S(+,+) and its mirror, 2 for S(+,-), 3 for both.
__device__ __forceinline__ void put_cell(double *__restrict__ amp, const CellPixels &x, int ch, double2 vp, double2 vm,
                                         bool add, int which = 3)
{
    if (which & 1) put_pixel(amp, x.pp, ch, vp.x, vp.y, add);
    if (x.twoN && (which & 2)) put_pixel(amp, x.pm, ch, vm.x, vm.y, add);
    if (x.twoM) {
        if (which & 1) put_pixel(amp, x.mm, ch, vp.x, -vp.y, add);
        if (x.twoN && (which & 2)) put_pixel(amp, x.mp, ch, vm.x, -vm.y, add);
    }
}

// A slot's channel and, from the lane that holds its first channel, the exact zeros
// of the channels outside the set.
__device__ __forceinline__ void put_slot(double *__restrict__ amp, const CellPixels &x, int CH, double2 vp, double2 vm,
                                         bool add, int which = 3)
{
    const int first = CH == 3 ? 1 : 0;
    put_cell(amp, x, first + x.c, vp, vm, add, which);
    if (x.c == 0 && !add) {
        const double2 o = make_double2(0.0, 0.0);
        if (CH == 3) put_cell(amp, x, 0, o, o, false);
        if (CH == 1)
            for (int ch = 1; ch < 4; ++ch) put_cell(amp, x, ch, o, o, false);
    }
}

// A slot's sums vp, vm over the points [j0, j1) of src (nonfinite.h), which of them (1, 2)
// being NaN: |q_M| value a, |q_N| value b, channel ch.
__device__ __forceinline__ void repair(const CartGeom &g, const PointSource &src, int64_t j0, int64_t j1, int a, int b,
                                       int ch, int which, double2 &vp, double2 &vm)
{
    const double qm = ((double)a + g.firstM) * g.stepM, qn = ((double)b + g.firstN) * g.stepN;
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
        if (!(which >> k & 1)) continue;
        const double q = k == 0 ? qn : -qn;
        const double2 v = nonfinite_sum(src, j0, j1, ch, g.swapped ? q : qm, g.swapped ? qm : q, k == 0 ? vp : vm);
        (k == 0 ? vp : vm) = v;
    }
}

__device__ __forceinline__ int which_nan(double2 vp, double2 vm) { return (is_nan(vp) ? 1 : 0) | (is_nan(vm) ? 2 : 0); }

}  // namespace cblk
}  // namespace numag
