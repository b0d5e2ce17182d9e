// Objects and orientations on gfx950 (Sec. 3.3 summation relation and dilute
// approximation; Sec. 3.1 sample rotation, extended to many orientations).
//
// Dilute and split modes need each object's amplitude F_k complete before its
// outer product F_k F_k^H is formed, so sums are not split over point ranges
// here.  The work is cut into accumulator slots: a slot is a set of objects
// (one object, or a contiguous group of roughly equal point count) and a range
// of rotations, sized so that every slot costs about the same; a large particle
// gets many rotation ranges, a small one a single range.  A work item is
// (slot, pixel block): every point of the slot's objects is summed for every rotation
// of its range with the matrix building blocks of the direct sums, then F F^H (and,
// in split mode, exp(-i q.R r^k) F for the coherent total) goes into the slot's FP64
// accumulators, which no other item touches.  Items are sorted by cost and handed out by
// a persistent kernel through an atomic counter (small polar ones in order) -- to
// workgroups of 8 waves on a Cartesian detector (cartesian_block.h), to single waves on a
// polar one (polar_block.h); slots are reduced in a fixed order, so results are reproducible
// bit for bit.
//
// Rotations are applied on the fly (X = R x, w' = (n, R m)) while a chunk's
// phasors are generated, so the point data is read once per chunk and never
// rewritten per orientation; the first points of the next object are loaded before
// the products of the current one.
//
// Accumulators hold only the independent half of the pixels (G(-q) = conj G(q) for
// real weights), in strips of sixteen (the columns of a |q_N| block at one |q_M| value and
// sign, or sixteen q rows of a theta column) in the order the lanes hold them: lane l has
// channel g = l / 16 of the strip's pixels, takes the other channels from lanes
// l ^ 16, 32, 48 and keeps four of the sixteen reals of G (kPacked), so that every access is
// a coalesced wave-wide row; the reduction puts them into pixel order.
//
// Measured, kernel time before (10.5 vector FP64 instructions per term over every pixel)
// and now: 16 particles (96,000 points) x 24 rotations, 128 x 128: 14.2 -> 5.70 ms (4.04 of
// it multiply-adds at 74.7 TFLOP/s); 96 objects (240,000 points) split, 256 x 256: 6.19 -> 2.50 ms
// (1.68; the largest object's items run alone at the end).
//
// The eight tiles of accumulators and an object's epilogue (F F^H, object phases) do not fit
// 256 registers: the compiler spills 98 in objects_kernel<8> and 94 in objects_polar_kernel<8>
// (fewer with fewer tiles, none up to three), outside the matrix loop, so that they cost once
// per object and rotation and count on small objects.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <vector>

#include "cartesian_block.h"
#include "polar_block.h"

namespace numag {

namespace {

__device__ __forceinline__ double uniform(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ Rot uniform_rot(const double *p)
{
    Rot R;
#pragma unroll
    for (int i = 0; i < 9; ++i) R.m[i] = uniform(p[i]);
    return R;
}

// Points of the sample rotated by R (the axes swapped for a transposed Cartesian grid).
struct RotLoader {
    struct Raw {
        double x[3], n, m[3];
    };
    const double *__restrict__ pos, *__restrict__ nuc, *__restrict__ mag;
    Rot R;
    int swapped;
    __device__ __forceinline__ Raw raw(int64_t j) const
    {
        Raw r{};
#pragma unroll
        for (int i = 0; i < 3; ++i) r.x[i] = pos[3 * j + i];
        if (nuc != nullptr) r.n = nuc[j];
        if (mag != nullptr) {
#pragma unroll
            for (int i = 0; i < 3; ++i) r.m[i] = mag[3 * j + i];
        }
        return r;
    }
    __device__ __forceinline__ cblk::Point<4> point(const Raw &r) const
    {
        cblk::Point<4> p;
        const double Y = R.m[3] * r.x[0] + R.m[4] * r.x[1] + R.m[5] * r.x[2];
        const double Z = R.m[6] * r.x[0] + R.m[7] * r.x[1] + R.m[8] * r.x[2];
        p.m = swapped ? Z : Y;
        p.n = swapped ? Y : Z;
        p.w[0] = r.n;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            p.w[1 + i] = R.m[3 * i] * r.m[0] + R.m[3 * i + 1] * r.m[1] + R.m[3 * i + 2] * r.m[2];
        return p;
    }
};

struct ObjArgs {
    const unsigned long long *tag_ptr;  // the plan tag at the start of the workspace
    unsigned long long tag;             // the tag of the plan these tables belong to
    const double *pos, *nuc, *mag;
    const int64_t *off;      // [K+1]
    const double *obj_pos;   // [K][3] or null
    const double *rot;       // [n_rot][9]
    const int2 *items;       // (slot, pixel block), sorted by cost
    const int4 *slots;       // (object lo, object hi, rotation lo, rotation hi)
    int n_items;
    int *counter;
    double *spec;            // [n_slots][strips][4][64]
    double *amp;             // [n_slots][strips][2][64] or null (split mode)
};

// Strips of a slot: [row block][column block][value of the block][sign], or [column][row
// group][value][half].  Kernels of up to two tiles a wave, on detectors that may fill little of
// them (one row block or group then), pass over the values and halves beyond the detector,
// which take no accumulators: 3000 objects of 20 points on 8 x 40 polar pixels 123 MB of
// workspace instead of 492.  In the larger ones, where they are few, a branch would cost more.
constexpr int kExactTiles = 2;
__host__ __device__ __forceinline__ int block_values(int na, int mt) { return mt <= kExactTiles ? na : 2 * mt; }
__host__ __device__ __forceinline__ int64_t slot_strips(const CartGeom &g, int mt)
{
    return 2 * (int64_t)g.nrb * g.nzb * block_values(g.na, mt);
}
__host__ __device__ __forceinline__ int64_t column_strips(const PolGeom &g, int mt)
{
    return mt <= kExactTiles ? (g.n0 + 15) / 16 : (int64_t)g.nrg * 4 * mt;
}
__host__ __device__ __forceinline__ int64_t slot_strips(const PolGeom &g, int mt) { return g.cols * column_strips(g, mt); }
// Lines of strips: blocks (Cartesian) or columns.
__host__ __device__ __forceinline__ int64_t slot_lines(const CartGeom &g) { return (int64_t)g.nrb * g.nzb; }
__host__ __device__ __forceinline__ int64_t slot_lines(const PolGeom &g) { return g.cols; }

// Entry of the packed spectral matrix that lane group g keeps in row e: its own diagonal
// entry, then one real of the pair (g, g ^ e): the real part in the group of the smaller
// channel, the imaginary part in the other.
__device__ constexpr int kPacked[4][4] = {{0, 4, 6, 8}, {1, 5, 12, 10}, {2, 14, 7, 11}, {3, 15, 13, 9}};

// The four entries of F F^H that a lane keeps.
__device__ __forceinline__ void spectral_part(double2 F, double (&v)[4])
{
    const int g = (threadIdx.x & 63) >> 4;
    v[0] = F.x * F.x + F.y * F.y;
#pragma unroll
    for (int e = 1; e < 4; ++e) {
        const double ox = __shfl_xor(F.x, 16 * e), oy = __shfl_xor(F.y, 16 * e);
        // Re F_a conj(F_b) is symmetric; Im of the smaller channel a (the other lane's)
        // with b (this one's) is a_i b_r - a_r b_i
        v[e] = g < (g ^ e) ? F.x * ox + F.y * oy : oy * F.x - ox * F.y;
    }
}

// Adds (first: writes) F F^H to the lane's four accumulators o[64 e].
__device__ __forceinline__ void add_spectral(double *__restrict__ o, bool first, double2 F)
{
    double v[4];
    spectral_part(F, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[64 * e] = first ? v[e] : o[64 * e] + v[e];
}

// Adds (first: writes) one channel of a pixel times the object's phasor y z.
__device__ __forceinline__ void add_amplitude(double *__restrict__ o, bool first, double2 v, double2 y, double2 z)
{
    const double2 r = cmul(cmul(y, z), v);
    o[0] = first ? r.x : o[0] + r.x;
    o[64] = first ? r.y : o[64] + r.y;
}

// Where the reductions flag results that are not finite, behind the item counter.
constexpr int kNonfinite = 32;

// Lab position (Y, Z) of object k.
__device__ __forceinline__ double2 object_yz(const ObjArgs &a, const double *R, int k)
{
    if (a.obj_pos == nullptr) return make_double2(0.0, 0.0);
    const double *o = a.obj_pos + 3 * (int64_t)k;
    return make_double2(R[3] * o[0] + R[4] * o[1] + R[5] * o[2], R[6] * o[0] + R[7] * o[1] + R[8] * o[2]);
}

template <int MT>
__global__ __launch_bounds__(cblk::kThreads, 2) void objects_kernel(ObjArgs a, CartGeom g)
{
    __shared__ cblk::Smem<MT> sm;
    __shared__ int s_item;
    if (*a.tag_ptr != a.tag) return;  // the workspace does not hold this plan's tables
    const int lane = threadIdx.x & 63;
    const int groups = (g.nzb + g.nz - 1) / g.nz;
    const int64_t strips = slot_strips(g, MT);
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(a.counter, 1);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(s_item);
        __syncthreads();
        if (it >= a.n_items) break;
        const int2 item = a.items[it];
        const int slot = __builtin_amdgcn_readfirstlane(item.x), blk = __builtin_amdgcn_readfirstlane(item.y);
        const int rb = blk / groups, zb0 = (blk % groups) * g.nz;
        const int zb = zb0 + cblk::wave_id() % g.nz;
        const int4 sv = a.slots[slot];
        const int k0 = __builtin_amdgcn_readfirstlane(sv.x), k1 = __builtin_amdgcn_readfirstlane(sv.y);
        const int r0 = __builtin_amdgcn_readfirstlane(sv.z), r1 = __builtin_amdgcn_readfirstlane(sv.w);
        const int64_t strip0 = slot * strips + 2 * ((int64_t)rb * g.nzb + zb) * block_values(g.na, MT);
        RotLoader ld{a.pos, a.nuc, a.mag, uniform_rot(a.rot + 9 * (int64_t)r0), g.swapped};
        RotLoader::Raw p, q;
        cblk::first_points(ld, a.off[k0], a.off[k0 + 1], p, q);
        for (int r = r0; r < r1; ++r) {
            if (r != r0) ld.R = uniform_rot(a.rot + 9 * (int64_t)r);
            for (int k = k0; k < k1; ++k) {
                cblk::v4d accC[MT], accS[MT];
                cblk::zero<MT>(accC, accS);
                cblk::accumulate<MT, 4>(ld, a.off[k], a.off[k + 1], g, rb, zb0, sm, p, q, accC, accS);
                const int kn = k + 1 < k1 ? k + 1 : k0;  // the next object (raw points do not depend on r)
                cblk::first_points(ld, a.off[kn], a.off[kn + 1], p, q);
                const bool first = r == r0 && k == k0;
                double2 z = make_double2(1.0, 0.0);
                double Xm = 0.0;
                if (a.amp != nullptr) {
                    const double2 X = object_yz(a, ld.R.m, k);
                    Xm = g.swapped ? X.y : X.x;
                    z = twiddle(((double)(cblk::kOff * zb + (lane & 15)) + g.firstN) * g.stepN *
                                (g.swapped ? X.x : X.y));
                }
                auto add = [&](int i, double2 vp, double2 vm) {
                    if (MT <= kExactTiles && i >= g.na) return;
                    const int64_t strip = strip0 + 2 * i;
                    double *o = a.spec + strip * 256 + lane;
                    add_spectral(o, first, vp);
                    add_spectral(o + 256, first, vm);
                    if (a.amp != nullptr) {
                        const double qm = ((double)(rb * g.na + i) + g.firstM) * g.stepM;
                        double *u = a.amp + strip * 128 + lane;
                        add_amplitude(u, first, vp, twiddle(qm * Xm), z);
                        add_amplitude(u + 128, first, vm, twiddle(qm * Xm), make_double2(z.x, -z.y));
                    }
                };
                cblk::finish<MT>(g, zb0, sm, accC, accS,
                                 [&](int t, int h, double2 vp, double2 vm) { add(2 * t + h, vp, vm); });
            }
        }
    }
}

// A work item belongs to one wave: (slot, theta column and row group).  MT < 0: detectors
// of one row block, whose four channels are two tiles of 4 x 16 (they half fill a tile of 16
// rows, which takes twice as long: 20 objects of 2,000 points, ten rotations, 16 x 361 pixels
// 3.67 -> 1.98 ms, 2.9 with 16 offsets, 2.64 by walking the rows; 32 x 181 1.79 -> 1.45, 1.62).
//
// Items by the counter, or (TURNS) in order.  (Forms of their own: with both in one kernel the
// sums take 4 % longer, 64 particles x 50 rotations on 128 x 128 305 ms against 293.)
constexpr int kFewRows = -1, kFewestRows = -3;  // (-3: detectors of up to 16 rows, a single strip)
template <int MT, bool TURNS>
__global__ __launch_bounds__(pblk::kThreads, MT <= 1 ? 3 : 2) void objects_polar_kernel(ObjArgs a, PolGeom g)
{
    __shared__ pblk::WaveSmem<MT, 4> sm[pblk::kWaves];
    if (*a.tag_ptr != a.tag) return;  // the workspace does not hold this plan's tables
    const int lane = threadIdx.x & 63, wave = cblk::wave_id();
    const int64_t strips = slot_strips(g, MT), per_col = column_strips(g, MT);
    int next = (int)blockIdx.x * pblk::kWaves + wave;
    for (;;) {
        int it;
        if constexpr (TURNS) {
            it = next;
            next += (int)gridDim.x * pblk::kWaves;
        } else {
            it = 0;
            if (lane == 0) it = atomicAdd(a.counter, 1);
            it = __builtin_amdgcn_readfirstlane(it);
        }
        if (it >= a.n_items) break;
        const int2 item = a.items[it];
        const int slot = __builtin_amdgcn_readfirstlane(item.x), blk = __builtin_amdgcn_readfirstlane(item.y);
        const int rg = blk / g.cols, col = blk % g.cols;
        const int4 sv = a.slots[slot];
        const int k0 = __builtin_amdgcn_readfirstlane(sv.x), k1 = __builtin_amdgcn_readfirstlane(sv.y);
        const int r0 = __builtin_amdgcn_readfirstlane(sv.z), r1 = __builtin_amdgcn_readfirstlane(sv.w);
        const int64_t strip0 = slot * strips + col * per_col + 2 * (int64_t)rg * block_values(g.na, MT);
        double sth, cth;
        sincos_cw((2.0 * 3.141592653589793 * (double)col) / (double)g.n_out, &sth, &cth);
        RotLoader ld{a.pos, a.nuc, a.mag, Rot{}, 0};
        for (int r = r0; r < r1; ++r) {
            ld.R = uniform_rot(a.rot + 9 * (int64_t)r);
            for (int k = k0; k < k1; ++k) {
                constexpr int N = pblk::Tiles<MT>::N;
                typename pblk::Tiles<MT>::T accC[N] = {}, accS[N] = {};
                pblk::accumulate<MT, 4, 4>(ld, a.off[k], a.off[k + 1], sth, cth, g.dq, rg * g.na, sm[wave], accC, accS);
                const bool first = r == r0 && k == k0;
                double uk = 0.0;
                double2 z = make_double2(1.0, 0.0);
                if (a.amp != nullptr) {
                    const double2 X = object_yz(a, ld.R.m, k);
                    uk = X.x * sth + X.y * cth;
                    z = twiddle(((double)(lane & (pblk::Tiles<MT>::kOffsets - 1)) + 0.5) * g.dq * uk);
                }
                auto add = [&](int i, double2 vp, double2 vm) {
                    // rows 32 a + 15 - b, 32 a + 16 + b
                    const int64_t strip = strip0 + 2 * i;
                    const bool all = MT > kExactTiles, lower = all || (i < g.na && 2 * (rg * g.na + i) < per_col);
                    const bool upper = all || (i < g.na && 2 * (rg * g.na + i) + 1 < per_col);
                    double *o = a.spec + strip * 256 + lane;
                    if (upper) add_spectral(o + 256, first, vp);
                    if (lower) add_spectral(o, first, vm);
                    if (a.amp != nullptr) {
                        const double c = ((double)(pblk::kRows * (rg * g.na + i)) + 15.5) * g.dq;
                        const double2 y = twiddle(c * uk);
                        double *u = a.amp + strip * 128 + lane;
                        if (upper) add_amplitude(u + 128, first, vp, y, z);
                        if (lower) add_amplitude(u, first, vm, y, make_double2(z.x, -z.y));
                    }
                };
                if constexpr (MT > 0) {
                    cblk::finish_whole<MT>(accC, accS,
                                           [&](int t, int h, double2 vp, double2 vm) { add(2 * t + h, vp, vm); });
                } else {
                    // tile t: channel 2 t + l / 16 % 2, the upper rows in the first half of the lanes
                    const double2 v0 = pblk::few_rows(accC[0], accS[0]), v1 = pblk::few_rows(accC[1], accS[1]);
                    const bool low = lane < 32;
                    const double2 send = low ? v1 : v0;
                    const double2 o = make_double2(pblk::other_half(send.x), pblk::other_half(send.y));
                    const double2 vp = low ? v0 : o, vm = low ? o : v1;
                    if constexpr (MT == kFewestRows) {  // both in the strip, strip_row
                        const bool upper = (lane & 8) != 0;
                        const double2 v = upper ? vp : vm;
                        add_spectral(a.spec + strip0 * 256 + lane, first, v);
                        if (a.amp != nullptr)
                            add_amplitude(a.amp + strip0 * 128 + lane, first, v, twiddle(7.5 * g.dq * uk),
                                          make_double2(z.x, upper ? z.y : -z.y));
                    } else {
                        add(0, vp, vm);
                    }
                }
            }
        }
    }
}

__global__ void fill_i32_kernel(int *p, int n, int v)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Pixel of lane column b of strip `at` of a line (row and column block, or column) and its
// mirror at -q; -1: none.
__device__ __forceinline__ void strip_pixel(const CartGeom &g, int mt, int line, int at, int b, int64_t &px,
                                            int64_t &mirror)
{
    const int rb = g.nrb == 1 ? 0 : line / g.nzb, a = rb * g.na + (at >> 1), jb = cblk::kOff * (line - rb * g.nzb) + b;
    px = mirror = -1;
    if (jb >= g.B) return;
    const int ip = g.nM - g.A + a, im = g.A - 1 - a, jp = g.nN - g.B + jb, jm = g.B - 1 - jb;
    if ((at & 1) == 0) {
        px = ip * g.strideM + jp * g.strideN;
        if (ip != im) mirror = im * g.strideM + jm * g.strideN;
    } else if (jp != jm) {
        px = ip * g.strideM + jm * g.strideN;
        if (ip != im) mirror = im * g.strideM + jp * g.strideN;
    }
}
__device__ __forceinline__ int strip_row(const PolGeom &g, int mt, int at, int b)
{
    if (g.mid == 8) return b < 8 ? 7 - b : b;
    const int per = block_values(g.na, mt), rg = g.nrg == 1 ? 0 : (at >> 1) / per;
    return pblk::slot_row(g, rg, (at >> 1) - rg * per, b, at & 1 ? 0 : 1);
}
__device__ __forceinline__ void strip_pixel(const PolGeom &g, int mt, int line, int at, int b, int64_t &px,
                                            int64_t &mirror)
{
    const int row = strip_row(g, mt, at, b);
    px = row < g.n0 ? (int64_t)row * g.n_out + line : -1;
    mirror = px >= 0 && g.nh > 0 ? px + g.nh : -1;
}

// Whether a strip has pixels (the matrix rows of the others hold what was in memory).
__device__ __forceinline__ bool strip_inside(const CartGeom &g, int mt, int line, int at)
{
    const int i = at >> 1;
    return i < g.na && (g.nrb == 1 || line / g.nzb * g.na + i < g.A);
}
__device__ __forceinline__ bool strip_inside(const PolGeom &g, int mt, int line, int at)
{
    if (mt <= kExactTiles) return true;
    const int per = block_values(g.na, mt), rg = g.nrg == 1 ? 0 : (at >> 1) / per, i = (at >> 1) - rg * per;
    return i < g.na && pblk::kRows * (rg * g.na + i) + 16 * (at & 1) < g.n0;
}

// (q_y, q_z) of lane column b of a strip.
__device__ __forceinline__ double2 strip_q(const CartGeom &g, int mt, int line, int at, int b)
{
    const int rb = line / g.nzb;
    const double qm = ((double)(rb * g.na + (at >> 1)) + g.firstM) * g.stepM;
    const double qn = ((double)(cblk::kOff * (line - rb * g.nzb) + b) + g.firstN) * g.stepN;
    const double n = at & 1 ? -qn : qn;
    return g.swapped ? make_double2(n, qm) : make_double2(qm, n);
}
__device__ __forceinline__ double2 strip_q(const PolGeom &g, int mt, int line, int at, int b)
{
    const double q = (double)strip_row(g, mt, at, b) * g.dq;
    double sth, cth;
    sincos_cw((2.0 * 3.141592653589793 * (double)line) / (double)g.n_out, &sth, &cth);
    return make_double2(q * sth, q * cth);
}

// out[s][pixel][v] = scale * sum of the slots of output s (slot_off CSR; null: all n_slots),
// in an order fixed by their number: the Q parts of a workgroup take contiguous shares, added
// up in turn.  PLANES = 16: spectra; 8: the coherent total, amplitudes (re, im) of the
// channels.  A workgroup takes a strip, through LDS into pixel order; the mirrored pixels take
// the conjugates.  A workspace that does not hold the plan's tables (tag mismatch) gives NaN.
template <int PLANES, int Q, class Geom>
__global__ __launch_bounds__(16 * PLANES * Q) void reduce_kernel(ObjArgs a, const double *__restrict__ slots,
                                                                 const int *__restrict__ slot_off, int n_slots, Geom g,
                                                                 int mt, int line0, int out0, int64_t P, double scale,
                                                                 double *__restrict__ out)
{
    constexpr int kStrip = 16 * PLANES;
    __shared__ double x[Q][16][PLANES + 1];
    const int part = Q == 1 ? 0 : threadIdx.x / kStrip, tid = Q == 1 ? threadIdx.x : threadIdx.x % kStrip;
    const int line = line0 + blockIdx.y, s = out0 + blockIdx.z, at = blockIdx.x;
    const uint32_t strip = (uint32_t)line * gridDim.x + at, strips = (uint32_t)slot_lines(g) * gridDim.x;
    if (!strip_inside(g, mt, line, at)) return;
    const bool ok = *a.tag_ptr == a.tag;
    double acc = 0.0;
    if (ok) {
        const int lo = slot_off != nullptr ? slot_off[s] : 0, hi = slot_off != nullptr ? slot_off[s + 1] : n_slots;
        const int first = Q == 1 ? lo : lo + (int)((int64_t)(hi - lo) * part / Q);
        const int last = Q == 1 ? hi : lo + (int)((int64_t)(hi - lo) * (part + 1) / Q);
        const double *p = slots + ((int64_t)first * strips + strip) * kStrip + tid;
        const int64_t slot = (int64_t)strips * kStrip;
#pragma unroll(Q == 1 ? 2 : 8)
        for (int i = first; i < last; ++i, p += slot) acc += *p;
    }
    const int lane = tid & 63, e = tid >> 6;
    x[part][lane & 15][PLANES == 16 ? kPacked[lane >> 4][e] : 2 * (lane >> 4) + e] = acc;
    if (acc != acc) a.counter[kNonfinite] = 1;
    __syncthreads();
    if (part != 0) return;
    const int b = tid / PLANES, v = tid % PLANES;
    double sum = x[0][b][v];
#pragma unroll
    for (int q = 1; q < Q; ++q) sum += x[q][b][v];
    const double val = ok ? scale * sum : __builtin_nan("");
    int64_t px, mirror;
    strip_pixel(g, mt, line, at, b, px, mirror);
    double *o = out + (int64_t)s * P * PLANES + v;
    const bool imag = (v & 1) != 0 && (PLANES == 8 || v >= 5);
    if (px >= 0) o[px * PLANES] = val;
    if (mirror >= 0) o[mirror * PLANES] = imag ? -val : val;
}

// Four parts a workgroup where an output has more than 64 slots: a part reads one after
// another.  (A part's waves read 512 bytes each: what they compute besides counts, so every
// workgroup takes one strip without a loop, and lines and outputs beyond a grid's 65,535 have
// launches of their own.  500 outputs of 8 x 40 polar pixels, half of the detector: 54 us with
// the tiles' padding, 20 now.)
template <int PLANES, class Geom>
int launch_reduce(const ObjArgs &a, const double *slots, const int *slot_off, int n_slots, int n_out,
                  const Geom &g, int mt, int64_t P, double scale, double *out, hipStream_t st)
{
    const bool split = n_slots > 64 * (int64_t)n_out;
    const int threads = 16 * PLANES * (split ? 4 : 1);
    const int64_t lines = slot_lines(g), per = slot_strips(g, mt) / lines;
    constexpr int kMost = 65535;
    for (int64_t line0 = 0; line0 < lines; line0 += kMost)
        for (int out0 = 0; out0 < n_out; out0 += kMost) {
            const dim3 grid((unsigned)per, (unsigned)std::min<int64_t>(lines - line0, kMost),
                            (unsigned)std::min(n_out - out0, kMost));
            if (split)
                hipLaunchKernelGGL((reduce_kernel<PLANES, 4, Geom>), grid, dim3(threads), 0, st, a, slots, slot_off,
                                   n_slots, g, mt, (int)line0, out0, P, scale, out);
            else
                hipLaunchKernelGGL((reduce_kernel<PLANES, 1, Geom>), grid, dim3(threads), 0, st, a, slots, slot_off,
                                   n_slots, g, mt, (int)line0, out0, P, scale, out);
            NUMAG_HIP_CHECK(hipGetLastError());
        }
    return NUMAG_OK;
}

// Results that came out as NaN, formed again term by term from the objects that hold a weight
// that is not finite: the matrix-core sums form a pixel as RR - II and the like, which is NaN
// where the terms' sum is infinite (nonfinite.h), and the other objects cannot change an
// infinite sum.  Nothing to do unless a reduction has set the flag (a launch of its own, since
// in the reductions its registers would take their occupancy).  A wave takes the strip of one
// output.
template <int PLANES, class Geom>
__device__ __forceinline__ void repair_strip(const ObjArgs &a, const Geom &g, int mt, int line, int at, int lo, int hi,
                                             double scale, double *__restrict__ out)
{
    constexpr int N = PLANES / 4;
    const int lane = threadIdx.x & 63, ch = lane >> 4, b = lane & 15;
    int64_t px, mirror;
    strip_pixel(g, mt, line, at, b, px, mirror);
    bool nan[N];
    bool any = false;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const int v = PLANES == 16 ? kPacked[ch][e] : 2 * ch + e;
        const double was = px >= 0 ? out[px * PLANES + v] : 0.0;
        nan[e] = was != was;
        any = any || nan[e];
    }
    if (!__any(any)) return;
    const double2 q = strip_q(g, mt, line, at, b);
    double sum[N] = {};
    bool found = false;
    for (int sl = lo; sl < hi; ++sl) {
        const int4 sv = a.slots[sl];
        for (int k = sv.x; k < sv.y; ++k) {
            bool finite = true;
            for (int64_t j = a.off[k] + lane; j < a.off[k + 1]; j += 64) {
                if (a.nuc != nullptr) finite = finite && isfinite(a.nuc[j]);
                if (a.mag != nullptr)
                    finite = finite && isfinite(a.mag[3 * j]) && isfinite(a.mag[3 * j + 1]) && isfinite(a.mag[3 * j + 2]);
            }
            if (__all(finite)) continue;
            found = true;
            for (int r = sv.z; r < sv.w; ++r) {
                const double *R = a.rot + 9 * (int64_t)r;
                double2 F = make_double2(0.0, 0.0);
                for (int64_t j = a.off[k]; j < a.off[k + 1]; ++j) {
                    double Y, Z, v;
                    sample_point(a.pos, a.nuc, a.mag, R, ch, j, Y, Z, v);
                    const double2 e = twiddle(q.x * Y + q.y * Z);
                    F.x += v * e.x;
                    F.y += v * e.y;
                }
                if constexpr (PLANES == 16) {
                    double v[4];
                    spectral_part(F, v);
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] += v[e];
                } else {
                    const double2 X = object_yz(a, R, k), v = cmul(twiddle(q.x * X.x + q.y * X.y), F);
                    sum[0] += v.x;
                    sum[1] += v.y;
                }
            }
        }
    }
    if (!found) return;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        if (!nan[e]) continue;
        const int v = PLANES == 16 ? kPacked[ch][e] : 2 * ch + e;
        const double val = scale * sum[e];
        if (px >= 0) out[px * PLANES + v] = val;
        if (mirror >= 0) out[mirror * PLANES + v] = (v & 1) != 0 && (PLANES == 8 || v >= 5) ? -val : val;
    }
}

template <class Geom>
__global__ __launch_bounds__(256) void nonfinite_objects_kernel(ObjArgs a, const int *__restrict__ slot_off, int n_slots,
                                                                int n_out, Geom g, int mt, int64_t P, double scale,
                                                                double *__restrict__ spec, double *__restrict__ amp)
{
    if (a.counter[kNonfinite] == 0 || *a.tag_ptr != a.tag) return;
    const int strips = (int)slot_strips(g, mt), per = strips / (int)slot_lines(g);
    for (int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); w < (int64_t)n_out * strips;
         w += (int64_t)gridDim.x * 4) {
        const int s = (int)(w / strips), strip = (int)(w % strips), line = strip / per, at = strip - line * per;
        if (!strip_inside(g, mt, line, at)) continue;
        repair_strip<16>(a, g, mt, line, at, slot_off[s], slot_off[s + 1], scale, spec + (int64_t)s * P * 16);
        if (amp != nullptr) repair_strip<8>(a, g, mt, line, at, 0, n_slots, 1.0, amp);
    }
}

int device_cus()
{
    static const int cus = [] {  // thread-safe one-time initialisation
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        return n;
    }();
    return cus;
}

// The full host-side plan: object groups, slots and sorted items.
struct Tables {
    ObjectsPlan p;
    std::vector<int4> slots;      // (object lo, hi, rotation lo, hi)
    std::vector<int> slot_off;    // outputs -> slots (CSR)
    std::vector<int2> items;      // (slot, block), by decreasing cost
};

// Column blocks per workgroup of a Cartesian plan (as a launch shape).  Eight share the row
// tables; fewer make more items and, where the last workgroup of a row would be half empty,
// fewer idle SIMDs.  Time of the item queue, largest first: whole rounds of the CUs for
// objects of one size, with the cheaper items of partial workgroups filling the last, else
// all items over the CUs plus three quarters of the largest.
// (With 8, 4, 2 and 1: 6 objects x 8 rotations, 170 x 180 pixels 1090, 952, 821, 1023 us; 30
// objects, 90 x 90, one rotation 123, 114, 85, 129; 4 objects, 200 x 100, one rotation 974,
// 639, 413, 271; 10 x 10, 150 x 150 1101, 1284, 1232, 1469.  20 x 10, 100 x 145, with the
// other axis packed 528 -> 390.  96 unequal objects, 256 x 256, one rotation 2.69 ms with 8,
// 2.45 with 4.)
int cart_shape(const Detector &d, const std::vector<int64_t> &off, int64_t K, int64_t W, int64_t n_rot, int64_t target)
{
    const double cus = (double)device_cus();
    int64_t most = 1;  // points of the largest object
    for (int64_t k = 0; k < K; ++k) most = std::max(most, off[k + 1] - off[k]);
    const bool equal = (double)most * (double)K <= 1.1 * (double)W;
    const double all = (double)std::max<int64_t>(W, 1) * (double)n_rot;
    int best = 32;
    double least = -1.0;
    for (int shape : {16, 32, 64, 8}) {
        CartGeom g{};
        int mt = 0;
        double group[2] = {};
        const double sum = cart_objects_geometry(d, shape, g, mt, group);
        const int64_t full = g.nzb / g.nz, rest = g.nzb % g.nz > 0 ? 1 : 0;
        const int64_t want = std::max<int64_t>(1, (target + (full + rest) * g.nrb - 1) / ((full + rest) * g.nrb));
        double t;
        if (equal) {
            const int64_t per_object = std::min<int64_t>(n_rot, (std::max(want, K) + K - 1) / K);
            const double slots = (double)(K * per_object);
            const double slot = (double)most * (double)((n_rot + per_object - 1) / per_object);
            const double nf = slots * (double)(full * g.nrb), nl = slots * (double)(rest * g.nrb);
            t = slot * (nf == 0.0 ? std::ceil(nl / cus) * group[1]
                                  : std::max(std::ceil(nf / cus) * group[0],
                                             nl == 0.0 ? 0.0 : (nf * group[0] + nl * group[1]) / cus + 0.5 * group[1]));
        } else {
            t = all * sum / cus + 0.75 * std::max((double)most, all / (double)want) * group[full > 0 ? 0 : 1];
        }
        if (least >= 0.0 && t >= 0.98 * least) continue;
        least = t;
        best = shape;
    }
    return best;
}

Tables make_tables(const Detector &d, bool hermitian, const std::vector<int64_t> &off, int64_t K, int64_t W,
                   int64_t n_rot, int mode, int spec_per_object)
{
    Tables T;
    ObjectsPlan &p = T.p;
    const Detector key = objects_detector(d, hermitian);
    const TuneShape ts = current_tune_shape(kTuneObjects, d, key, W);
    TuneShape entry{};
    const bool tuned = tuned_shape(kTuneObjects, key, W, &entry);
    if (d.kind == NUMAG_GRID_POLAR) {
        polar_geometry(d, 4, ts.shape, p.pg, p.mt);
        if (p.pg.na == 1) p.mt = kFewRows;
        if (d.n0 <= 16) {
            p.mt = kFewestRows;
            p.pg.mid = 8;
        }
        p.n_blocks = (int64_t)p.pg.cols * p.pg.nrg;
        p.strips = slot_strips(p.pg, p.mt);
    } else {
        cart_objects_geometry(d, tuned ? ts.shape : cart_shape(d, off, K, W, n_rot, ts.target), p.cg, p.mt, nullptr);
        p.n_blocks = (int64_t)((p.cg.nzb + p.cg.nz - 1) / p.cg.nz) * p.cg.nrb;
        p.strips = slot_strips(p.cg, p.mt);
    }
    const int64_t nblocks = p.n_blocks;
    // slot groups wanted (each spans all pixel blocks)
    const int64_t want = std::max<int64_t>(1, (ts.target + nblocks - 1) / std::max<int64_t>(nblocks, 1));
    // object groups: single objects, or contiguous groups of roughly equal point counts
    std::vector<int2> groups;
    if (spec_per_object) {
        for (int64_t k = 0; k < K; ++k) groups.push_back(make_int2((int)k, (int)k + 1));
    } else {
        const int64_t G = std::max<int64_t>(1, std::min<int64_t>(want, K));
        int64_t k = 0;
        for (int64_t g = 0; g < G && k < K; ++g) {
            const int64_t target = (W * (g + 1)) / G;
            const int64_t k0 = k;
            while (k < K && (off[k + 1] <= target || k == k0)) ++k;
            if (g == G - 1) k = K;
            groups.push_back(make_int2((int)k0, (int)k));
        }
    }
    // rotation ranges per group, proportional to the group's cost
    const double total = (double)std::max<int64_t>(W, 1) * (double)n_rot;
    const double per_slot = total / (double)std::max<int64_t>(want, (int64_t)groups.size());
    T.slot_off.push_back(0);
    for (const int2 &g : groups) {
        const double cost = (double)(off[g.y] - off[g.x] + 1) * (double)n_rot;
        int64_t H = (int64_t)std::ceil(cost / per_slot);
        H = std::max<int64_t>(1, std::min<int64_t>(H, n_rot));
        if (mode == NUMAG_MODE_SPLIT) H = 1;
        for (int64_t h = 0; h < H; ++h)
            T.slots.push_back(make_int4(g.x, g.y, (int)(n_rot * h / H), (int)(n_rot * (h + 1) / H)));
        if (spec_per_object) T.slot_off.push_back((int)T.slots.size());
    }
    if (!spec_per_object) T.slot_off.push_back((int)T.slots.size());
    p.n_slots = (int)T.slots.size();
    p.n_out = spec_per_object ? (int)K : 1;
    // items, most expensive first
    std::vector<std::pair<int64_t, int2>> it;
    it.reserve((size_t)p.n_slots * nblocks);
    for (int s = 0; s < p.n_slots; ++s) {
        const int4 sl = T.slots[s];
        const int64_t cost = (off[sl.y] - off[sl.x] + 1) * (int64_t)(sl.w - sl.z);
        for (int64_t b = 0; b < nblocks; ++b) it.push_back({cost, make_int2(s, (int)b)});
    }
    std::stable_sort(it.begin(), it.end(), [](const auto &a, const auto &b) { return a.first > b.first; });
    for (auto &x : it) T.items.push_back(x.second);
    p.n_items = (int64_t)T.items.size();
    return T;
}

size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

// The persistent kernel's part of an object-mode plan: the work tables and where
// they and the accumulators sit in the workspace.
struct ObjPlanTables {
    Tables T;
    size_t o_off, o_items, o_slots, o_slot_off, o_counter, o_spec, o_amp;
};

Detector objects_detector(const Detector &d, bool hermitian)
{
    Detector dk = d;
    if (hermitian) {
        if (d.kind == NUMAG_GRID_CARTESIAN) dk.n0 = (d.n0 + 1) / 2;  // rows [0, h): the first h n1 pixels
        else dk.n1 = d.n1 / 2;  // theta in [0, pi); n_theta stays the full count
    }
    return dk;
}

void build_objects_plan(ObjPlan &pl)
{
    auto c = std::make_shared<ObjPlanTables>();
    const bool hermitian = pl.path == NUMAG_PATH_DIRECT_HERMITIAN;
    c->T = make_tables(pl.d, hermitian, pl.off, pl.K, pl.W, pl.n_rot, pl.mode, pl.spec_per_object);
    const Tables &T = c->T;
    size_t used = kPlanTagBytes;
    auto take = [&](size_t bytes) {
        const size_t r = used;
        used += al(bytes);
        return r;
    };
    c->o_off = take(sizeof(int64_t) * (pl.K + 1));
    pl.o_rot = take(sizeof(double) * 9 * pl.n_rot);
    c->o_items = take(sizeof(int2) * T.items.size());
    c->o_slots = take(sizeof(int4) * T.slots.size());
    c->o_slot_off = take(sizeof(int) * T.slot_off.size());
    const size_t image_bytes = used;
    c->o_counter = take(sizeof(int) * 64);
    c->o_spec = take(sizeof(double) * 256 * (size_t)T.p.n_slots * T.p.strips);
    c->o_amp = pl.mode == NUMAG_MODE_SPLIT ? take(sizeof(double) * 128 * (size_t)T.p.n_slots * T.p.strips) : 0;
    // both paths sum the same pixels; the whole-detector one's size stays the larger
    if (!hermitian) take(1);
    pl.ws_bytes = used;
    // host image of the tag and the tables (rotations are filled by the caller)
    pl.image.assign(image_bytes, 0);
    std::memcpy(pl.image.data(), &pl.tag, sizeof(pl.tag));
    std::memcpy(pl.image.data() + c->o_off, pl.off.data(), sizeof(int64_t) * (pl.K + 1));
    std::memcpy(pl.image.data() + c->o_items, T.items.data(), sizeof(int2) * T.items.size());
    std::memcpy(pl.image.data() + c->o_slots, T.slots.data(), sizeof(int4) * T.slots.size());
    std::memcpy(pl.image.data() + c->o_slot_off, T.slot_off.data(), sizeof(int) * T.slot_off.size());
    pl.tables = c;
}

int launch_objects_plan(const ObjPlan &pl, const numag_sample &s, double *spec_out, double *amp_out, void *ws,
                        hipStream_t st)
{
    const ObjPlanTables &c = *pl.tables;
    const ObjectsPlan &p = c.T.p;
    const int64_t P = (int64_t)pl.d.n0 * pl.d.n1;
    char *base = (char *)ws;
    const unsigned long long *tag_ptr = (const unsigned long long *)base;
    const unsigned long long tag = pl.tag;
    int *d_counter = (int *)(base + c.o_counter);
    double *d_spec = (double *)(base + c.o_spec);
    double *d_amp = pl.mode == NUMAG_MODE_SPLIT ? (double *)(base + c.o_amp) : nullptr;

    // (a kernel, so that the sequence can be captured; the accumulators are written by
    // the first object of their slot)
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(64), 0, st, d_counter, 64, 0);
    NUMAG_HIP_CHECK(hipGetLastError());

    ObjArgs args{};
    args.tag_ptr = tag_ptr;
    args.tag = tag;
    args.pos = s.pos;
    args.nuc = s.nuc;
    args.mag = s.mag;
    args.off = (const int64_t *)(base + c.o_off);
    args.obj_pos = s.obj_pos;
    args.rot = (const double *)(base + pl.o_rot);
    args.items = (const int2 *)(base + c.o_items);
    args.slots = (const int4 *)(base + c.o_slots);
    args.n_items = (int)p.n_items;
    args.counter = d_counter;
    args.spec = d_spec;
    args.amp = d_amp;
    const bool pol = pl.d.kind == NUMAG_GRID_POLAR;
    // persistent grid: as many workgroups as fit the chip at once (two of 4 waves, three of one
    // tile, or one of 8 waves, per CU; the third: 73 -> 62 us and 101 -> 86 in the cases below)
    const int64_t fit = (!pol ? 1 : p.mt <= 1 ? 3 : 2) * (int64_t)device_cus();
    const int64_t want = pol ? (p.n_items + pblk::kWaves - 1) / pblk::kWaves : p.n_items;
    const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(want, fit)));
    // The counter takes an atomic every 12 ns, 25 us for a turn of the chip's waves: small items
    // would wait for it.  They are sorted by cost, so waves that take them in order end within
    // one item of each other; larger ones the counter evens out better.  The line is at an item
    // of 25 us, 160 points, rotations and tiles (500 objects of 40 points, two rotations, one
    // tile, all by the counter and now: 8 x 40 pixels 260 -> 62 us, 16 x 64 397 -> 86; of four
    // tiles, 200 x 120: 730 by the counter, 790 in order).
    const bool small = (double)pl.W * (double)pl.n_rot * std::max(p.mt, 1) < 160.0 * (double)p.n_slots;
    {
        TimedLaunch timed(NUMAG_KERNEL_OBJECTS, st);
#define NUMAG_LAUNCH_OBJ_P(MT)                                                                                  \
    if (small)                                                                                                  \
        hipLaunchKernelGGL((objects_polar_kernel<MT, true>), grid, dim3(pblk::kThreads), 0, st, args, p.pg);       \
    else                                                                                                        \
        hipLaunchKernelGGL((objects_polar_kernel<MT, false>), grid, dim3(pblk::kThreads), 0, st, args, p.pg)
#define NUMAG_LAUNCH_OBJ(MT)                                                                                    \
    case MT:                                                                                                    \
        if (!pol) {                                                                                             \
            hipLaunchKernelGGL((objects_kernel<MT>), grid, dim3(cblk::kThreads), 0, st, args, p.cg);               \
            break;                                                                                              \
        }                                                                                                       \
        NUMAG_LAUNCH_OBJ_P(MT);                                                                                 \
        break
        switch (p.mt) {
            case kFewestRows:
                NUMAG_LAUNCH_OBJ_P(kFewestRows);
                break;
            case kFewRows:
                NUMAG_LAUNCH_OBJ_P(kFewRows);
                break;
            NUMAG_LAUNCH_OBJ(1);
            NUMAG_LAUNCH_OBJ(2);
            NUMAG_LAUNCH_OBJ(3);
            NUMAG_LAUNCH_OBJ(4);
            NUMAG_LAUNCH_OBJ(5);
            NUMAG_LAUNCH_OBJ(6);
            NUMAG_LAUNCH_OBJ(7);
            NUMAG_LAUNCH_OBJ(8);
        }
#undef NUMAG_LAUNCH_OBJ
#undef NUMAG_LAUNCH_OBJ_P
    }
    NUMAG_HIP_CHECK(hipGetLastError());
    const int *d_off = (const int *)(base + c.o_slot_off);
    const double scale = 1.0 / (double)pl.n_rot;
    const auto finish = [&](const auto &g) {
        int rc = launch_reduce<16>(args, d_spec, d_off, p.n_slots, p.n_out, g, p.mt, P, scale, spec_out, st);
        if (rc == NUMAG_OK && d_amp != nullptr)
            rc = launch_reduce<8>(args, d_amp, nullptr, p.n_slots, 1, g, p.mt, P, 1.0, amp_out, st);
        if (rc != NUMAG_OK) return rc;
        const dim3 grid((unsigned)std::min<int64_t>((p.n_out * p.strips + 3) / 4, 2 * (int64_t)device_cus()));
        hipLaunchKernelGGL((nonfinite_objects_kernel<std::decay_t<decltype(g)>>), grid, dim3(256), 0, st, args, d_off,
                           p.n_slots, p.n_out, g, p.mt, P, scale, spec_out, d_amp != nullptr ? amp_out : nullptr);
        NUMAG_HIP_CHECK(hipGetLastError());
        return NUMAG_OK;
    };
    return pol ? finish(p.pg) : finish(p.cg);
}

}  // namespace numag
