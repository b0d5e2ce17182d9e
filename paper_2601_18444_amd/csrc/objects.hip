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
// a persistent kernel through an atomic counter -- to workgroups of 8 waves on a
// Cartesian detector (cartesian_block.h), to single waves on a polar one
// (polar_block.h); slots are reduced in a fixed order, so results are reproducible
// bit for bit.
//
// Rotations are applied on the fly (X = R x, w' = (n, R m)) while a chunk's
// phasors are generated, so the point data is read once per chunk and never
// rewritten per orientation; the first points of the next object are loaded before
// the products of the current one.
//
// Accumulators hold only the independent half of the pixels (G(-q) = conj G(q) for
// real weights), in the order the lanes hold them: lane l has channel g = l / 16 of
// the pixels of one slot, takes the other channels from lanes l ^ 16, 32, 48 and
// keeps four of the sixteen reals of G (kPacked), so that every access is a
// coalesced wave-wide row; the reduction puts them into pixel order.
//
// Measured, kernel time before (10.5 vector FP64 instructions per term over every pixel)
// and now: 16 particles (96,000 points) x 24 rotations, 128 x 128: 14.2 -> 5.70 ms (4.04 of
// it multiply-adds at 74.7 TFLOP/s); 96 objects (240,000 points) split, 256 x 256: 6.19 -> 2.50 ms
// (1.68; the largest object's items run alone at the end).
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
    double *spec;            // [n_slots][tiles][2 halves][2 signs][4][64]
    double *amp;             // [n_slots][tiles][2 halves][4][64] or null (split mode)
};

// Entry of the packed spectral matrix that lane group g keeps in row e: its own diagonal
// entry, then one real of the pair (g, g ^ e): the real part in the group of the smaller
// channel, the imaginary part in the other.
__device__ constexpr int kPacked[4][4] = {{0, 4, 6, 8}, {1, 5, 12, 10}, {2, 14, 7, 11}, {3, 15, 13, 9}};

// Adds (first: writes) F F^H of one sign to the lane's four accumulators o[64 e].  (Fused
// products are written out, so that every inlined copy rounds alike.)
__device__ __forceinline__ void add_spectral(double *__restrict__ o, bool first, double2 F)
{
    const int g = (threadIdx.x & 63) >> 4;
    double v[4];
    v[0] = fma(F.x, F.x, F.y * F.y);
#pragma unroll
    for (int e = 1; e < 4; ++e) {
        const double ox = __shfl_xor(F.x, 16 * e), oy = __shfl_xor(F.y, 16 * e);
        // Re F_a conj(F_b) is symmetric; Im of the smaller channel a (the other lane's)
        // with b (this one's) is a_i b_r - a_r b_i
        v[e] = g < (g ^ e) ? fma(F.x, ox, F.y * oy) : fma(oy, F.x, -(ox * F.y));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) o[64 * e] = first ? v[e] : o[64 * e] + v[e];
}

// Adds (first: writes) one channel of the pixel pair times the object's phasors y z, y conj z.
__device__ __forceinline__ void add_amplitude(double *__restrict__ o, bool first, double2 vp, double2 vm, double2 y,
                                              double2 z)
{
    auto mul = [](double2 u, double2 v) {
        return make_double2(fma(u.x, v.x, -(u.y * v.y)), fma(u.x, v.y, u.y * v.x));
    };
    const double2 a = mul(mul(y, z), vp), b = mul(mul(y, make_double2(z.x, -z.y)), vm);
    o[0] = first ? a.x : o[0] + a.x;
    o[64] = first ? a.y : o[64] + a.y;
    o[128] = first ? b.x : o[128] + b.x;
    o[192] = first ? b.y : o[192] + b.y;
}

// Lab position (Y, Z) of object k.
__device__ __forceinline__ double2 object_yz(const ObjArgs &a, const Rot &R, int k)
{
    if (a.obj_pos == nullptr) return make_double2(0.0, 0.0);
    const double *o = a.obj_pos + 3 * (int64_t)k;
    return make_double2(R.m[3] * o[0] + R.m[4] * o[1] + R.m[5] * o[2],
                        R.m[6] * o[0] + R.m[7] * o[1] + R.m[8] * o[2]);
}

// An object's sum v, if NaN, over its points [j0, j1) under the rotation R (in memory) from
// its terms that are not finite (nonfinite.h).
__device__ __forceinline__ double2 object_repair(const ObjArgs &a, const double *R, int64_t j0, int64_t j1, double qy,
                                                 double qz, double2 v)
{
    if (!is_nan(v)) return v;
    const int ch = (threadIdx.x & 63) >> 4;
    return nonfinite_terms([&](int64_t j, double &Y, double &Z,
                               double &w) { sample_point(a.pos, a.nuc, a.mag, R, ch, j, Y, Z, w); },
                           j0, j1, qy, qz, v);
}

// Sums of an object put aside by a wave that holds a NaN among them, until the matrix
// accumulators are free: which of its tile halves (wave-uniform).
template <int MT>
struct Aside {
    double2 v[2 * MT][2];
    unsigned which;
    __device__ __forceinline__ Aside() : which(0) {}
    __device__ __forceinline__ void take(int i, double2 vp, double2 vm)
    {
        v[i][0] = vp;
        v[i][1] = vm;
        which |= 1u << i;
    }
};

// Whether a wave may hold a NaN among its finished sums (the parts of all tiles added up).
template <int MT>
__device__ __forceinline__ bool may_hold_nan(const cblk::v4d (&accC)[MT], const cblk::v4d (&accS)[MT])
{
    double s = 0.0;
    cblk::finish_whole<MT>(accC, accS, [&](int, int, double2 vp, double2 vm) { s += (vp.x + vp.y) + (vm.x + vm.y); });
    return __any(s != s) != 0;
}

template <int MT>
__global__ __launch_bounds__(cblk::kThreads, 2) void objects_kernel(ObjArgs a, CartGeom g)
{
    __shared__ cblk::Smem<MT> sm;
    __shared__ int s_item;
    if (*a.tag_ptr != a.tag) return;  // the workspace does not hold this plan's tables
    const int lane = threadIdx.x & 63;
    const int groups = (g.nzb + g.nz - 1) / g.nz;
    const int64_t tiles = (int64_t)g.nrb * g.nzb * MT;
    if (4 * g.na < 8 * MT) {  // rows no slot writes: no stray NaN for may_hold_nan
        for (int i = threadIdx.x; i < (int)(sizeof(sm.y) / sizeof(double)); i += cblk::kThreads) (&sm.y[0][0][0])[i] = 0.0;
    }
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
        const int64_t tile0 = slot * tiles + ((int64_t)rb * g.nzb + zb) * MT;
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
                    const double2 X = object_yz(a, ld.R, k);
                    Xm = g.swapped ? X.y : X.x;
                    z = twiddle(((double)(cblk::kOff * zb + (lane & 15)) + g.firstN) * g.stepN *
                                (g.swapped ? X.x : X.y));
                }
                auto add = [&](int i, double2 vp, double2 vm) {
                    const int64_t th = tile0 * 2 + i;
                    double *o = a.spec + th * 512 + lane;
                    add_spectral(o, first, vp);
                    add_spectral(o + 256, first, vm);
                    if (a.amp != nullptr) {
                        const double qm = ((double)(rb * g.na + i) + g.firstM) * g.stepM;
                        add_amplitude(a.amp + th * 256 + lane, first, vp, vm, twiddle(qm * Xm), z);
                    }
                };
                Aside<MT> aside;
                const int b = cblk::kOff * zb + (lane & 15);
                auto put_aside = [&](int t, int h, double2 vp, double2 vm) { aside.take(2 * t + h, vp, vm); };
                auto put = [&](int t, int h, double2 vp, double2 vm) { add(2 * t + h, vp, vm); };
                if (g.nz != cblk::kWaves) {
                    cblk::finish_groups<MT>(g, zb0, sm, accC, accS, [&](int t, int h, double2 vp, double2 vm) {
                        if (__builtin_expect(__any(is_nan(vp) || is_nan(vm)) != 0, 0))
                            put_aside(t, h, vp, vm);
                        else
                            put(t, h, vp, vm);
                    });
                } else if (zb < g.nzb) {
                    if (__builtin_expect(may_hold_nan<MT>(accC, accS), 0))
                        cblk::finish_whole<MT>(accC, accS, put_aside);
                    else
                        cblk::finish_whole<MT>(accC, accS, put);
                }
                while (__builtin_expect(aside.which != 0, 0)) {
                    const int i = __builtin_ctz(aside.which);
                    aside.which &= aside.which - 1;
                    const double qm = ((double)(rb * g.na + i) + g.firstM) * g.stepM;
                    const double qn = ((double)b + g.firstN) * g.stepN;
                    const bool on = i < g.na && rb * g.na + i < g.A && b < g.B;
                    double2 v[2] = {aside.v[i][0], aside.v[i][1]};
#pragma unroll 1
                    for (int s = 0; on && s < 2; ++s) {
                        const double q = s == 0 ? qn : -qn;
                        v[s] = object_repair(a, a.rot + 9 * (int64_t)r, a.off[k], a.off[k + 1], g.swapped ? q : qm,
                                             g.swapped ? qm : q, v[s]);
                    }
                    add(i, v[0], v[1]);
                }
            }
        }
    }
}

// A work item belongs to one wave: (slot, theta column and row group).
template <int MT>
__global__ __launch_bounds__(pblk::kThreads, 2) void objects_polar_kernel(ObjArgs a, PolGeom g)
{
    __shared__ pblk::WaveSmem<MT, 4> sm[pblk::kWaves];
    if (*a.tag_ptr != a.tag) return;  // the workspace does not hold this plan's tables
    const int lane = threadIdx.x & 63, wave = cblk::wave_id();
    const int64_t tiles = (int64_t)g.nrg * g.cols * MT;
    for (;;) {
        int it = 0;
        if (lane == 0) it = atomicAdd(a.counter, 1);
        it = __builtin_amdgcn_readfirstlane(it);
        if (it >= a.n_items) break;
        const int2 item = a.items[it];
        const int slot = __builtin_amdgcn_readfirstlane(item.x), blk = __builtin_amdgcn_readfirstlane(item.y);
        const int rg = blk / g.cols, col = blk % g.cols;
        const int4 sv = a.slots[slot];
        const int k0 = __builtin_amdgcn_readfirstlane(sv.x), k1 = __builtin_amdgcn_readfirstlane(sv.y);
        const int r0 = __builtin_amdgcn_readfirstlane(sv.z), r1 = __builtin_amdgcn_readfirstlane(sv.w);
        const int64_t tile0 = slot * tiles + ((int64_t)rg * g.cols + col) * MT;
        double sth, cth;
        sincos_cw((2.0 * 3.141592653589793 * (double)col) / (double)g.n_out, &sth, &cth);
        RotLoader ld{a.pos, a.nuc, a.mag, Rot{}, 0};
        for (int r = r0; r < r1; ++r) {
            ld.R = uniform_rot(a.rot + 9 * (int64_t)r);
            for (int k = k0; k < k1; ++k) {
                cblk::v4d accC[MT], accS[MT];
                cblk::zero<MT>(accC, accS);
                pblk::accumulate<MT, 4>(ld, a.off[k], a.off[k + 1], sth, cth, g.dq, rg * g.na, sm[wave], accC, accS);
                const bool first = r == r0 && k == k0;
                double uk = 0.0;
                double2 z = make_double2(1.0, 0.0);
                if (a.amp != nullptr) {
                    const double2 X = object_yz(a, ld.R, k);
                    uk = X.x * sth + X.y * cth;
                    z = twiddle(((double)(lane & 15) + 0.5) * g.dq * uk);
                }
                auto add = [&](int i, double2 vp, double2 vm) {
                    const int64_t th = tile0 * 2 + i;
                    double *o = a.spec + th * 512 + lane;
                    add_spectral(o, first, vp);
                    add_spectral(o + 256, first, vm);
                    if (a.amp != nullptr) {
                        const double c = ((double)(pblk::kRows * (rg * g.na + i)) + 15.5) * g.dq;
                        add_amplitude(a.amp + th * 256 + lane, first, vp, vm, twiddle(c * uk), z);
                    }
                };
                auto row = [&](int i, int s) { return pblk::slot_row(g, rg, i, lane & 15, s); };
                Aside<MT> aside;
                if (__builtin_expect(may_hold_nan<MT>(accC, accS), 0))
                    cblk::finish_whole<MT>(accC, accS, [&](int t, int h, double2 vp, double2 vm) {
                        aside.take(2 * t + h, vp, vm);
                    });
                else
                    cblk::finish_whole<MT>(accC, accS,
                                           [&](int t, int h, double2 vp, double2 vm) { add(2 * t + h, vp, vm); });
                while (__builtin_expect(aside.which != 0, 0)) {
                    const int i = __builtin_ctz(aside.which);
                    aside.which &= aside.which - 1;
                    double2 v[2] = {aside.v[i][0], aside.v[i][1]};
#pragma unroll 1
                    for (int s = 0; s < 2; ++s) {
                        const double q = (double)row(i, s) * g.dq;
                        if (i < g.na && row(i, s) < g.n0)
                            v[s] = object_repair(a, a.rot + 9 * (int64_t)r, a.off[k], a.off[k + 1], q * sth, q * cth,
                                                 v[s]);
                    }
                    add(i, v[0], v[1]);
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

// Pixels of a slot tile (t, h), lane column b: (+) and (-), and their mirrors at -q; -1: none.
template <int POLAR>
__device__ __forceinline__ void tile_pixels(const CartGeom &cg, const PolGeom &pg, int MT, int64_t th, int b,
                                            int64_t (&px)[2], int64_t (&mirror)[2])
{
    px[0] = px[1] = mirror[0] = mirror[1] = -1;
    const int h = (int)(th & 1), t = (int)((th >> 1) % MT);
    const int64_t blk = (th >> 1) / MT;
    if (POLAR) {
        const int rg = (int)(blk / pg.cols), col = (int)(blk % pg.cols);
        const int e = 2 * t + h, a = rg * pg.na + e;
        if (e >= pg.na) return;
        const int rp = pblk::kRows * a + 16 + b, rm = pblk::kRows * a + 15 - b;
        if (rp < pg.n0) px[0] = (int64_t)rp * pg.n_out + col;
        if (rm < pg.n0) px[1] = (int64_t)rm * pg.n_out + col;
        if (pg.nh > 0)
            for (int s = 0; s < 2; ++s)
                if (px[s] >= 0) mirror[s] = px[s] + pg.nh;
    } else {
        const cblk::CellPixels x =
            cblk::cell_pixels(cg, 4, (int)(blk / cg.nzb), (int)(blk % cg.nzb), 8 * t + 4 * h, b);
        if (!x.ok) return;
        px[0] = x.pp;
        if (x.twoN) px[1] = x.pm;
        if (x.twoM) {
            mirror[0] = x.mm;
            if (x.twoN) mirror[1] = x.mp;
        }
    }
}

// out[s][pixel][v] = scale * sum of the slots of output s (slot_off CSR, ascending), one
// workgroup per (output, tile half, sign), through LDS into pixel order; the mirrored
// pixels take conj G.  A workspace that does not hold the plan's tables (tag mismatch)
// gives NaN.
template <int POLAR>
__global__ __launch_bounds__(256) void spec_reduce_kernel(const unsigned long long *tag_ptr, unsigned long long tag,
                                                          const double *__restrict__ slots,
                                                          const int *__restrict__ slot_off, CartGeom cg, PolGeom pg,
                                                          int MT, int64_t n_th, int64_t P, double scale,
                                                          double *__restrict__ out)
{
    __shared__ double x[16][17];
    const int tid = threadIdx.x;
    const int64_t th = blockIdx.x >> 1;
    const int sign = blockIdx.x & 1, s = blockIdx.y;
    {
        const int lane = tid & 63, e = tid >> 6;
        double v = __builtin_nan("");
        if (*tag_ptr == tag) {
            const double *p = slots + ((th * 2 + sign) * 4 + e) * 64 + lane;
            double acc = 0.0;
            for (int sl = slot_off[s]; sl < slot_off[s + 1]; ++sl) acc += p[(int64_t)sl * n_th * 512];
            v = scale * acc;
        }
        x[lane & 15][kPacked[lane >> 4][e]] = v;
    }
    __syncthreads();
    const int b = tid >> 4, v = tid & 15;
    int64_t px[2], mirror[2];
    tile_pixels<POLAR>(cg, pg, MT, th, b, px, mirror);
    const double val = x[b][v];
    double *o = out + (int64_t)s * P * 16 + v;
    if (px[sign] >= 0) o[px[sign] * 16] = val;
    if (mirror[sign] >= 0) o[mirror[sign] * 16] = (v >= 5 && (v & 1)) ? -val : val;
}

// Coherent total: the amplitude slots summed in order, mirrored pixels conjugated.
template <int POLAR>
__global__ __launch_bounds__(256) void amp_reduce_kernel(const unsigned long long *tag_ptr, unsigned long long tag,
                                                         const double *__restrict__ slots, int n_slots, CartGeom cg,
                                                         PolGeom pg, int MT, int64_t n_th, double *__restrict__ amp)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = (int)(idx & 63);
    const int64_t th = idx >> 6;
    if (th >= n_th) return;
    double v[4];
    const bool ok = *tag_ptr == tag;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = ok ? 0.0 : __builtin_nan("");
    if (ok)
        for (int sl = 0; sl < n_slots; ++sl) {
            const double *p = slots + ((int64_t)sl * n_th + th) * 256 + lane;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] += p[64 * k];
        }
    int64_t px[2], mirror[2];
    tile_pixels<POLAR>(cg, pg, MT, th, lane & 15, px, mirror);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (px[s] >= 0) cblk::put_pixel(amp, px[s], lane >> 4, v[2 * s], v[2 * s + 1], false);
        if (mirror[s] >= 0) cblk::put_pixel(amp, mirror[s], lane >> 4, v[2 * s], -v[2 * s + 1], false);
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
    const TuneShape ts = current_tune_shape(kTuneObjects, key, W);
    TuneShape entry{};
    const bool tuned = tuned_shape(kTuneObjects, key, W, &entry) && valid_tune_shape(kTuneObjects, key, entry);
    if (d.kind == NUMAG_GRID_POLAR) {
        polar_geometry(d, 4, ts.shape, p.pg, p.mt);
        p.n_blocks = (int64_t)p.pg.cols * p.pg.nrg;
        p.n_th = p.n_blocks * p.mt * 2;
    } else {
        cart_objects_geometry(d, tuned ? ts.shape : cart_shape(d, off, K, W, n_rot, ts.target), p.cg, p.mt, nullptr);
        p.n_blocks = (int64_t)((p.cg.nzb + p.cg.nz - 1) / p.cg.nz) * p.cg.nrb;
        p.n_th = (int64_t)p.cg.nzb * p.cg.nrb * p.mt * 2;
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
    // accumulators of a slot: 256 doubles of spectra and 256 of amplitudes per tile half
    // and sign pair hold the independent half of the pixels; the whole-detector path asks
    // for twice that, as a slot of every pixel takes
    const size_t th = (size_t)T.p.n_th * (hermitian ? 1 : 2);
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
    c->o_spec = take(sizeof(double) * 512 * (size_t)T.p.n_slots * th);
    c->o_amp = pl.mode == NUMAG_MODE_SPLIT ? take(sizeof(double) * 256 * (size_t)T.p.n_slots * th) : 0;
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
    // persistent grid: as many workgroups as fit the chip at once (two of 4 waves, or one
    // of 8, per CU)
    const int64_t fit = (pol ? 2 : 1) * (int64_t)device_cus();
    const int64_t want = pol ? (p.n_items + pblk::kWaves - 1) / pblk::kWaves : p.n_items;
    {
        TimedLaunch timed(NUMAG_KERNEL_OBJECTS, st);
        const dim3 g((unsigned)std::max<int64_t>(1, std::min<int64_t>(want, fit)));
#define NUMAG_LAUNCH_OBJ(MT)                                                                                    \
    case MT:                                                                                                    \
        if (pol) hipLaunchKernelGGL((objects_polar_kernel<MT>), g, dim3(pblk::kThreads), 0, st, args, p.pg);     \
        else hipLaunchKernelGGL((objects_kernel<MT>), g, dim3(cblk::kThreads), 0, st, args, p.cg);              \
        break
        switch (p.mt) {
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
    }
    NUMAG_HIP_CHECK(hipGetLastError());

    const dim3 gs((unsigned)(p.n_th * 2), p.n_out), ga((unsigned)((p.n_th * 64 + 255) / 256));
    const int *d_off = (const int *)(base + c.o_slot_off);
    const double scale = 1.0 / (double)pl.n_rot;
    if (pol)
        hipLaunchKernelGGL((spec_reduce_kernel<1>), gs, dim3(256), 0, st, tag_ptr, tag, d_spec, d_off, p.cg, p.pg, p.mt,
                           p.n_th, P, scale, spec_out);
    else
        hipLaunchKernelGGL((spec_reduce_kernel<0>), gs, dim3(256), 0, st, tag_ptr, tag, d_spec, d_off, p.cg, p.pg, p.mt,
                           p.n_th, P, scale, spec_out);
    NUMAG_HIP_CHECK(hipGetLastError());
    if (d_amp != nullptr) {
        if (pol)
            hipLaunchKernelGGL((amp_reduce_kernel<1>), ga, dim3(256), 0, st, tag_ptr, tag, d_amp, p.n_slots, p.cg, p.pg,
                               p.mt, p.n_th, amp_out);
        else
            hipLaunchKernelGGL((amp_reduce_kernel<0>), ga, dim3(256), 0, st, tag_ptr, tag, d_amp, p.n_slots, p.cg, p.pg,
                               p.mt, p.n_th, amp_out);
        NUMAG_HIP_CHECK(hipGetLastError());
    }
    return NUMAG_OK;
}

}  // namespace numag
