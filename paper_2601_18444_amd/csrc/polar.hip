// Direct Fourier sums on the paper's polar (q, theta) detector (Sec. 3.2), on the
// building block of polar_block.h.
//
// Measured, kernel time before (lanes walking q rows with a two-term recurrence, about
// 10 vector FP64 instructions per term, every column summed) and now:
//   100,003 points, 256 x 360       5.30 -> 1.28 ms (0.99 of it multiply-adds at 74.7 TFLOP/s)
//   24,000 points, 1000 x 1000      9.55 -> 3.22 ms (2.6)
// The rest is the tables: about 240 vector instructions per 32 points and column.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "polar_block.h"

namespace numag {

// Row blocks per wave of a launch shape.
static int shape_blocks(int shape)
{
    constexpr int blocks[kPolarShapeCount] = {2, 1, 4, 8, 16};
    return blocks[shape];
}

template <int CH, int NW>
struct PolarRecLoader {
    using Rec = typename std::conditional<NW == CH, PointRec, PairRec>::type;
    using Raw = cblk::Point<NW>;
    const Rec *__restrict__ pts;
    __device__ __forceinline__ Raw raw(int64_t j) const
    {
        const Rec &r = pts[j];
        Raw p;
        p.m = r.Y;
        p.n = r.Z;
#pragma unroll
        for (int c = 0; c < NW; ++c) p.w[c] = r.w[(NW == 3 ? 1 : 0) + c];
        return p;
    }
    __device__ __forceinline__ Raw point(const Raw &r) const { return r; }
    // (pairs: none, their caller sees to infinite weights)
    __host__ __device__ __forceinline__ PointSource source() const
    {
        PointSource s{};
        if constexpr (NW == CH) s.rec = pts;
        return s;
    }
};

// Points straight from a sample (no object offsets), with the arithmetic of the records.
template <int CH>
struct PolarSampleLoader {
    struct Raw {
        double x[3], n, m[3];
    };
    const double *__restrict__ pos, *__restrict__ nuc, *__restrict__ mag;
    Rot R;
    __device__ __forceinline__ Raw raw(int64_t j) const
    {
        Raw r{};
#pragma unroll
        for (int i = 0; i < 3; ++i) r.x[i] = pos[3 * j + i];
        if (CH != 3) r.n = nuc[j];
        if (CH != 1) {
#pragma unroll
            for (int i = 0; i < 3; ++i) r.m[i] = mag[3 * j + i];
        }
        return r;
    }
    __device__ __forceinline__ cblk::Point<CH> point(const Raw &r) const
    {
        auto row = [&](int i, const double (&v)[3]) {
            return R.m[3 * i] * v[0] + R.m[3 * i + 1] * v[1] + R.m[3 * i + 2] * v[2];
        };
        cblk::Point<CH> p;
        p.m = row(1, r.x);
        p.n = row(2, r.x);
        if (CH != 3) p.w[0] = r.n;
        if (CH != 1) {
#pragma unroll
            for (int i = 0; i < 3; ++i) p.w[(CH == 4 ? 1 : 0) + i] = row(i, r.m);
        }
        return p;
    }
    __host__ __device__ __forceinline__ PointSource source() const { return PointSource{nullptr, pos, nuc, mag, R}; }
};

// Workgroups per CU: registers and LDS allow two, and three of the tiles of 4 x 16.
__host__ __device__ constexpr int polar_per_cu(int mt) { return mt > 0 ? 2 : 3; }

// One wave: one theta column, one row group, one point range.  Partials
// [split][row group][column][tile][half][4][64] (store == 0; [tile][2][64] of the 4 x 16
// tiles), or amp (1: written, 2: added).
template <int MT, int CH, int NW, class Loader>
__global__ __launch_bounds__(pblk::kThreads, polar_per_cu(MT)) void direct_polar_kernel(Loader ld, int64_t W,
                                                                                        int64_t per, PolGeom g,
                                                                                        int store,
                                                                                        double *__restrict__ out)
{
    __shared__ pblk::WaveSmem<MT, CH, NW> sm[pblk::kWaves];
    const int lane = threadIdx.x & 63, wave = cblk::wave_id();
    const int col = blockIdx.x * pblk::kWaves + wave, rg = blockIdx.y;
    if (col >= g.cols) return;  // no workgroup barriers below
    g.mid = pblk::Tiles<MT>::kOffsets;  // (a constant)
    const int64_t jbeg = (int64_t)blockIdx.z * per;
    const int64_t jend = min(W, jbeg + per);
    double sth, cth;
    sincos_cw((2.0 * 3.141592653589793 * (double)col) / (double)g.n_out, &sth, &cth);
    constexpr int N = pblk::Tiles<MT>::N;
    typename pblk::Tiles<MT>::T accC[N] = {}, accS[N] = {};
    pblk::accumulate<MT, CH, NW>(ld, jbeg, jend, sth, cth, g.dq, rg * g.na, sm[wave], accC, accS);
    const int64_t block = (((int64_t)blockIdx.z * g.nrg + rg) * g.cols + col) * N;
    unsigned bad = 0;  // NaN sums of this lane, two bits per tile half (or tile)
    // `which` (1, 2) of slot's sums vp, vm, put away unless NaN
    auto put = [&](int i, int slot, double2 vp, double2 vm, int which) {
        const int nan = which & (NW == CH ? pblk::which_nan(g, CH, rg, slot, pblk::lane_offset(g), vp, vm) : 0);
        bad |= (unsigned)nan << (2 * i);
        pblk::put_slot(out, g, CH, rg, col, slot, pblk::lane_offset(g), vp, vm, store == 2, which & ~nan);
    };
    if constexpr (MT > 0) {
        cblk::finish_whole<MT>(accC, accS, [&](int t, int h, double2 vp, double2 vm) {
            if (store != 0) return put(2 * t + h, 8 * t + 4 * h + (lane >> 4), vp, vm, 3);
            double *o = out + ((block + t) * 2 + h) * 256 + lane;
            o[0] = vp.x;
            o[64] = vp.y;
            o[128] = vm.x;
            o[192] = vm.y;
        });
    } else {
#pragma unroll
        for (int t = 0; t < N; ++t) {
            const double2 v = pblk::few_rows(accC[t], accS[t]);
            if (store != 0) {
                put(t, 2 * t + (lane >> 4 & 1), v, v, 1 + (lane >> 5));
                continue;
            }
            double *o = out + (block + t) * 128 + lane;
            o[0] = v.x;
            o[64] = v.y;
        }
    }
    while (NW == CH && __builtin_expect(bad != 0, 0)) {
        const int i = __builtin_ctz(bad) >> 1, which = (int)(bad >> (2 * i) & 3);
        const int slot = MT > 0 ? 4 * i + (lane >> 4) : 2 * i + (lane >> 4 & 1);
        bad &= ~(3u << (2 * i));
        double2 vp = make_double2(__builtin_nan(""), __builtin_nan("")), vm = vp;
        pblk::repair(g, ld.source(), jbeg, jend, CH, rg, slot, pblk::lane_offset(g), sth, cth, which, vp, vm);
        pblk::put_slot(out, g, CH, rg, col, slot, pblk::lane_offset(g), vp, vm, store == 2, which);
    }
}

// Fixed-order sum of the split partials, written (or added) to the pixels: blocks of a row
// group, column and tile half (tile of 4 x 16: FEW).
template <bool FEW>
__global__ __launch_bounds__(256) void polar_combine_kernel(const double *__restrict__ part, PolGeom g, int n, int CH,
                                                            int nsplit, PointSource src, int64_t W, int accumulate,
                                                            double *__restrict__ amp)
{
    constexpr int V = FEW ? 2 : 4;
    if (!FEW) g.mid = pblk::kRows / 2;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = (int)(idx & 63);
    const int64_t block = idx >> 6;
    const int64_t blocks = (int64_t)g.nrg * g.cols * n;
    if (block >= blocks) return;
    const int i = (int)(block % n);
    const int64_t rc = block / n;
    const double *p = part + block * (64 * V) + lane;
    double v[V] = {};
#pragma unroll 4
    for (int s = 0; s < nsplit; ++s, p += blocks * (64 * V)) {
#pragma unroll
        for (int k = 0; k < V; ++k) v[k] += p[64 * k];
    }
    const int rg = (int)(rc / g.cols), col = (int)(rc % g.cols);
    const int slot = FEW ? 2 * i + (lane >> 4 & 1) : 4 * i + (lane >> 4), which = FEW ? 1 + (lane >> 5) : 3;
    double2 vp = make_double2(v[0], v[1]), vm = make_double2(v[V - 2], v[V - 1]);
    const int nan = W > 0 ? which & pblk::which_nan(g, CH, rg, slot, pblk::lane_offset(g), vp, vm) : 0;
    if (__builtin_expect(nan != 0, 0)) {
        double sth, cth;
        sincos_cw((2.0 * 3.141592653589793 * (double)col) / (double)g.n_out, &sth, &cth);
        pblk::repair(g, src, 0, W, CH, rg, slot, pblk::lane_offset(g), sth, cth, nan, vp, vm);
    }
    pblk::put_slot(amp, g, CH, rg, col, slot, pblk::lane_offset(g), vp, vm, accumulate != 0, which);
}

// ---------------------------------------------------------------------------
// Work split.
// ---------------------------------------------------------------------------
int default_polar_shape(const Detector &d)
{
    if (d.n0 <= 32) return 1;
    if (d.n0 <= 64) return 0;
    return d.n0 <= 128 ? 2 : d.n0 <= 256 ? 3 : 4;
}

void polar_geometry(const Detector &d, int channels, int shape, PolGeom &g, int &mt)
{
    g.n0 = d.n0;
    g.n_out = d.n_theta;
    // theta + pi is a column of an even detector: its sums are conjugates
    g.nh = d.n_theta % 2 == 0 ? d.n_theta / 2 : 0;
    g.cols = g.nh > 0 ? g.nh : d.n_theta;
    const int blocks = (d.n0 + pblk::kRows - 1) / pblk::kRows;
    const int cap = std::min(shape_blocks(shape), std::min(pblk::kMaxNA, 8 * cblk::kMaxMT / channels));
    g.nrg = (blocks + cap - 1) / cap;
    g.na = (blocks + g.nrg - 1) / g.nrg;
    g.mid = pblk::kRows / 2;
    g.dq = d.step0;
    mt = (g.na * channels + 7) / 8;
}

// The direct sums' tiles: of 4 x 16 (PolarPlan::mt <= 0) where a wave's slots fit two.
static void direct_polar_geometry(const Detector &d, int channels, PolarPlan &p)
{
    polar_geometry(d, channels, p.shape, p.g, p.mt);
    if (p.g.na * channels > 4) return;
    p.mt = p.g.na * channels <= 2 ? 0 : -1;
    if (d.n0 <= 16) {  // offsets of one half block
        p.mt -= 2;
        p.g.mid = 8;
    }
}

static size_t polar_split_bytes(const PolGeom &g, int mt)
{
    return (size_t)g.nrg * g.cols * (mt > 0 ? mt * 512 : pblk::few_tiles(mt) * 128) * sizeof(double);
}

static void polar_splits(PolarPlan &p, int64_t W, int64_t target, size_t max_partial)
{
    const int64_t blocks = (int64_t)((p.g.cols + pblk::kWaves - 1) / pblk::kWaves) * p.g.nrg;
    int64_t want = std::min<int64_t>(target / blocks, (W + pblk::kChunk - 1) / pblk::kChunk);
    if (max_partial > 0)
        want = std::min<int64_t>(want, (int64_t)(max_partial / std::max<size_t>(1, polar_split_bytes(p.g, p.mt))));
    want = std::max<int64_t>(1, std::min<int64_t>(want, 65535));
    int64_t per = (W + want - 1) / want;
    per = std::max<int64_t>(4, (per + 3) / 4 * 4);
    p.per = per;
    p.nsplit = (int)std::max<int64_t>(1, (W + per - 1) / per);
}

// Rounds of the workgroups that fit the chip times the cycles of one split (a matrix
// instruction holds its SIMD's FP64 pipe 64 cycles, one of 4 x 16 20, the tables of a chunk
// take about 150 vector instructions of 4), plus the partial sums at about 1700 bytes a cycle.
static PolarPlan polar_default_plan(const Detector &d, int64_t W, int channels, size_t max_partial, int64_t target)
{
    PolarPlan best{};
    double best_cost = -1.0;
    for (int rounds = 1; rounds <= 8; ++rounds) {
        PolarPlan p{};
        p.channels = channels;
        p.shape = default_polar_shape(d);
        direct_polar_geometry(d, channels, p);
        const int64_t blocks = (int64_t)((p.g.cols + pblk::kWaves - 1) / pblk::kWaves) * p.g.nrg;
        const int per_cu = polar_per_cu(p.mt);
        polar_splits(p, W, target > 0 ? target : std::max<int64_t>(256 * per_cu * rounds, blocks), max_partial);
        const double pts = (double)std::min<int64_t>(p.per, std::max<int64_t>(W, 1));
        const double step = p.mt > 0 ? 132.0 * p.mt : (p.g.mid == 8 ? 22.0 : 44.0) * pblk::few_tiles(p.mt);
        const double cycles = per_cu * (3000.0 + std::ceil(pts / pblk::kChunk) * 700.0 +
                                        std::ceil(pts / 4.0) * (step + 40.0));
        const double bytes = (double)polar_split_bytes(p.g, p.mt) * p.nsplit;
        const double cost = std::ceil((double)(blocks * p.nsplit) / (256.0 * per_cu)) * cycles +
                            (p.nsplit > 1 ? 8000.0 + 2.0 * bytes / 1700.0 : 0.0);
        if (best_cost < 0.0 || cost < 0.98 * best_cost) {
            best_cost = cost;
            best = p;
        }
    }
    return best;
}

TuneShape default_polar_tune(const Detector &d, int64_t W)
{
    const PolarPlan p = polar_default_plan(d, W, 4, 0, env_target());
    return TuneShape{p.shape, (int)((int64_t)((p.g.cols + pblk::kWaves - 1) / pblk::kWaves) * p.g.nrg * p.nsplit)};
}

PolarPlan plan_direct_polar(const Detector &d, int64_t W, int channels, bool hermitian, size_t max_partial)
{
    Detector key = d;
    if (hermitian) key.n1 = d.n1 / 2;
    TuneShape ts{};
    if (!tuned_shape(kTuneDirect, key, W, &ts))
        return polar_default_plan(d, W, channels, max_partial, env_target());
    if (ts.target == 0) ts.target = default_polar_tune(d, W).target;
    PolarPlan p{};
    p.channels = channels;
    p.shape = ts.shape;
    direct_polar_geometry(d, channels, p);
    polar_splits(p, W, ts.target, max_partial);
    return p;
}

size_t polar_partial_bytes(const PolarPlan &p)
{
    return p.nsplit > 1 ? polar_split_bytes(p.g, p.mt) * (size_t)p.nsplit : 0;
}

template <int CH, int NW, class Loader>
static void launch_polar_tiles(const Loader &ld, int64_t W, const PolarPlan &p, int store, double *out,
                               hipStream_t s)
{
    const dim3 grid((p.g.cols + pblk::kWaves - 1) / pblk::kWaves, p.g.nrg, p.nsplit), block(pblk::kThreads);
    // at most 16 row blocks: 2 CH tiles
#define NUMAG_LAUNCH_POLAR(MT)   \
    case MT:                     \
        if constexpr (MT <= 2 * CH && (MT > 0 || CH <= 2 * pblk::few_tiles(MT)) && (MT != -3 || CH > 2)) \
            hipLaunchKernelGGL((direct_polar_kernel<MT, CH, NW, Loader>), grid, block, 0, s, ld, W, p.per, p.g, store, out); \
        break
    switch (p.mt) {
        NUMAG_LAUNCH_POLAR(-3);
        NUMAG_LAUNCH_POLAR(-2);
        NUMAG_LAUNCH_POLAR(-1);
        NUMAG_LAUNCH_POLAR(0);
        NUMAG_LAUNCH_POLAR(1);
        NUMAG_LAUNCH_POLAR(2);
        NUMAG_LAUNCH_POLAR(3);
        NUMAG_LAUNCH_POLAR(4);
        NUMAG_LAUNCH_POLAR(5);
        NUMAG_LAUNCH_POLAR(6);
        NUMAG_LAUNCH_POLAR(7);
        NUMAG_LAUNCH_POLAR(8);
    }
#undef NUMAG_LAUNCH_POLAR
}

// src, W: the points, for results that are not finite (W = 0: left as they are).
static int combine_polar(const PolarPlan &p, const PointSource &src, int64_t W, const double *partial, double *amp,
                         int accumulate, hipStream_t s)
{
    NUMAG_HIP_CHECK(hipGetLastError());
    if (p.nsplit <= 1) return NUMAG_OK;
    const int n = p.mt > 0 ? 2 * p.mt : pblk::few_tiles(p.mt);  // tile halves, or tiles of 4 x 16
    const dim3 grid((unsigned)(((int64_t)p.g.nrg * p.g.cols * n * 64 + 255) / 256));
    if (p.mt > 0)
        hipLaunchKernelGGL((polar_combine_kernel<false>), grid, dim3(256), 0, s, partial, p.g, n, p.channels, p.nsplit,
                           src, W, accumulate, amp);
    else
        hipLaunchKernelGGL((polar_combine_kernel<true>), grid, dim3(256), 0, s, partial, p.g, n, p.channels, p.nsplit,
                           src, W, accumulate, amp);
    NUMAG_HIP_CHECK(hipGetLastError());
    return NUMAG_OK;
}

int launch_direct_polar(const PointRec *pts, int64_t W, const PolarPlan &p, double *partial, double *amp,
                        int accumulate, hipStream_t s)
{
    const int store = p.nsplit > 1 ? 0 : (accumulate ? 2 : 1);
    {
        TimedLaunch timed(NUMAG_KERNEL_DIRECT, s);
        double *out = p.nsplit > 1 ? partial : amp;
        switch (p.channels) {
            case 1: launch_polar_tiles<1, 1>(PolarRecLoader<1, 1>{pts}, W, p, store, out, s); break;
            case 3: launch_polar_tiles<3, 3>(PolarRecLoader<3, 3>{pts}, W, p, store, out, s); break;
            default: launch_polar_tiles<4, 4>(PolarRecLoader<4, 4>{pts}, W, p, store, out, s); break;
        }
    }
    return combine_polar(p, PointSource{pts, nullptr, nullptr, nullptr, Rot{}}, W, partial, amp, accumulate, s);
}

int launch_sample_polar(const double *pos, const double *nuc, const double *mag, const Rot &R, int64_t W,
                        const PolarPlan &p, double *partial, double *amp, hipStream_t s)
{
    const int store = p.nsplit > 1 ? 0 : 1;
    {
        TimedLaunch timed(NUMAG_KERNEL_DIRECT, s);
        double *out = p.nsplit > 1 ? partial : amp;
        switch (p.channels) {
            case 1: launch_polar_tiles<1, 1>(PolarSampleLoader<1>{pos, nuc, mag, R}, W, p, store, out, s); break;
            case 3: launch_polar_tiles<3, 3>(PolarSampleLoader<3>{pos, nuc, mag, R}, W, p, store, out, s); break;
            default: launch_polar_tiles<4, 4>(PolarSampleLoader<4>{pos, nuc, mag, R}, W, p, store, out, s); break;
        }
    }
    return combine_polar(p, PointSource{nullptr, pos, nuc, mag, R}, W, partial, amp, 0, s);
}

int launch_polar_pairs(const PairRec *pts, int64_t n, const PolarPlan &p, double *partial, double *amp, hipStream_t s)
{
    const int store = p.nsplit > 1 ? 0 : 1;
    {
        TimedLaunch timed(NUMAG_KERNEL_DIRECT, s);
        double *out = p.nsplit > 1 ? partial : amp;
        switch (p.channels) {
            case 1: launch_polar_tiles<1, 2>(PolarRecLoader<1, 2>{pts}, n, p, store, out, s); break;
            case 2: launch_polar_tiles<2, 4>(PolarRecLoader<2, 4>{pts}, n, p, store, out, s); break;
            case 3: launch_polar_tiles<3, 6>(PolarRecLoader<3, 6>{pts}, n, p, store, out, s); break;
            default: launch_polar_tiles<4, 8>(PolarRecLoader<4, 8>{pts}, n, p, store, out, s); break;
        }
    }
    return combine_polar(p, PointSource{}, 0, partial, amp, 0, s);
}

}  // namespace numag
