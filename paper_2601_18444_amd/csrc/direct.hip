// Direct Fourier sums on gfx950, Cartesian detector: the general (any point
// cloud, any rotation) path, plus the point preparation and the split combine
// shared with the polar path (polar.hip).
//
// Sums (Sec. 3.3, DSFT):  S_c(q_p) = sum_j w_{j,c} exp(-i q_p . X_j),  q = (0, q_y, q_z).
//
// The phase separates in the lab frame, exp(-i (q_y Y + q_z Z)) =
// exp(-i q_y Y) exp(-i q_z Z), and the detector is symmetric about q = 0: the sums are
// real contractions over points on the FP64 matrix cores (cartesian_block.h), four
// multiply-adds per point and pixel for the four channels.  Everything is FP64 (FP32
// phasors lose the 1e-5 gate at 10^-6 of the maximum on 2.6e5-point samples, however
// the sums are folded).
//
// Work is split over point ranges (split-K); a fixed-order FP64 combine sums the
// partial results, so results are bitwise reproducible.
//
// Measured, kernel time before (a lane walking 8 pixels of a row with a two-term phasor
// recurrence, 10.5 vector FP64 instructions per term) and now:
//   262,144 points, 256 x 256 pixels   6.30 -> 2.12 ms (65 of the card's 74.7 TFLOP/s)
//   30,011 points, 201 x 333, 3 channels  0.64 (half detector) -> 0.265 ms
//   4,169 points, 128 x 128               64 -> 29 us;  500 points, 48 x 81  53 -> 12 us
// Of the 2.12 ms, 1.84 are the multiply-adds at the measured matrix rate and 0.19 the
// generation of the phasor tables (0.77 with one column block per workgroup instead of
// eight: the table of row operands is shared by the waves of a workgroup).  Letting
// half of the waves generate while the others sum gained nothing (2.15 ms): vector and
// matrix FP64 instructions share one pipe.
#include <algorithm>
#include <cmath>

#include "cartesian_block.h"

namespace numag {


Detector make_detector(const numag_qgrid &g)
{
    Detector d{};
    d.kind = g.kind;
    d.n0 = g.n0;
    d.n1 = g.n1;
    d.n_theta = g.n1;
    d.qmax = g.qmax;
    if (g.kind == NUMAG_GRID_CARTESIAN) {
        d.step0 = g.n0 > 1 ? (2.0 * g.qmax) / (double)(g.n0 - 1) : 0.0;
        d.step1 = g.n1 > 1 ? (2.0 * g.qmax) / (double)(g.n1 - 1) : 0.0;
        d.origin0 = g.n0 > 1 ? -g.qmax : 0.0;
        d.origin1 = g.n1 > 1 ? -g.qmax : 0.0;
    } else {
        d.step0 = g.n0 > 1 ? g.qmax / (double)(g.n0 - 1) : 0.0;
        d.step1 = 0.0;  // theta_m = (2 pi m) / n_theta, computed as written
        d.origin0 = 0.0;
        d.origin1 = 0.0;
    }
    return d;
}

// ---------------------------------------------------------------------------
// sample assembly and rotation (Sec. 3.2): X = R (x + r^k), w' = (n, R m).
// ---------------------------------------------------------------------------
// Lab-frame record of point j at sample-frame position x: X = R x (only Y, Z enter
// the phase), weights (n, R m).
__device__ __forceinline__ PointRec point_record(const double (&x)[3], const Rot &R, const double *__restrict__ nuc,
                                                 const double *__restrict__ mag, int64_t j)
{
    PointRec r;
    r.Y = R.m[3] * x[0] + R.m[4] * x[1] + R.m[5] * x[2];
    r.Z = R.m[6] * x[0] + R.m[7] * x[1] + R.m[8] * x[2];
    r.w[0] = nuc != nullptr ? nuc[j] : 0.0;
    double m0 = 0.0, m1 = 0.0, m2 = 0.0;
    if (mag != nullptr) {
        m0 = mag[3 * j + 0];
        m1 = mag[3 * j + 1];
        m2 = mag[3 * j + 2];
    }
    r.w[1] = R.m[0] * m0 + R.m[1] * m1 + R.m[2] * m2;
    r.w[2] = R.m[3] * m0 + R.m[4] * m1 + R.m[5] * m2;
    r.w[3] = R.m[6] * m0 + R.m[7] * m1 + R.m[8] * m2;
    r.pad[0] = r.pad[1] = 0.0;
    return r;
}

// Objects whose offsets r^k one preparation launch adds: the points
// [start[0], start[n]) belong to objects k0 .. k0 + n - 1, object k0 + i holding
// [start[i], start[i + 1]).  Passed by value, so no host-to-device copy is needed.
constexpr int kObjGroup = 64;
struct ObjGroup {
    int n;
    int64_t k0;
    int64_t start[kObjGroup + 1];
};

// Writes out[j - out_base] for the points j in [g.start[0], g.start[g.n]);
// obj_pos == nullptr: no object offsets.
__global__ void prepare_points_kernel(const double *__restrict__ pos, const double *__restrict__ nuc,
                                      const double *__restrict__ mag, int reg, numag_regular rg, ObjGroup g,
                                      const double *__restrict__ obj_pos, Rot R, int64_t out_base,
                                      PointRec *__restrict__ out)
{
    const int64_t j = g.start[0] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= g.start[g.n]) return;
    double x[3];
    if (reg) {
        int64_t nyz = (int64_t)rg.n[1] * rg.n[2];
        int64_t ix = j / nyz, rem = j % nyz;
        int64_t iy = rem / rg.n[2], iz = rem % rg.n[2];
        x[0] = rg.origin[0] + (double)ix * rg.step[0];
        x[1] = rg.origin[1] + (double)iy * rg.step[1];
        x[2] = rg.origin[2] + (double)iz * rg.step[2];
    } else {
        x[0] = pos[3 * j + 0];
        x[1] = pos[3 * j + 1];
        x[2] = pos[3 * j + 2];
    }
    if (obj_pos != nullptr) {
        int lo = 0, hi = g.n - 1;  // largest i with start[i] <= j
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (g.start[mid] <= j) lo = mid; else hi = mid - 1;
        }
        const int64_t k = g.k0 + lo;
        x[0] += obj_pos[3 * k + 0];
        x[1] += obj_pos[3 * k + 1];
        x[2] += obj_pos[3 * k + 2];
    }
    out[j - out_base] = point_record(x, R, nuc, mag, j);
}

int launch_prepare_points(const double *pos, const double *nuc, const double *mag, int64_t j_lo, int64_t j_hi,
                          const numag_regular *regular, const int64_t *h_offsets, int64_t K,
                          const double *obj_pos, const Rot &R, PointRec *out, hipStream_t s)
{
    if (j_hi <= j_lo) return NUMAG_OK;
    numag_regular rg{};
    if (regular != nullptr) rg = *regular;
    const int tpb = 256;
    auto launch = [&](const ObjGroup &g) -> int {
        const int64_t n = g.start[g.n] - g.start[0];
        if (n <= 0) return NUMAG_OK;
        hipLaunchKernelGGL(prepare_points_kernel, dim3((unsigned)((n + tpb - 1) / tpb)), dim3(tpb), 0, s, pos, nuc,
                           mag, regular != nullptr ? 1 : 0, rg, g, obj_pos, R, j_lo, out);
        NUMAG_HIP_CHECK(hipGetLastError());
        return NUMAG_OK;
    };
    ObjGroup g{};
    if (obj_pos == nullptr || K <= 1 || h_offsets == nullptr) {
        g.n = 1;
        g.k0 = 0;
        g.start[0] = j_lo;
        g.start[1] = j_hi;
        return launch(g);
    }
    // first object holding a point >= j_lo: the last k with off[k] <= j_lo among non-empty objects
    int64_t k = std::upper_bound(h_offsets, h_offsets + K + 1, j_lo) - h_offsets - 1;
    while (k < K && h_offsets[k + 1] <= j_lo) ++k;
    while (k < K && h_offsets[k] < j_hi) {
        g.n = 0;
        g.k0 = k;
        while (g.n < kObjGroup && k < K && h_offsets[k] < j_hi) {
            g.start[g.n] = std::max(h_offsets[k], j_lo);
            ++g.n;
            ++k;
        }
        g.start[g.n] = std::min(h_offsets[k], j_hi);
        const int rc = launch(g);
        if (rc != NUMAG_OK) return rc;
    }
    return NUMAG_OK;
}

// ---------------------------------------------------------------------------
// Cartesian direct sum.
// ---------------------------------------------------------------------------
template <int CH>
struct PrepLoader {
    using Raw = cblk::Point<CH>;
    const PointRec *__restrict__ pts;
    int swapped;
    __device__ __forceinline__ Raw raw(int64_t j) const
    {
        const PointRec &r = pts[j];
        Raw p;
        p.m = swapped ? r.Z : r.Y;
        p.n = swapped ? r.Y : r.Z;
#pragma unroll
        for (int c = 0; c < CH; ++c) p.w[c] = r.w[cblk::ch_first<CH>() + c];
        return p;
    }
    __device__ __forceinline__ cblk::Point<CH> point(const Raw &r) const { return r; }
    __host__ __device__ __forceinline__ PointSource source() const { return PointSource{pts, nullptr, nullptr, nullptr, Rot{}}; }
};

// Points straight from a sample (no object offsets), the record's arithmetic.
template <int CH>
struct SampleLoader {
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
        const double Y = row(1, r.x), Z = row(2, r.x);
        p.m = swapped ? Z : Y;
        p.n = swapped ? Y : Z;
        if (CH != 3) p.w[0] = r.n;
        if (CH != 1) {
#pragma unroll
            for (int i = 0; i < 3; ++i) p.w[(CH == 4 ? 1 : 0) + i] = row(i, r.m);
        }
        return p;
    }
    __host__ __device__ __forceinline__ PointSource source() const { return PointSource{nullptr, pos, nuc, mag, R}; }
};

// Where a workgroup's sums go: partials [split][row block][column block][tile][half][4][64]
// (PARTIAL; combined below), or straight into amp (written, or with `add` added).  Two
// kernels: a small call waits for its instructions to be fetched (4,169 points, 128 x 128:
// the partial sums' kernel 30.3 us with both in one, 43 kB, 28.3 without, 18 kB).
template <int MT, int CH, bool PARTIAL, class Loader>
__global__ __launch_bounds__(cblk::kThreads, 2) void direct_cartesian_kernel(Loader ld, int64_t W, int64_t per,
                                                                              int nsplit, CartGeom g, int add,
                                                                              double *__restrict__ out)
{
    __shared__ cblk::Smem<MT> sm;
    const int lane = threadIdx.x & 63;
    const int zb0 = (int)(blockIdx.x / nsplit) * g.nz, rb = blockIdx.y, split = (int)(blockIdx.x % nsplit);
    const int64_t jbeg = (int64_t)split * per;
    const int64_t jend = min(W, jbeg + per);
    cblk::v4d accC[MT], accS[MT];
    cblk::zero<MT>(accC, accS);
    typename Loader::Raw p, q;
    cblk::first_points(ld, jbeg, jend, p, q);
    cblk::accumulate<MT, CH>(ld, jbeg, jend, g, rb, zb0, sm, p, q, accC, accS);
    const int zb = zb0 + cblk::wave_id() % g.nz;
    unsigned bad = 0;  // NaN sums of this lane, two bits per tile half
    cblk::finish<MT>(g, zb0, sm, accC, accS, [&](int t, int h, double2 vp, double2 vm) {
        if (PARTIAL) {
            double *o = out + (((((int64_t)split * g.nrb + rb) * g.nzb + zb) * MT + t) * 2 + h) * 256 + lane;
            o[0] = vp.x;
            o[64] = vp.y;
            o[128] = vm.x;
            o[192] = vm.y;
        } else {
            const cblk::CellPixels x = cblk::cell_pixels(g, CH, rb, zb, 8 * t + 4 * h + (lane >> 4), lane & 15);
            if (x.ok) {
                const int nan = cblk::which_nan(vp, vm);
                bad |= (unsigned)nan << (2 * (2 * t + h));
                cblk::put_slot(out, x, CH, vp, vm, add != 0, 3 & ~nan);
            }
        }
    });
    while (!PARTIAL && __builtin_expect(bad != 0, 0)) {
        const int i = __builtin_ctz(bad) >> 1, which = (int)(bad >> (2 * i) & 3);
        bad &= ~(3u << (2 * i));
        const int s = 4 * i + (lane >> 4);
        const cblk::CellPixels x = cblk::cell_pixels(g, CH, rb, zb, s, lane & 15);
        const int ch = cblk::ch_first<CH>() + x.c;
        double2 vp = make_double2(__builtin_nan(""), __builtin_nan("")), vm = vp;
        cblk::repair(g, ld.source(), jbeg, jend, rb * g.na + s / CH, cblk::kOff * zb + (lane & 15), ch, which, vp, vm);
        cblk::put_cell(out, x, ch, vp, vm, add != 0, which);
    }
}

// Fixed-order sum of the split partials, written (or added) to the pixels.
__global__ __launch_bounds__(256, 8) void cart_combine_kernel(const double *__restrict__ part, CartGeom g, int MT, int CH,
                                                           int nsplit, PointSource src, int64_t W, int accumulate,
                                                           double *__restrict__ amp)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = (int)(idx & 63);
    const int64_t block = idx >> 6;  // (row block, column block, tile, half)
    const int64_t blocks = (int64_t)g.nrb * g.nzb * MT * 2;
    if (block >= blocks) return;
    const int h = (int)(block & 1), t = (int)((block >> 1) % MT);
    const int64_t rz = (block >> 1) / MT;
    const int rb = (int)(rz / g.nzb), zb = (int)(rz % g.nzb), slot = 8 * t + 4 * h + (lane >> 4);
    const cblk::CellPixels x = cblk::cell_pixels(g, CH, rb, zb, slot, lane & 15);
    if (!x.ok) return;
    const double *p = part + block * 256 + lane;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int s = 0; s < nsplit; ++s, p += blocks * 256) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += p[64 * k];
    }
    double2 vp = make_double2(v[0], v[1]), vm = make_double2(v[2], v[3]);
    const int nan = cblk::which_nan(vp, vm);
    if (__builtin_expect(nan != 0, 0))
        cblk::repair(g, src, 0, W, rb * g.na + slot / CH, cblk::kOff * zb + (lane & 15), (CH == 3 ? 1 : 0) + x.c, nan,
                     vp, vm);
    cblk::put_slot(amp, x, CH, vp, vm, accumulate != 0);
}

int env_target()
{
    static const int cached = [] {  // thread-safe one-time initialisation
        const char *e = getenv("NUMAG_TARGET_WGS");
        const int v = e != nullptr ? atoi(e) : 0;
        return v > 0 ? v : 0;
    }();
    return cached;
}

// ---------------------------------------------------------------------------
// Work split of the Cartesian sums.
// ---------------------------------------------------------------------------
constexpr int64_t kCartCUs = 256;     // one workgroup of 8 waves per CU at a time
constexpr int kMaxSplits = 65535;

// Rows, columns and strides of the cells, row blocks for `channels`, with the detector's
// rows (sw = 0) or columns packed into the matrix rows; the number of matrix tiles.
static int64_t oriented_geometry(const Detector &d, int channels, int sw, CartGeom &g, int &mt)
{
    g.nM = sw ? d.n1 : d.n0;
    g.nN = sw ? d.n0 : d.n1;
    g.A = (g.nM + 1) / 2;
    g.B = (g.nN + 1) / 2;
    const int per_block = 8 * cblk::kMaxMT / channels;  // |q_M| values of a full row block
    g.nrb = (g.A + per_block - 1) / per_block;
    g.na = (g.A + g.nrb - 1) / g.nrb;
    mt = (g.na * channels + 7) / 8;
    g.nzb = (g.B + cblk::kOff - 1) / cblk::kOff;
    g.swapped = sw;
    g.firstM = g.nM % 2 == 0 ? 0.5 : 0.0;
    g.stepM = sw ? d.step1 : d.step0;
    g.firstN = g.nN % 2 == 0 ? 0.5 : 0.0;
    g.stepN = sw ? d.step0 : d.step1;
    g.strideM = sw ? 1 : d.n1;
    g.strideN = sw ? d.n1 : 1;
    return (int64_t)g.nrb * mt * g.nzb;
}

// The orientation with fewer matrix tiles (thin detectors put their short axis into the
// packed rows).
void cart_geometry(const Detector &d, int channels, CartGeom &g, int &mt)
{
    CartGeom t{};
    int m = 0;
    const int64_t rows = oriented_geometry(d, channels, 0, g, mt);
    if (oriented_geometry(d, channels, 1, t, m) >= rows) return;
    g = t;
    mt = m;
}

// Column blocks per workgroup of a launch shape (the labels are those tables hold).
int cart_nz(int shape) { return shape == 32 ? 8 : shape == 16 ? 4 : shape == 64 ? 2 : 1; }

static size_t cart_split_bytes(const CartGeom &g, int mt) { return (size_t)g.nrb * g.nzb * mt * 512 * sizeof(double); }

// Point splits: a launch of about `target` workgroups, each split a multiple of 4
// points (one matrix step), at least one step per point group of a workgroup.
static void cart_splits(CartPlan &p, int64_t W, int64_t target, size_t max_partial)
{
    p.col_groups = (p.g.nzb + p.g.nz - 1) / p.g.nz;
    const int64_t blocks = (int64_t)p.col_groups * p.g.nrb;
    int64_t want = target / blocks;
    want = std::min<int64_t>(want, (W + 4 * (cblk::kWaves / p.g.nz) - 1) / (4 * (cblk::kWaves / p.g.nz)));
    if (max_partial > 0)
        want = std::min<int64_t>(want, (int64_t)(max_partial / std::max<size_t>(1, cart_split_bytes(p.g, p.mt))));
    want = std::max<int64_t>(1, std::min<int64_t>(want, kMaxSplits));
    int64_t per = (W + want - 1) / want;
    per = std::max<int64_t>(4, (per + 3) / 4 * 4);
    p.per = per;
    p.nsplit = (int)std::max<int64_t>(1, (W + per - 1) / per);
}

// Estimates in cycles.  A matrix instruction holds the FP64 pipe of its SIMD 66 cycles; the
// tables of a chunk with what comes with them (loads, barrier, the waits that the sums do
// not cover) were fitted to the times of 50,000 points on 150 x 150 pixels with 1, 2, 4 and
// 8 column blocks per workgroup; the object kernel, which rotates the points as well, takes
// 3280 (16 particles x 24 rotations, 128 x 128 pixels).
static double table_cycles(const CartGeom &g, int channels)
{
    return 2.0 * (550.0 + std::ceil(g.na / 16.0) * (410.0 + 10.0 * channels));
}
// one step (4 points) of the busiest SIMD of a workgroup with `blocks` column blocks
static double step_cycles(const CartGeom &g, int mt, int blocks)
{
    return (g.nz == 8 ? (blocks > 4 ? 2.0 : 1.0) : g.nz / 4.0) * (132.0 * mt + 60.0);
}

// Estimated time of a plan: partial sums move at about 1700 bytes a cycle each way.
// Workgroups whose column blocks run out are cheaper and are launched last.
static double cart_cost(const CartPlan &p, int64_t W)
{
    const double pts = (double)std::min<int64_t>(p.per, std::max<int64_t>(W, 1));
    const double steps = std::ceil(pts / 4.0);
    const double fixed = 4000.0 + std::ceil(pts / cblk::kChunk) * table_cycles(p.g, p.channels) +
                         (p.g.nz < 8 ? 400.0 * p.mt : 0.0);
    const double full = (double)(p.g.nzb / p.g.nz) * p.g.nrb * p.nsplit, last = (double)p.g.nrb * p.nsplit;
    const int rest = p.g.nzb % p.g.nz;
    const double cf = fixed + steps * step_cycles(p.g, p.mt, p.g.nz), cl = fixed + steps * step_cycles(p.g, p.mt, rest);
    double t = 0.0;
    if (rest == 0) {
        t = std::ceil(full / (double)kCartCUs) * cf;
    } else if (full == 0.0) {
        t = std::ceil(last / (double)kCartCUs) * cl;
    } else if (full + last <= (double)kCartCUs) {
        t = cf;
    } else {
        t = std::max(std::ceil(full / (double)kCartCUs) * cf, (full * cf + last * cl) / (double)kCartCUs + 0.5 * cl);
    }
    const double bytes = (double)cart_split_bytes(p.g, p.mt) * p.nsplit;
    return t + (p.nsplit > 1 ? 8000.0 + 2.0 * bytes / 1700.0 : 0.0);
}

constexpr double kObjTables = 3280.0;

// Cycles of a chunk of the object kernel, summed over the workgroups of a detector.
static double chunk_cycles(const CartGeom &g, int mt)
{
    const int full = g.nzb / g.nz, rest = g.nzb % g.nz;
    const double steps = cblk::kChunk / 4.0, tables = kObjTables;
    return g.nrb * (full * (tables + steps * step_cycles(g, mt, g.nz)) +
                    (rest > 0 ? tables + steps * step_cycles(g, mt, rest) : 0.0));
}

double cart_objects_geometry(const Detector &d, int shape, CartGeom &g, int &mt, double *group)
{
    CartGeom t[2]{};
    int m[2];
    double c[2];
    for (int sw = 0; sw < 2; ++sw) {
        oriented_geometry(d, 4, sw, t[sw], m[sw]);
        t[sw].nz = cart_nz(shape);
        c[sw] = chunk_cycles(t[sw], m[sw]);
    }
    const int k = c[1] < c[0] ? 1 : 0;
    g = t[k];
    mt = m[k];
    if (group != nullptr) {
        group[0] = kObjTables + cblk::kChunk / 4.0 * step_cycles(g, mt, g.nz);
        group[1] = kObjTables + cblk::kChunk / 4.0 * step_cycles(g, mt, g.nzb % g.nz);
    }
    return c[k];
}

// The cheapest of the plans for `shapes` and `targets` (0: 1 to 4 rounds of the CUs), in both
// orientations unless one takes a quarter more tiles.  Column blocks that do not fill the
// last workgroup, and an orientation with fewer tiles but more of those, cost most where
// one round is all there is; measured against one round of equal workgroups in the
// orientation with fewer tiles: 20,000 points, 500 x 600 pixels 961 -> 823 us; 8,000,
// 999 x 801 1047 -> 920; 50,000, 150 x 150 285 -> 258; 4,169, 128 x 128 unchanged.
template <size_t N>
static CartPlan cheapest_plan(const Detector &d, int64_t W, int channels, size_t max_partial, const int (&shapes)[N],
                              int64_t target)
{
    CartPlan best{};
    double best_cost = -1.0;
    CartPlan o[2]{};
    int64_t tiles[2];
    for (int sw = 0; sw < 2; ++sw) {
        o[sw].channels = channels;
        tiles[sw] = oriented_geometry(d, channels, sw, o[sw].g, o[sw].mt);
    }
    const int first = tiles[1] < tiles[0] ? 1 : 0;
    for (int k = 0; k < 2; ++k) {
        CartPlan &p = o[k == 0 ? first : 1 - first];
        if (k == 1 && 4 * tiles[1 - first] > 5 * tiles[first]) break;
        for (int shape : shapes) {
            p.shape = shape;
            p.g.nz = cart_nz(shape);
            if (N > 1 && p.g.nz > 2 && p.g.nz / 2 >= p.g.nzb) continue;  // column blocks that no wave would have
            const int64_t blocks = (int64_t)((p.g.nzb + p.g.nz - 1) / p.g.nz) * p.g.nrb;
            for (int rounds = 1; rounds <= 4; ++rounds) {
                cart_splits(p, W, target > 0 ? target : std::max<int64_t>(rounds * kCartCUs, blocks), max_partial);
                const double cost = cart_cost(p, W);
                if (best_cost < 0.0 || cost < 0.98 * best_cost) {
                    best_cost = cost;
                    best = p;
                }
                if (target > 0) break;
            }
        }
    }
    return best;
}

static CartPlan cart_default_plan(const Detector &d, int64_t W, int channels, size_t max_partial)
{
    return cheapest_plan(d, W, channels, max_partial, {32, 16, 64, 8}, env_target());
}

double cart_default_cost(const Detector &d, int64_t W, int channels)
{
    const CartPlan p = cart_default_plan(d, W, channels, 0);
    // (the combination adds the splits one after another, which counts for small detectors)
    return cart_cost(p, W) + (p.nsplit > 1 ? 140.0 * p.nsplit : 0.0);
}

TuneShape default_tune_shape(int kernel, const Detector &d, int64_t W)
{
    switch (kernel) {
        case kTuneDirect: {
            if (d.kind == NUMAG_GRID_POLAR) return default_polar_tune(d, W);
            const CartPlan p = cart_default_plan(d, W, 4, 0);
            return TuneShape{p.shape, (int)((int64_t)p.col_groups * p.g.nrb * p.nsplit)};
        }
        case kTuneAdjoint:
            return TuneShape{0, default_adjoint_target(d, W)};
        default: {  // the persistent object kernel: shapes as for the direct sums, work items
            // (eight per workgroup or wave that fits the chip: the largest go first, so the
            // last ones even the load out; 16 particles x 24 rotations on 128 x 128 take
            // 6.0 ms with half as many, 5.74 with these, 5.64 with twice as many)
            if (d.kind == NUMAG_GRID_POLAR) return TuneShape{default_polar_shape(d), 16384};
            // column blocks per workgroup: the fewest cycles of a chunk (objects.hip, where
            // the objects are known, also weighs how evenly their items fill the chip)
            CartGeom g{};
            int mt = 0, best = 32;
            double least = -1.0;
            for (int shape : {16, 32, 64, 8}) {
                const double c = cart_objects_geometry(d, shape, g, mt, nullptr);
                if (least >= 0.0 && c >= least) continue;
                least = c;
                best = shape;
            }
            return TuneShape{best, 2048};
        }
    }
}

TuneShape current_tune_shape(int kernel, const Detector &d, const Detector &key, int64_t W)
{
    TuneShape s{};
    if (tuned_shape(kernel, key, W, &s)) {
        if (s.target == 0) s.target = default_tune_shape(kernel, d, W).target;
        return s;
    }
    return default_tune_shape(kernel, d, W);
}

CartPlan plan_direct_cartesian(const Detector &d, int64_t W, int channels, bool hermitian, size_t max_partial)
{
    Detector key = d;
    if (hermitian) key.n0 = (d.n0 + 1) / 2;
    TuneShape ts{};
    if (!tuned_shape(kTuneDirect, key, W, &ts)) return cart_default_plan(d, W, channels, max_partial);
    if (ts.target == 0) ts.target = default_tune_shape(kTuneDirect, d, W).target;
    return cheapest_plan(d, W, channels, max_partial, {ts.shape}, ts.target);
}

size_t cart_partial_bytes(const CartPlan &p)
{
    return p.nsplit > 1 ? cart_split_bytes(p.g, p.mt) * (size_t)p.nsplit : 0;
}

template <int CH, bool PARTIAL, class Loader>
static void launch_cart_tiles(const Loader &ld, int64_t W, const CartPlan &p, int add, double *out, hipStream_t s)
{
    // full column groups first
    const dim3 grid((unsigned)(p.nsplit * p.col_groups), p.g.nrb), block(cblk::kThreads);
#define NUMAG_LAUNCH_CART(MT)                                                                                       \
    hipLaunchKernelGGL((direct_cartesian_kernel<MT, CH, PARTIAL, Loader>), grid, block, 0, s, ld, W, p.per, p.nsplit, \
                       p.g, add, out)
    switch (p.mt) {
        case 1: NUMAG_LAUNCH_CART(1); break;
        case 2: NUMAG_LAUNCH_CART(2); break;
        case 3: NUMAG_LAUNCH_CART(3); break;
        case 4: NUMAG_LAUNCH_CART(4); break;
        case 5: NUMAG_LAUNCH_CART(5); break;
        case 6: NUMAG_LAUNCH_CART(6); break;
        case 7: NUMAG_LAUNCH_CART(7); break;
        default: NUMAG_LAUNCH_CART(8); break;
    }
#undef NUMAG_LAUNCH_CART
}

static int combine_cartesian(const CartPlan &p, const PointSource &src, int64_t W, const double *partial, double *amp,
                             int accumulate, hipStream_t s)
{
    NUMAG_HIP_CHECK(hipGetLastError());
    if (p.nsplit <= 1) return NUMAG_OK;
    const int64_t n = (int64_t)p.g.nrb * p.g.nzb * p.mt * 128;
    hipLaunchKernelGGL(cart_combine_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, partial, p.g, p.mt,
                       p.channels, p.nsplit, src, W, accumulate, amp);
    NUMAG_HIP_CHECK(hipGetLastError());
    return NUMAG_OK;
}

// The sum kernel, and the combine if the points are split.
template <int CH, class Loader>
static int sum_cartesian(const Loader &ld, int64_t W, const CartPlan &p, double *partial, double *amp, int accumulate,
                         hipStream_t s)
{
    {
        TimedLaunch timed(NUMAG_KERNEL_DIRECT, s);
        if (p.nsplit > 1)
            launch_cart_tiles<CH, true>(ld, W, p, 0, partial, s);
        else
            launch_cart_tiles<CH, false>(ld, W, p, accumulate, amp, s);
    }
    return combine_cartesian(p, ld.source(), W, partial, amp, accumulate, s);
}

int launch_direct_cartesian(const PointRec *pts, int64_t W, const CartPlan &p, double *partial, double *amp,
                            int accumulate, hipStream_t s)
{
    const int sw = p.g.swapped;
    switch (p.channels) {
        case 1: return sum_cartesian<1>(PrepLoader<1>{pts, sw}, W, p, partial, amp, accumulate, s);
        case 3: return sum_cartesian<3>(PrepLoader<3>{pts, sw}, W, p, partial, amp, accumulate, s);
        default: return sum_cartesian<4>(PrepLoader<4>{pts, sw}, W, p, partial, amp, accumulate, s);
    }
}

int launch_sample_cartesian(const double *pos, const double *nuc, const double *mag, const Rot &R, int64_t W,
                            const CartPlan &p, double *partial, double *amp, hipStream_t s)
{
    const int sw = p.g.swapped;
    switch (p.channels) {
        case 1: return sum_cartesian<1>(SampleLoader<1>{pos, nuc, mag, R, sw}, W, p, partial, amp, 0, s);
        case 3: return sum_cartesian<3>(SampleLoader<3>{pos, nuc, mag, R, sw}, W, p, partial, amp, 0, s);
        default: return sum_cartesian<4>(SampleLoader<4>{pos, nuc, mag, R, sw}, W, p, partial, amp, 0, s);
    }
}

__global__ void fill_kernel(double *__restrict__ out, int64_t n, double value)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = value;
}

int launch_fill(double *out, int64_t n, double value, hipStream_t s)
{
    if (n <= 0) return NUMAG_OK;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, n, value);
    NUMAG_HIP_CHECK(hipGetLastError());
    return NUMAG_OK;
}

}  // namespace numag
