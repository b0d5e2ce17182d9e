// Gradient of a loss on the unpolarized cross section (Sec. 2.4) with respect
// to every input weight: the adjoint (transposed) Fourier sum on gfx950.
//
//   I_p = (scale/V)(|S_N|^2 + bH^2 |Q|^2),  Q = -Pp S_M,  L = sum_p w_p (I_p - T_p)^2
//   dL/dn_j   = Re sum_p a_N(p) exp(-i q_p . X_j),   a_N = 4 w r (scale/V) conj(S_N)
//   dL/dm'_ja = Re sum_p a_a(p) exp(-i q_p . X_j),   a_a = 4 w r (scale/V) bH^2 conj((Pp S_M)_a)
// with r = I_p - T_p and m' = R m (so dL/dm = R^T dL/dm').
//
// The adjoint sum is the transposed contraction of the forward sums
// (cartesian_block.h, polar_block.h).  With the residual weights of the four pixels
// (+-q_M, +-q_N) of a cell folded into four real coefficients (Re[a(p') exp(+i q.X)] =
// Re[conj a(p') exp(-i q.X)] takes the pixels at -q onto those at q, for any target and
// loss weights),
//   G_c(j) = sum_a [ yr_a(j) T_{a,re,c}(j) + yi_a(j) T_{a,im,c}(j) ],
//   T_{a,re,c}(j) = sum_b RR_{abc} zr_b(j) + RI_{abc} zi_b(j),  T_{a,im,c} likewise with IR, II,
// so the work is real matrix products (coefficients) x (phasors of the points), one
// multiply-add per point, pixel and channel, on v_mfma_f64_16x16x4f64, against ten
// vector FP64 operations per point and pixel of a walk along the detector rows.
//
// The residual kernel writes the coefficients in the order the matrix instruction takes
// its first operand, so a wave's operand load is one 16-byte read per lane and tile.
//
// Measured, kernel time before (a lane walking the detector rows of four points with a
// two-term recurrence) and now: 262,144 points, 256 x 256: 6.14 -> 2.01 ms (68 of the
// card's 74.7 TFLOP/s; 2.37 with the coefficients staged through registers, which
// spilled); error of the gradient against 64 bits 8.2e-14 -> 6.6e-15, the walk of 256
// columns being gone.  20,000 points, 150 x 181 polar: 228 -> 222 us: every column of an
// odd detector is summed, so the multiply-adds fall only from 10 to 8 per term and the
// column tables (about 200 vector instructions per 32 points and column) take the rest;
// an even detector needs half of both.
#include <algorithm>
#include <cmath>

#include "cartesian_block.h"
#include "nonfinite.h"
#include "polar_block.h"

namespace numag {

constexpr int kResThreads = 256;

// Residual weights of one pixel (four complex numbers, a[8]) and its loss term.
__device__ __forceinline__ double residual_pixel(const Detector &d, const numag_consts &k, int64_t p,
                                                 const double *__restrict__ amp, const double *__restrict__ target,
                                                 const double *__restrict__ weight, double (&a)[8])
{
    double s, c;
    pixel_qhat(d, p, s, c);
    const double *A = amp + p * 8;
    // V = Pp S_M with Pp = I - qhat qhat^T, qhat = (0, s, c)
    const double dot_r = s * A[4] + c * A[6], dot_i = s * A[5] + c * A[7];
    const double Vr[3] = {A[2], A[4] - s * dot_r, A[6] - c * dot_r};
    const double Vi[3] = {A[3], A[5] - s * dot_i, A[7] - c * dot_i};
    const double cf = k.scale / k.V;
    const double b2 = k.bH * k.bH;
    const double absV2 =
        Vr[0] * Vr[0] + Vi[0] * Vi[0] + Vr[1] * Vr[1] + Vi[1] * Vi[1] + Vr[2] * Vr[2] + Vi[2] * Vi[2];
    const double I = cf * (A[0] * A[0] + A[1] * A[1] + b2 * absV2);
    // dL/dI_p: 2 w (I - T) for the built-in loss, or the caller's upstream
    // gradient (held in `weight`) when no target is given.
    double dLdI, lp = 0.0;
    if (target != nullptr) {
        const double r = I - target[p];
        const double w = weight[p];
        lp = w * r * r;
        dLdI = 2.0 * w * r;
    } else {
        dLdI = weight[p];
    }
    const double g = 2.0 * dLdI * cf;
    a[0] = g * A[0];
    a[1] = -g * A[1];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        a[2 + 2 * x] = g * b2 * Vr[x];
        a[3 + 2 * x] = -g * b2 * Vi[x];
    }
    return lp;
}

// Coefficients [row block or (column, row group)][column block][step][tile][lane] of
// (re, im) column parts: step s holds b = 16 v + 4 s + lane / 16, tile t and lane % 16 = 8 h
// + 4 part + c the row a = 2 t + h, part (re, im), channel c.
__device__ __forceinline__ int64_t coef_index(int64_t block, int MT, int e, int b16, int part, int c)
{
    return ((block * 4 + (b16 >> 2)) * MT + (e >> 1)) * 64 + 16 * (b16 & 3) + 8 * (e & 1) + 4 * part + c;
}

// One thread per cell of the padded grid: the residual weights of its pixels, folded,
// as coefficients (zeros outside the detector), and per-block loss partials.
// Cartesian cells (POLAR = 0): cell (a, b) of CartGeom; polar ones: offset b of row
// block a of column col, with column col + nh as the mirror.
template <int POLAR>
__global__ __launch_bounds__(kResThreads) void residual_kernel(Detector d, numag_consts k, CartGeom cg, PolGeom pg,
                                                               int MT, int64_t n_cells,
                                                               const double *__restrict__ amp,
                                                               const double *__restrict__ target,
                                                               const double *__restrict__ weight,
                                                               double2 *__restrict__ coef,
                                                               double *__restrict__ loss_part)
{
    const int64_t idx = (int64_t)blockIdx.x * kResThreads + threadIdx.x;
    double lp = 0.0;
    if (idx < n_cells) {
        // pixels (+,+), (+,-), (-,+), (-,-) of the cell; -1: none
        int64_t px[4] = {-1, -1, -1, -1};
        int64_t block;  // index of the 16-column coefficient block
        int e, b16;
        if (POLAR) {
            const int ne = 2 * MT;
            b16 = (int)(idx & 15);
            const int64_t r = idx >> 4;
            e = (int)(r % ne);
            block = r / ne;  // col * nrg + rg
            const int rg = (int)(block % pg.nrg), col = (int)(block / pg.nrg);
            const int a = rg * pg.na + e;
            if (e < pg.na && b16 < pg.mid) {
                const int rp = pblk::kRows * a + pg.mid + b16, rm = pblk::kRows * a + pg.mid - 1 - b16;
                if (rp < pg.n0) px[0] = (int64_t)rp * pg.n_out + col;
                if (rm < pg.n0) px[1] = (int64_t)rm * pg.n_out + col;
                if (pg.nh > 0) {
                    if (px[1] >= 0) px[2] = px[1] + pg.nh;
                    if (px[0] >= 0) px[3] = px[0] + pg.nh;
                }
            }
        } else {
            const int nb = 16 * cg.nzb, ne = 2 * MT;
            const int b = (int)(idx % nb);
            const int64_t r = idx / nb;
            e = (int)(r % ne);
            const int rb = (int)(r / ne);
            b16 = b & 15;
            block = (int64_t)rb * cg.nzb + (b >> 4);
            const cblk::CellPixels x = cblk::cell_pixels(cg, 4, rb, b >> 4, 4 * e, b16);
            if (x.ok) {
                px[0] = x.pp;
                if (x.twoN) px[1] = x.pm;
                if (x.twoM) {
                    px[3] = x.mm;
                    if (x.twoN) px[2] = x.mp;
                }
            }
        }
        double f[8] = {0.0}, g[8] = {0.0};  // folded weights of (+,+) and (+,-)
        for (int q = 0; q < 4; ++q) {
            if (px[q] < 0) continue;
            double a[8];
            lp += residual_pixel(d, k, px[q], amp, target, weight, a);
            double(&t)[8] = (q == 0 || q == 3) ? f : g;
#pragma unroll
            for (int v = 0; v < 8; ++v) t[v] += (q >= 2 && (v & 1)) ? -a[v] : a[v];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double fr = f[2 * c], fi = f[2 * c + 1], gr = g[2 * c], gi = g[2 * c + 1];
            coef[coef_index(block, MT, e, b16, 0, c)] = make_double2(fr + gr, gi - fi);     // RR, RI
            coef[coef_index(block, MT, e, b16, 1, c)] = make_double2(-fi - gi, gr - fr);    // IR, II
        }
    }
    if (loss_part == nullptr) return;
    __shared__ double s_l[kResThreads];
    s_l[threadIdx.x] = lp;
    __syncthreads();
    for (int w = kResThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s_l[threadIdx.x] += s_l[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss_part[blockIdx.x] = s_l[0];
}

__global__ void loss_sum_kernel(const double *__restrict__ part, int n, double *__restrict__ loss)
{
    __shared__ double s_l[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) acc += part[i];
    s_l[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s_l[threadIdx.x] += s_l[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = s_l[0];
}

// ---------------------------------------------------------------------------
// Cartesian adjoint.  A wave owns 32 points (two matrix column tiles); lane l holds
// point l % 16 of a tile and, of a step's four |q_N| values, number l / 16.  The 8 waves of
// a workgroup share the coefficients of one 16-column block at a time through LDS
// (double-buffered).  The column phasors live in registers: 16 offsets, four per lane,
// times the block's centre, which advances by a product per block; the row phasors are
// needed once per row block, when the tiles are folded into the point's four sums:
// accumulator register r of lane l is row 4 r + l / 16, so lane l sums channel l / 16.
// A split is a range of row blocks and one of column blocks.
// ---------------------------------------------------------------------------
constexpr int kAdjWaves = 8;
constexpr int kAdjThreads = 64 * kAdjWaves;
constexpr int kAdjNP = 2;
constexpr int kAdjPoints = 16 * kAdjNP * kAdjWaves;  // points per workgroup

struct AdjSplit {
    int nr, nv;        // ranges of row blocks and of column blocks
    int per_r, per_v;  // blocks per range
};

template <int MT>
__global__ __launch_bounds__(kAdjThreads, 2) void adjoint_cartesian_kernel(
    const PointRec *__restrict__ pts, int64_t W, CartGeom g, AdjSplit sp, const double2 *__restrict__ coef,
    double *__restrict__ gpart)
{
    constexpr int kStage = 4 * MT * 64;  // coefficients of a 16-column block
    __shared__ double2 s_c[2][kStage];
    const int lane = threadIdx.x & 63, wave = cblk::wave_id();
    const int pt = lane & 15, kq = lane >> 4;
    const int64_t j0 = (int64_t)blockIdx.x * kAdjPoints + wave * (16 * kAdjNP) + pt;
    const int rb0 = (int)(blockIdx.y / sp.nv) * sp.per_r, rb1 = min(g.nrb, rb0 + sp.per_r);
    const int v0 = (int)(blockIdx.y % sp.nv) * sp.per_v, v1 = min(g.nzb, v0 + sp.per_v);

    double m[kAdjNP], n[kAdjNP], G[kAdjNP];
    double2 off[kAdjNP][4], adv[kAdjNP];
    // centre of the first column block of the split
    const double qc = ((double)(16 * v0) + g.firstN + 7.5) * g.stepN;
#pragma unroll
    for (int u = 0; u < kAdjNP; ++u) {
        const int64_t j = j0 + 16 * u;
        const bool ok = j < W;
        const double y = ok ? pts[j].Y : 0.0, z = ok ? pts[j].Z : 0.0;
        m[u] = g.swapped ? z : y;
        n[u] = g.swapped ? y : z;
        G[u] = 0.0;
        adv[u] = twiddle(16.0 * g.stepN * n[u]);
#pragma unroll
        for (int s = 0; s < 4; ++s) off[u][s] = twiddle(((double)(4 * s + kq) - 7.5) * g.stepN * n[u]);
    }

    // block i of the walk over (row block, column block)
    const int nv = v1 - v0, total = max(0, rb1 - rb0) * max(0, nv);
    auto stage = [&](int i) {
        cblk::copy_to_lds(coef + ((int64_t)(rb0 + i / nv) * g.nzb + v0 + i % nv) * kStage, s_c[i & 1], kStage,
                          kAdjWaves);
    };
    cblk::v4d acc[MT][kAdjNP];
    if (total > 0) stage(0);
    cblk::wait_copies();
    __syncthreads();
    int i = 0;
#pragma unroll 1
    for (int rb = rb0; rb < rb1; ++rb) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int u = 0; u < kAdjNP; ++u) acc[t][u] = cblk::v4d{0.0, 0.0, 0.0, 0.0};
        double2 ctr[kAdjNP];
#pragma unroll
        for (int u = 0; u < kAdjNP; ++u)
            ctr[u] = phasor(half_turns(qc), n[u], fabs(n[u]) < phasor_range((g.B + 32.0) * g.stepN));
#pragma unroll 1
        for (int v = v0; v < v1; ++v, ++i) {
            if (i + 1 < total) stage(i + 1);  // arrives under the products
            const double2 *sc = &s_c[i & 1][lane];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                double2 z[kAdjNP];
#pragma unroll
                for (int u = 0; u < kAdjNP; ++u) z[u] = cmul(ctr[u], off[u][s]);
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    const double2 a = sc[(s * MT + t) * 64];
#pragma unroll
                    for (int u = 0; u < kAdjNP; ++u)
                        acc[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, z[u].x, acc[t][u], 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < kAdjNP; ++u)
                        acc[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, z[u].y, acc[t][u], 0, 0, 0);
                }
            }
#pragma unroll
            for (int u = 0; u < kAdjNP; ++u) ctr[u] = cmul(ctr[u], adv[u]);
            cblk::wait_copies();
            __syncthreads();
        }
        // fold the tiles of this row block: rows a = 2 t + h
        const double qm = ((double)(rb * g.na) + g.firstM) * g.stepM;
#pragma unroll
        for (int u = 0; u < kAdjNP; ++u) {
            double2 y, dm;
            phasor2(half_turns(qm), m[u], half_turns(g.stepM), m[u],
                    fabs(m[u]) < phasor_range((g.A + 32.0) * g.stepM), y, dm);
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    G[u] = fma(y.x, acc[t][u][2 * h], fma(y.y, acc[t][u][2 * h + 1], G[u]));
                    y = cmul(y, dm);
                }
        }
    }
#pragma unroll
    for (int u = 0; u < kAdjNP; ++u) {
        const int64_t j = j0 + 16 * u;
        if (j < W) gpart[((int64_t)blockIdx.y * W + j) * 4 + kq] = G[u];
    }
}

// ---------------------------------------------------------------------------
// Polar adjoint.  At one theta the q rows separate into block centres and offsets
// (polar_block.h), so a column's residual weights are a coefficient block per 8 row
// blocks: T = coefficients x offset phasors (16 columns deep), folded with the centres'.
// A wave owns 32 points (two matrix column tiles), generates its column tables into its
// own LDS with two lanes per point and loads a block's coefficients into registers before
// it does, so that waves run free of workgroup barriers and one generates while another
// of its SIMD multiplies.  A split is a range of theta columns.
// ---------------------------------------------------------------------------
constexpr int kPolWaves = 8;
constexpr int kPolThreads = 64 * kPolWaves;
constexpr int kPolNP = 2;
constexpr int kPolPoints = 16 * kPolNP * kPolWaves;  // points per workgroup
constexpr int kPolNA = 8;                            // row blocks per coefficient block

// v of lane k (wave-uniform) as a uniform value.
__device__ __forceinline__ double lane_value(double v, int k)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, k), hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// MT tiles of 16 coefficient rows, two row blocks each; MT = 0: one block of rows, whose eight
// coefficient rows are two tiles of 4 x 16, MT = -2 of up to 16 rows, with half the offsets (a third of the cycles of a tile of 16 that they
// would half fill, and registers and LDS for twice the waves).  20,000 points, adjoint sums with
// their residuals, tiles of 16 and now: 16 x 361 212 -> 92 us (134 by walking the rows; 133 with 16
// offsets), 32 x 181 113 -> 77 (121); 100,000 points 16 x 361 356 (344; 564 with 16 offsets).
template <int MT>
struct PolWaveTables {
    double2 off[32][pblk::Tiles<MT>::kOffsets + 1];
    double2 ctr[32][MT <= 0 ? 1 : 2 * MT + 1];
};

template <int MT>
__global__ __launch_bounds__(kPolThreads, MT <= 0 ? 4 : 2) void adjoint_polar_kernel(const PointRec *__restrict__ pts, int64_t W,
                                                                       PolGeom g, int cols_per_split,
                                                                       const double2 *__restrict__ coef,
                                                                       double *__restrict__ gpart)
{
    constexpr bool kOne = MT <= 0;
    constexpr int kOff = pblk::Tiles<MT>::kOffsets, kSteps = kOff / 4;
    constexpr int NT = kOne ? 2 : MT;
    constexpr int kStage = 4 * (kOne ? 1 : MT) * 64;
    __shared__ PolWaveTables<MT> s_t[kPolWaves];
    const int lane = threadIdx.x & 63, wave = cblk::wave_id();
    const int pt = lane & 15, kq = lane >> 4;
    const int half = lane >> 5, gp = lane & 31;
    const int64_t jw = (int64_t)blockIdx.x * kPolPoints + wave * 32;
    const int c0 = blockIdx.y * cols_per_split, c1 = min(g.cols, c0 + cols_per_split);
    PolWaveTables<MT> &tab = s_t[wave];
    const bool ok = jw + gp < W;
    const double Y = ok ? pts[jw + gp].Y : 0.0, Z = ok ? pts[jw + gp].Z : 0.0;
    double G[kPolNP];
#pragma unroll
    for (int u = 0; u < kPolNP; ++u) G[u] = 0.0;

    // (kOne: tile t holds part t of the four channels, coef_index)
    const int at = kOne ? 16 * kq + (pt & 3) : lane;
    const double2 *src = coef + (int64_t)c0 * g.nrg * kStage + at;
    const double2 *last = coef + ((int64_t)c1 * g.nrg - 1) * kStage + at;
    double2 co[kSteps][NT];  // coefficients of a block, loaded one block ahead of their use (kOne: with the
                             // tables, since they would spill)
    auto load = [&](const double2 *from) {
#pragma unroll
        for (int k = 0; k < kSteps * NT; ++k) co[k / NT][k % NT] = from[kOne ? 64 * (k / NT) + 4 * (k % NT) : 64 * k];
    };
    if (!kOne && c0 < c1) load(src);
    double2 dir = make_double2(0.0, 0.0);  // (sin, cos) of the angles of 64 columns, one per lane
#pragma unroll 1
    for (int col = c0; col < c1; ++col) {
        const int cl = (col - c0) & 63;
        if (cl == 0) sincos_cw((2.0 * 3.141592653589793 * (double)(col + lane)) / (double)g.n_out, &dir.x, &dir.y);
        const double sth = lane_value(dir.x, cl), cth = lane_value(dir.y, cl);
        const double u0 = Y * sth + Z * cth;
        __builtin_amdgcn_s_setprio(2);  // as in polar_block.h: tables before products
        double2 first, step;  // centre of the group's first block, centre step (second half)
        pblk::offsets<kOff>(tab.off, g.dq, u0, first, step);
        double2 adv = make_double2(1.0, 0.0);  // from one row group to the next
        if (g.nrg > 1) {
            const double q = (double)(pblk::kRows * g.na) * g.dq;
            adv = phasor(half_turns(q), u0, fabs(u0) < phasor_range(q));
        }
#pragma unroll 1
        for (int rg = 0; rg < g.nrg; ++rg) {
            if (half != 0) pblk::centres<kOne ? 1 : 2 * MT>(tab.ctr[gp], first, step);
            if (g.nrg > 1) first = cmul(first, adv);
            if (kOne) load(src);
            wave_fence();
            __builtin_amdgcn_s_setprio(0);
            typename pblk::Tiles<MT>::T acc[NT][kPolNP] = {};
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                double2 z[kPolNP];
#pragma unroll
                for (int u = 0; u < kPolNP; ++u) z[u] = tab.off[16 * u + pt][4 * s + kq];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const double2 a = co[s][t];
#pragma unroll
                    for (int u = 0; u < kPolNP; ++u) acc[t][u] = pblk::mfma(a.x, z[u].x, acc[t][u]);
#pragma unroll
                    for (int u = 0; u < kPolNP; ++u) acc[t][u] = pblk::mfma(a.y, z[u].y, acc[t][u]);
                }
            }
            src += kStage;
            if (!kOne) load(src < last ? src : last);  // (the last block again at the end, unused)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < kPolNP; ++u) {
                if constexpr (kOne) {
                    const double2 y = tab.ctr[16 * u + pt][0];
                    G[u] = fma(y.x, acc[0][u], fma(y.y, acc[1][u], G[u]));
                } else {
#pragma unroll
                    for (int t = 0; t < MT; ++t)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const double2 y = tab.ctr[16 * u + pt][2 * t + h];
                            G[u] = fma(y.x, acc[t][u][2 * h], fma(y.y, acc[t][u][2 * h + 1], G[u]));
                        }
                }
            }
            wave_fence();
        }
    }
#pragma unroll
    for (int u = 0; u < kPolNP; ++u) {
        const int64_t j = jw + 16 * u + pt;
        if (j < W) gpart[((int64_t)blockIdx.y * W + j) * 4 + kq] = G[u];
    }
}

// What the residual weights are formed from.
struct Residual {
    Detector d;
    numag_consts k;
    const double *amp, *target, *weight;
};

// A point's four sums, those that came out as NaN formed again from the pixels whose residual
// weights are not finite (nonfinite.h): a weight, target or amplitude of infinity makes
// inf - inf in a cell's coefficients where the pixel's own term is infinite.
__device__ __forceinline__ void repair_gradient(const Residual &r, double Y, double Z, double (&g)[4])
{
    const int64_t P = (int64_t)r.d.n0 * r.d.n1;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    bool any[4] = {false, false, false, false};
    const bool point = isfinite(Y) && isfinite(Z);
#pragma unroll 1
    for (int64_t p = 0; p < P; ++p) {
        bool finite = point && isfinite(r.weight[p]) && (r.target == nullptr || isfinite(r.target[p]));
        for (int v = 0; v < 8; ++v) finite = finite && isfinite(r.amp[8 * p + v]);
        if (finite) continue;
        double a[8], sn, cs;
        residual_pixel(r.d, r.k, p, r.amp, r.target, r.weight, a);
        const int row = (int)(p / r.d.n1), col = (int)(p % r.d.n1);
        double phi;
        if (r.d.kind == NUMAG_GRID_CARTESIAN) {
            phi = axis_value(r.d.origin0, row, r.d.step0) * Y + axis_value(r.d.origin1, col, r.d.step1) * Z;
        } else {
            pixel_qhat(r.d, p, sn, cs);
            phi = (double)row * r.d.step0 * (Y * sn + Z * cs);
        }
        const double2 e = phasor_signs(phi);
        bool all = true;
        for (int c = 0; c < 4; ++c) {
            if (!point || !isfinite(a[2 * c]) || !isfinite(a[2 * c + 1])) {
                s[c] = fma(-a[2 * c + 1], e.y, fma(a[2 * c], e.x, s[c]));
                any[c] = true;
            }
            all = all && any[c] && s[c] != s[c];
        }
        if (all) break;
    }
    for (int c = 0; c < 4; ++c)
        if (any[c] && g[c] != g[c]) g[c] = s[c];
}

__global__ __launch_bounds__(256, 8) void grad_finalize_kernel(const double *__restrict__ gpart, int nsplit, int64_t W, Rot R,
                                     const PointRec *__restrict__ pts, Residual res, double *__restrict__ dnuc,
                                     double *__restrict__ dmag)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= W) return;
    double g[4] = {0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < nsplit; ++s)
        for (int v = 0; v < 4; ++v) g[v] += gpart[((int64_t)s * W + j) * 4 + v];
    if (__builtin_expect(g[0] != g[0] || g[1] != g[1] || g[2] != g[2] || g[3] != g[3], 0))
        repair_gradient(res, pts[j].Y, pts[j].Z, g);
    if (dnuc != nullptr) dnuc[j] = g[0];
    if (dmag != nullptr) {
        for (int b = 0; b < 3; ++b)
            dmag[3 * j + b] = R.m[0 * 3 + b] * g[1] + R.m[1 * 3 + b] * g[2] + R.m[2 * 3 + b] * g[3];
    }
}

// ---------------------------------------------------------------------------
// Work split.
// ---------------------------------------------------------------------------
// Everything launch_grad derives from the detector and the point count.
struct GradPlan {
    CartGeom cg;
    PolGeom pg;
    int mt;
    int64_t n_cells;   // padded cells (residual threads)
    int64_t n_blocks;  // coefficient blocks of 4 mt 64 double2
    int64_t pblocks;   // point blocks
    AdjSplit sp;       // Cartesian ranges
    int cols_per, nsplit;
};

// Ranges the detector is split into, so that point blocks x ranges fill the chip (one
// workgroup per CU at a time; two on a polar detector of one row block): of the counts up to
// four rounds of these workgroups, the one
// with the fewest coefficient blocks on the busiest CU; a split costs the point's
// phasors and partial gradients, about one block's time.  A table entry's target sets
// the workgroups instead.
static GradPlan grad_plan(const Detector &d, int64_t W, bool hermitian, bool use_table = true)
{
    GradPlan p{};
    const bool cart = d.kind == NUMAG_GRID_CARTESIAN;
    int64_t units;
    if (cart) {
        cart_geometry(d, 4, p.cg, p.mt);
        p.cg.na = 2 * p.mt;
        p.cg.nrb = (p.cg.A + p.cg.na - 1) / p.cg.na;
        p.n_blocks = (int64_t)p.cg.nrb * p.cg.nzb;
        units = p.n_blocks;
    } else {
        p.pg.n0 = d.n0;
        p.pg.n_out = d.n_theta;
        p.pg.nh = d.n_theta % 2 == 0 ? d.n_theta / 2 : 0;
        p.pg.cols = p.pg.nh > 0 ? p.pg.nh : d.n_theta;
        p.pg.dq = d.step0;
        p.pg.mid = d.n0 <= 16 ? 8 : pblk::kRows / 2;
        const int blocks = (d.n0 + pblk::kRows - 1) / pblk::kRows;
        p.pg.nrg = (blocks + kPolNA - 1) / kPolNA;
        p.pg.na = (blocks + p.pg.nrg - 1) / p.pg.nrg;
        p.mt = (p.pg.na + 1) / 2;
        p.pg.na = std::min(2 * p.mt, blocks);
        p.pg.nrg = (blocks + p.pg.na - 1) / p.pg.na;
        p.n_blocks = (int64_t)p.pg.cols * p.pg.nrg;
        units = p.pg.cols;
    }
    p.n_cells = p.n_blocks * 2 * p.mt * 16;
    const int per_wg = cart ? kAdjPoints : kPolPoints;
    p.pblocks = std::max<int64_t>(1, (W + per_wg - 1) / per_wg);
    Detector key = d;
    if (hermitian) {
        if (cart) key.n0 = (d.n0 + 1) / 2;
        else key.n1 = d.n1 / 2;
    }
    auto set = [&](int64_t want) {
        want = std::max<int64_t>(1, std::min<int64_t>(want, std::min<int64_t>(units, 65535)));
        if (cart) {  // ranges of row blocks first: a range of column blocks folds every row block again
            int64_t nr = std::min<int64_t>(want, p.cg.nrb);
            p.sp.per_r = (int)((p.cg.nrb + nr - 1) / nr);
            p.sp.nr = (p.cg.nrb + p.sp.per_r - 1) / p.sp.per_r;
            const int64_t nv = std::max<int64_t>(1, std::min<int64_t>(want / p.sp.nr, p.cg.nzb));
            p.sp.per_v = (int)((p.cg.nzb + nv - 1) / nv);
            p.sp.nv = (p.cg.nzb + p.sp.per_v - 1) / p.sp.per_v;
            p.nsplit = p.sp.nr * p.sp.nv;
        } else {
            p.cols_per = (int)((p.pg.cols + want - 1) / want);
            p.nsplit = (p.pg.cols + p.cols_per - 1) / p.cols_per;
        }
    };
    TuneShape ts{};
    int64_t target = env_target() > 0 ? 2 * (int64_t)env_target() : 0;
    if (use_table && tuned_shape(kTuneAdjoint, key, W, &ts) && ts.target > 0)
        target = ts.target;
    if (target > 0) {
        set((target + p.pblocks - 1) / p.pblocks);
        return p;
    }
    int64_t best = 1;
    double best_cost = -1.0;
    const int64_t fit = !cart && p.pg.na == 1 ? 512 : 256;
    for (int r = 0; r <= 8; ++r) {  // half rounds
        const int64_t want = std::max<int64_t>(1, fit / 2 * r / p.pblocks);
        set(want);
        const double per = cart ? (double)p.sp.per_r * p.sp.per_v + 0.2 * p.sp.per_r : (double)p.cols_per * p.pg.nrg;
        const double rounds = std::ceil((double)(p.pblocks * p.nsplit) / (double)fit);
        const double cost = rounds * (per + 0.5) + 2e-6 * (double)p.nsplit * (double)W;
        if (best_cost < 0.0 || cost < 0.99 * best_cost) {
            best_cost = cost;
            best = want;
        }
    }
    set(best);
    return p;
}

int default_adjoint_target(const Detector &d, int64_t W)
{
    // (the key detector of a half path stands for itself here: only the count is reported)
    const GradPlan p = grad_plan(d, W, false, false);
    return (int)std::min<int64_t>(p.pblocks * p.nsplit, 1 << 20);
}

static size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

// Scratch of launch_grad: coefficients, loss partials, gradient partials of the splits.
size_t grad_workspace_bytes(const Detector &d, int64_t W, bool hermitian)
{
    const GradPlan p = grad_plan(d, W, hermitian);
    const int64_t nres = (p.n_cells + kResThreads - 1) / kResThreads;
    return al((size_t)p.n_blocks * 4 * p.mt * 64 * sizeof(double2)) + al((size_t)nres * sizeof(double)) +
           al((size_t)p.nsplit * (size_t)std::max<int64_t>(W, 1) * 4 * sizeof(double));
}

int launch_grad(const PointRec *pts, int64_t W, const Detector &d, const numag_consts &c, const double *amp,
                const double *target, const double *weight, double *loss, double *dnuc, double *dmag, const Rot &R,
                void *ws, size_t ws_bytes, hipStream_t s, bool hermitian)
{
    const GradPlan p = grad_plan(d, W, hermitian);
    const bool cart = d.kind == NUMAG_GRID_CARTESIAN;
    const int64_t nres = (p.n_cells + kResThreads - 1) / kResThreads;
    char *base = (char *)ws;
    auto take = [&](size_t bytes) {
        char *r = base;
        base += al(bytes);
        return r;
    };
    double2 *coef = (double2 *)take((size_t)p.n_blocks * 4 * p.mt * 64 * sizeof(double2));
    double *lpart = (double *)take((size_t)nres * sizeof(double));
    double *gpart = (double *)take((size_t)p.nsplit * (size_t)std::max<int64_t>(W, 1) * 4 * sizeof(double));
    if ((size_t)(base - (char *)ws) > ws_bytes) {
        set_error("numag_grad: workspace too small");
        return NUMAG_E_WORKSPACE;
    }
    if (cart)
        hipLaunchKernelGGL((residual_kernel<0>), dim3((unsigned)nres), dim3(kResThreads), 0, s, d, c, p.cg, p.pg, p.mt,
                           p.n_cells, amp, target, weight, coef, loss != nullptr ? lpart : nullptr);
    else
        hipLaunchKernelGGL((residual_kernel<1>), dim3((unsigned)nres), dim3(kResThreads), 0, s, d, c, p.cg, p.pg, p.mt,
                           p.n_cells, amp, target, weight, coef, loss != nullptr ? lpart : nullptr);
    NUMAG_HIP_CHECK(hipGetLastError());
    if (loss != nullptr) {
        hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(256), 0, s, lpart, (int)nres, loss);
        NUMAG_HIP_CHECK(hipGetLastError());
    }
    if (W <= 0) return NUMAG_OK;
    const dim3 grid((unsigned)p.pblocks, p.nsplit);
    {
        TimedLaunch timed(NUMAG_KERNEL_ADJOINT, s);
#define NUMAG_LAUNCH_ADJ_C(MT)                                                                                     \
    case MT:                                                                                                       \
        hipLaunchKernelGGL((adjoint_cartesian_kernel<MT>), grid, dim3(kAdjThreads), 0, s, pts, W, p.cg, p.sp, coef, \
                           gpart);                                                                                 \
        break
#define NUMAG_LAUNCH_ADJ_P(MT)                                                                                     \
    case MT:                                                                                                       \
        hipLaunchKernelGGL((adjoint_polar_kernel<MT>), grid, dim3(kPolThreads), 0, s, pts, W, p.pg, p.cols_per, coef, \
                           gpart);                                                                                 \
        break
        if (cart) {
            switch (p.mt) {
                NUMAG_LAUNCH_ADJ_C(1);
                NUMAG_LAUNCH_ADJ_C(2);
                NUMAG_LAUNCH_ADJ_C(3);
                NUMAG_LAUNCH_ADJ_C(4);
                NUMAG_LAUNCH_ADJ_C(5);
                NUMAG_LAUNCH_ADJ_C(6);
                NUMAG_LAUNCH_ADJ_C(7);
                NUMAG_LAUNCH_ADJ_C(8);
            }
        } else {
            switch (p.pg.mid == 8 ? -2 : p.pg.na == 1 ? 0 : p.mt) {
                NUMAG_LAUNCH_ADJ_P(-2);
                NUMAG_LAUNCH_ADJ_P(0);
                NUMAG_LAUNCH_ADJ_P(1);
                NUMAG_LAUNCH_ADJ_P(2);
                NUMAG_LAUNCH_ADJ_P(3);
                NUMAG_LAUNCH_ADJ_P(4);
            }
        }
#undef NUMAG_LAUNCH_ADJ_C
#undef NUMAG_LAUNCH_ADJ_P
    }
    NUMAG_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(grad_finalize_kernel, dim3((unsigned)((W + 255) / 256)), dim3(256), 0, s, gpart, p.nsplit, W, R,
                       pts, Residual{d, c, amp, target, weight}, dnuc, dmag);
    NUMAG_HIP_CHECK(hipGetLastError());
    return NUMAG_OK;
}

}  // namespace numag
