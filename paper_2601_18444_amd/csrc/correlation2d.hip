// Two-dimensional correlation function (Sec. 2.6 eq. crav2d) and the angular
// spectrum (Sec. 2.5 eqs. CosineSinceIntensities, ModalAmplitudes) on gfx950.
//
// C(r) = int int f(q, theta) exp(i q rho cos(theta - alpha)) q dq dtheta is, with
// q = q (sin theta, cos theta) and r = rho (sin alpha, cos alpha) in the detector
// plane, the quadrature sum over detector pixels p
//     C(r) = sum_p wq_p f_p exp(i q_p . r),
// wq the trapezoidal weights (h_i q_i dtheta on the polar detector, dq_y dq_z
// with halved edges on a Cartesian one).  That is a direct Fourier sum whose
// "points" are the pixels, placed at -q_p so that the sums' exp(-i ...) becomes
// exp(+i q.r), with real weights wq_p f_p; the real-space grid plays the role of
// the detector.
//  - Cartesian detector and Cartesian real-space grid: the pixels are a regular grid, and
//    the sum factors (separable.hip), four data sets a pass, but for thin and very large
//    grids (factored()).  220 x 190 pixels to 180 x 170 points, 4 sets: 36 us, against 306
//    as a direct sum.
//  - Polar real-space grid, and a detector that has the pixel at -q for every one at q (a
//    Cartesian one, a polar one with an even number of columns): the polar sums with the
//    two pixels as one point of two weights (polar_block.h), half the points, four data
//    sets a pass.  200 x 360 pixels to 150 x 240 points, 2 sets: 226 us, against 450 over
//    all pixels in three channels.
//  - else: the direct sums over all pixels, their weight channels carrying up to four data
//    sets at once: one set alone in channel 0 (the kernels' one-channel form), two or three
//    in channels 1-3, four in all four.
#include <algorithm>

#include "nonfinite.h"
#include "numag_internal.h"
#include "phasor.h"

namespace numag {

// Position and quadrature weight of pixel (row, col).
__device__ __forceinline__ void quadrature_pixel(const Detector &d, int row, int col, double &qy, double &qz, double &wq)
{
    if (d.kind == NUMAG_GRID_CARTESIAN) {
        qy = axis_value(d.origin0, row, d.step0);
        qz = axis_value(d.origin1, col, d.step1);
        const double cy = (row == 0 || row == d.n0 - 1) ? 0.5 : 1.0;
        const double cz = (col == 0 || col == d.n1 - 1) ? 0.5 : 1.0;
        const double dy = d.n0 > 1 ? d.step0 : 1.0, dz = d.n1 > 1 ? d.step1 : 1.0;
        wq = cy * cz * dy * dz;
    } else {
        const double q = axis_value(0.0, row, d.step0);
        const double th = (2.0 * 3.141592653589793 * (double)col) / (double)d.n1;
        double s, c;
        sincos(th, &s, &c);
        qy = q * s;
        qz = q * c;
        const double h = (row == 0 || row == d.n0 - 1) ? 0.5 * d.step0 : d.step0;
        wq = h * q * (2.0 * 3.141592653589793 / (double)d.n1);
    }
}

// Pixels of detector d as points: Y = -q_y, Z = -q_z, weight channel c0 + c =
// wq * f_(set0 + c), the other channels zero.
__global__ void corr2d_points_kernel(Detector d, const double *__restrict__ f, int n_f, int set0, int c0,
                                     PointRec *__restrict__ out)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    double qy, qz, wq;
    quadrature_pixel(d, (int)(p / d.n1), (int)(p % d.n1), qy, qz, wq);
    PointRec r;
    r.Y = -qy;
    r.Z = -qz;
    for (int c = 0; c < 4; ++c) {
        const int set = set0 + c - c0;
        r.w[c] = (c >= c0 && set < n_f) ? wq * f[(int64_t)set * P + p] : 0.0;
    }
    r.pad[0] = r.pad[1] = 0.0;
    out[p] = r;
}

// Pairs of pixels at q and -q.
__host__ __device__ static inline bool has_pairs(const Detector &d)
{
    return d.kind == NUMAG_GRID_CARTESIAN || d.n1 % 2 == 0;
}
static inline int64_t n_pairs(const Detector &d) { return ((int64_t)d.n0 * d.n1 + 1) / 2; }

// Pair j: pixel p and its partner o (the middle of an odd Cartesian detector is its own),
// at -q_p, with the sums and the differences of wq f of data sets set0 .. set0 + 3.
__global__ void corr2d_pairs_kernel(Detector d, const double *__restrict__ f, int n_f, int set0, int64_t n,
                                    PairRec *__restrict__ out)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    int64_t p = j, o = P - 1 - j;
    if (d.kind != NUMAG_GRID_CARTESIAN) {
        const int nh = d.n1 / 2;
        p = j / nh * d.n1 + j % nh;
        o = p + nh;
    }
    double qy, qz, wq;
    quadrature_pixel(d, (int)(p / d.n1), (int)(p % d.n1), qy, qz, wq);
    PairRec r;
    r.Y = -qy;
    r.Z = -qz;
    for (int c = 0; c < 4; ++c) {
        const double *fs = f + (int64_t)(set0 + c) * P;
        const double fp = set0 + c < n_f ? fs[p] : 0.0, fo = set0 + c < n_f && o != p ? fs[o] : 0.0;
        r.w[2 * c] = wq * (fp + fo);
        r.w[2 * c + 1] = wq * (fp - fo);
    }
    out[j] = r;
}

// Weights of a regular grid of pixels: wq f of data set set0 as `nuc`, of the next three as
// `mag`.
__global__ void corr2d_weights_kernel(Detector d, const double *__restrict__ f, int n_f, int set0,
                                      double *__restrict__ nuc, double *__restrict__ mag)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    double qy, qz, wq;
    quadrature_pixel(d, (int)(p / d.n1), (int)(p % d.n1), qy, qz, wq);
    for (int c = 0; c < 4; ++c) {
        const double v = set0 + c < n_f ? wq * f[(int64_t)(set0 + c) * P + p] : 0.0;
        if (c == 0)
            nuc[p] = v;
        else
            mag[3 * p + c - 1] = v;
    }
}

// C_out[set0 + c][t] = channel c0 + c of amp[t], c < m.  A value that came out as NaN is
// formed again from the terms of the pixels whose data are not finite (nonfinite.h; whichever
// way the sums were taken).
__global__ void corr2d_scatter_kernel(const double *__restrict__ amp, int64_t R, int m, int set0, int c0, Detector d,
                                      Detector rd, const double *__restrict__ f, double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= R * 4) return;
    const int64_t t = i / 4;
    const int c = (int)(i % 4);
    if (c >= m) return;
    double2 v = make_double2(amp[t * 8 + 2 * (c0 + c)], amp[t * 8 + 2 * (c0 + c) + 1]);
    if (__builtin_expect(is_nan(v), 0)) {
        const int64_t P = (int64_t)d.n0 * d.n1;
        const double *fs = f + (int64_t)(set0 + c) * P;
        double ry, rz, unused;
        quadrature_pixel(rd, (int)(t / rd.n1), (int)(t % rd.n1), ry, rz, unused);
        v = nonfinite_terms(
            [&](int64_t p, double &Y, double &Z, double &w) {
                w = fs[p];
                Y = Z = 0.0;
                if (isfinite(w)) return;
                double wq;
                quadrature_pixel(d, (int)(p / d.n1), (int)(p % d.n1), Y, Z, wq);
                w *= wq;
                Y = -Y;
                Z = -Z;
            },
            0, P, ry, rz, v);
    }
    double *o = out + ((int64_t)(set0 + c) * R + t) * 2;
    o[0] = v.x;
    o[1] = v.y;
}

static size_t al2(size_t b) { return (b + 255) & ~(size_t)255; }

enum Route { kSeparable, kPairs, kDirect };

// The pixels of a Cartesian detector at -q, as a regular grid of one layer.
static numag_regular pixel_grid(const Detector &d)
{
    numag_regular g{};
    g.n[0] = 1;
    g.n[1] = d.n0;
    g.n[2] = d.n1;
    g.origin[1] = -d.origin0;
    g.origin[2] = -d.origin1;
    g.step[0] = 1.0;
    g.step[1] = -d.step0;
    g.step[2] = -d.step1;
    return g;
}

// Whether the sum over a Cartesian detector's pixels is factored (a Cartesian real-space
// grid).  The factored sum takes a step per four detector rows and one per four columns, one
// after the other where the detector is long and few waves share its steps, and holds the
// first contraction for every row; the direct sums take pixels x points.  In cycles, the
// factored sums from 1000 x 2, 2 x 1000 and 2000 x 3 pixels to as many points (61, 48 and
// 125 us; the direct sums 18, 18 and 27 to 30); 2000 x 20 to 20 x 2000 is 137 and 125 to 236,
// 32 x 32 18 and 22, 100 x 100 to 30 x 30 22 and 45 to 53.  A thin pair of grids (10^5 x 10 to
// 10 x 10^5) would need 320 GB where the direct sums' records take 128 MB, which bounds it,
// and a launch takes 2^31 threads.
static bool factored_is_cheaper(const Detector &d, const Detector &rd)
{
    const int64_t P = (int64_t)d.n0 * d.n1, R = (int64_t)rd.n0 * rd.n1;
    const double na = (rd.n0 + 1) / 2, nb = (rd.n1 + 1) / 2, ny = d.n0, nz = d.n1;
    if (16 * P + 16 * (na * ny + nb * nz) > (double)((int64_t)1 << 31)) return false;
    const size_t ws = separable_workspace_bytes(pixel_grid(d), rd, NUMAG_PATH_SEPARABLE_F64, 1);
    if (ws > (size_t)(P + R) * 64 + ((size_t)256 << 20)) return false;
    const double flops = 16.0 * ny * nb * nz + 32.0 * na * nb * ny;
    const double f = 46000.0 + 113.0 * ny + 72.0 * nz + flops / 15000.0;
    return f <= 38000.0 + 0.1 * (double)P + cart_default_cost(rd, P, 4);
}

// The same for the thread's last sizes: a call asks several times (its workspace's size, its
// layout, its launch), and the estimate of the direct sums compares 32 plans, 0.4 us (calls of 40
// us are bound by the host).
static bool factored(const Detector &d, const Detector &rd)
{
    struct Last {
        int n[4];
        bool factored;
    };
    static thread_local Last last{{-1, -1, -1, -1}, false};
    const int n[4] = {d.n0, d.n1, rd.n0, rd.n1};
    if (!std::equal(n, n + 4, last.n)) {
        last.factored = factored_is_cheaper(d, rd);
        std::copy(n, n + 4, last.n);
    }
    return last.factored;
}

static Route corr2d_route(const Detector &d, const Detector &rd)
{
    if (rd.kind == NUMAG_GRID_CARTESIAN)
        return d.kind == NUMAG_GRID_CARTESIAN && factored(d, rd) ? kSeparable : kDirect;
    return has_pairs(d) ? kPairs : kDirect;
}

// Bytes of split partial sums, whatever the channel set.
static size_t corr2d_partial_bytes(const Detector &d, const Detector &rd)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    size_t b = 0;
    if (corr2d_route(d, rd) == kPairs) {
        for (int ch : {4, 3, 2, 1}) b = std::max(b, polar_partial_bytes(plan_direct_polar(rd, n_pairs(d), ch, true)));
        return b;
    }
    for (int ch : {4, 3, 1})
        b = std::max(b, rd.kind == NUMAG_GRID_CARTESIAN ? cart_partial_bytes(plan_direct_cartesian(rd, P, ch, true))
                                                        : polar_partial_bytes(plan_direct_polar(rd, P, ch, true)));
    return b;
}

struct Corr2dLayout {
    size_t in, part, amp, total;  // points or weights, partial sums or the separable path's, one pass's sums
};

static Corr2dLayout corr2d_layout(const Detector &d, const Detector &rd)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    Corr2dLayout L{};
    switch (corr2d_route(d, rd)) {
        case kSeparable:
            L.in = al2((size_t)P * 4 * sizeof(double));
            L.part = al2(separable_workspace_bytes(pixel_grid(d), rd, NUMAG_PATH_SEPARABLE_F64, 1));
            break;
        case kPairs:
            L.in = al2((size_t)n_pairs(d) * sizeof(PairRec));
            L.part = al2(corr2d_partial_bytes(d, rd));
            break;
        default:
            L.in = al2((size_t)P * sizeof(PointRec));
            L.part = al2(corr2d_partial_bytes(d, rd));
    }
    L.amp = al2((size_t)rd.n0 * rd.n1 * 8 * sizeof(double));
    L.total = L.in + L.part + L.amp;
    return L;
}

size_t correlation_2d_workspace_bytes(const Detector &d, const Detector &rd) { return corr2d_layout(d, rd).total; }

int launch_correlation_2d(const Detector &d, const double *f, int n_f, const Detector &rd, double *C, void *ws,
                          size_t ws_bytes, hipStream_t s)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    const int64_t R = (int64_t)rd.n0 * rd.n1;
    const Corr2dLayout L = corr2d_layout(d, rd);
    if (ws_bytes < L.total) {
        set_error("numag_correlation_2d: workspace too small");
        return NUMAG_E_WORKSPACE;
    }
    char *base = (char *)ws;
    PointRec *pts = (PointRec *)base;
    double *part = (double *)(base + L.in);
    double *amp = (double *)(base + L.in + L.part);
    const Route route = corr2d_route(d, rd);
    for (int set0 = 0; set0 < n_f; set0 += 4) {
        const int m = std::min(4, n_f - set0);
        int c0 = 0, rc;
        if (route == kSeparable) {
            double *nuc = (double *)base, *mag = nuc + P;
            hipLaunchKernelGGL(corr2d_weights_kernel, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, d, f, n_f,
                               set0, nuc, mag);
            NUMAG_HIP_CHECK(hipGetLastError());
            rc = launch_separable(nuc, mag, pixel_grid(d), rd, NUMAG_PATH_SEPARABLE_F64, 1, amp, part, L.part, s,
                                  true);
        } else if (route == kPairs) {
            const int64_t n = n_pairs(d);
            hipLaunchKernelGGL(corr2d_pairs_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, d, f, n_f,
                               set0, n, (PairRec *)base);
            NUMAG_HIP_CHECK(hipGetLastError());
            // a triple takes channels 1-3 of the result, as in the direct sums
            c0 = m == 3 ? 1 : 0;
            rc = launch_polar_pairs((PairRec *)base, n, plan_direct_polar(rd, n, m, true), part, amp, s);
        } else {
            // the sum kernels' channel set for this pass: 1 (channel 0), 3 (channels 1-3) or 4
            const int channels = m == 1 ? 1 : (m == 4 ? 4 : 3);
            c0 = channels == 3 ? 1 : 0;
            hipLaunchKernelGGL(corr2d_points_kernel, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, d, f, n_f,
                               set0, c0, pts);
            NUMAG_HIP_CHECK(hipGetLastError());
            rc = rd.kind == NUMAG_GRID_CARTESIAN
                     ? launch_direct_cartesian(pts, P, plan_direct_cartesian(rd, P, channels, true), part, amp, 0, s)
                     : launch_direct_polar(pts, P, plan_direct_polar(rd, P, channels, true), part, amp, 0, s);
        }
        if (rc != NUMAG_OK) return rc;
        hipLaunchKernelGGL(corr2d_scatter_kernel, dim3((unsigned)((R * 4 + 255) / 256)), dim3(256), 0, s, amp, R, m,
                           set0, c0, d, rd, f, C);
        NUMAG_HIP_CHECK(hipGetLastError());
    }
    return NUMAG_OK;
}

// ---------------------------------------------------------------------------
// Angular spectrum on the polar detector: periodic trapezoid over theta of
// f sin(k theta), f cos(k theta) with prefactor (2 - delta_k0) / (2 pi).
// One workgroup per (data set, q row); a group of G lanes takes an order, its lanes the
// columns, so that few columns leave no more lanes idle than they must.  (The periodic
// trapezoid weights every column with h.)  One thread per order walked all columns with two
// sincos each: 2 data sets, 200 x 360 pixels, orders to 8 248 -> 9.3 us; 20,000 sets of
// 10 x 12 pixels, orders to 63 1037 us, 3387 with 64 lanes an order, 992 with 16.
// ---------------------------------------------------------------------------
template <int G>
__global__ __launch_bounds__(256) void angular_spectrum_kernel(Detector d, const double *__restrict__ f, int k_max,
                                                               double *__restrict__ Is, double *__restrict__ Ic)
{
    const int set = blockIdx.y;
    const int lane = threadIdx.x & (G - 1), groups = (int)blockDim.x / G;
    const int64_t P = (int64_t)d.n0 * d.n1;
    const double h = 2.0 * 3.141592653589793 / (double)d.n1;
    for (int row = blockIdx.x; row < d.n0; row += gridDim.x) {
        const double *fr = f + (int64_t)set * P + (int64_t)row * d.n1;
        for (int64_t k0 = 0; k0 <= k_max; k0 += groups) {  // (the shuffles need whole waves)
            const int64_t k = k0 + threadIdx.x / G;
            double ss = 0.0, cc = 0.0;
            if (k <= k_max)
                for (int m = lane; m < d.n1; m += G) {
                    double s0, c0;
                    sincos_cw((double)k * (h * (double)m), &s0, &c0);
                    ss += fr[m] * s0;
                    cc += fr[m] * c0;
                }
#pragma unroll
            for (int o = G / 2; o > 0; o >>= 1) {
                ss += __shfl_xor(ss, o);
                cc += __shfl_xor(cc, o);
            }
            if (lane == 0 && k <= k_max) {
                const double pref = h * ((k == 0 ? 1.0 : 2.0) / (2.0 * 3.141592653589793));
                const int64_t o = ((int64_t)set * d.n0 + row) * ((int64_t)k_max + 1) + k;
                Is[o] = pref * ss;
                Ic[o] = pref * cc;
            }
        }
    }
}

// a_k = sum_i I_k(q_i);  A_k = a_k / sum_j sqrt(a_s_j^2 + a_c_j^2).  One workgroup per data
// set; a wave takes every fourth order, its lanes the rows (248 -> 5.3 us for 2 data sets,
// 200 rows, orders to 8, against one thread per data set).
__global__ __launch_bounds__(256) void modal_amplitude_kernel(const double *__restrict__ Is,
                                                              const double *__restrict__ Ic, int n_q, int k_max,
                                                              double *__restrict__ As, double *__restrict__ Ac)
{
    const int64_t set = blockIdx.x, n_k = k_max + 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __shared__ double part[4];
    double norm = 0.0;
    for (int k = wave; k <= k_max; k += 4) {
        double as = 0.0, ac = 0.0;
        for (int i = lane; i < n_q; i += 64) {
            as += Is[(set * n_q + i) * n_k + k];
            ac += Ic[(set * n_q + i) * n_k + k];
        }
        as = wave_sum(as);
        ac = wave_sum(ac);
        if (lane == 0) {
            As[set * n_k + k] = as;
            Ac[set * n_k + k] = ac;
        }
        norm += sqrt(as * as + ac * ac);
    }
    if (lane == 0) part[wave] = norm;
    __syncthreads();
    norm = (part[0] + part[1]) + (part[2] + part[3]);
    for (int64_t k = threadIdx.x; k < n_k; k += 256) {
        As[set * n_k + k] /= norm;
        Ac[set * n_k + k] /= norm;
    }
}

int launch_angular_spectrum(const Detector &d, const double *f, int n_f, int k_max, double *Is, double *Ic,
                            double *As, double *Ac, hipStream_t s)
{
    if (n_f <= 0) return NUMAG_OK;
    int G = 4;
    while (G < 64 && G < d.n1) G *= 2;
    const int threads = ((int64_t)k_max + 1) * G <= 64 ? 64 : 256;
    const dim3 grid((unsigned)std::min<int64_t>(d.n0, max_workgroups(threads)), n_f);
#define NUMAG_LAUNCH_ANG(G_)                                                                                      \
    case G_:                                                                                                      \
        hipLaunchKernelGGL((angular_spectrum_kernel<G_>), grid, dim3(threads), 0, s, d, f, k_max, Is, Ic);        \
        break
    switch (G) {
        NUMAG_LAUNCH_ANG(4);
        NUMAG_LAUNCH_ANG(8);
        NUMAG_LAUNCH_ANG(16);
        NUMAG_LAUNCH_ANG(32);
        NUMAG_LAUNCH_ANG(64);
    }
#undef NUMAG_LAUNCH_ANG
    NUMAG_HIP_CHECK(hipGetLastError());
    if (As != nullptr && Ac != nullptr) {
        hipLaunchKernelGGL(modal_amplitude_kernel, dim3(n_f), dim3(256), 0, s, Is, Ic, d.n0, k_max, As, Ac);
        NUMAG_HIP_CHECK(hipGetLastError());
    }
    return NUMAG_OK;
}

}  // namespace numag
