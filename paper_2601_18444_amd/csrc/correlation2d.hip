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
// the detector.  It therefore runs on the same Cartesian / polar direct-sum
// kernels, and their weight channels carry up to four data sets at once: one set
// runs alone in channel 0 (the kernels' one-channel form, 4.5 instead of 10.5
// instructions per term), two or three in channels 1-3, four in all four.
#include <algorithm>

#include "numag_internal.h"
#include "phasor.h"

namespace numag {


// Pixels of detector d as points: Y = -q_y, Z = -q_z, weight channel c0 + c =
// wq * f_(set0 + c), the other channels zero.
__global__ void corr2d_points_kernel(Detector d, const double *__restrict__ f, int n_f, int set0, int c0,
                                     PointRec *__restrict__ out)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    const int row = (int)(p / d.n1), col = (int)(p % d.n1);
    double qy, qz, wq;
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

// C_out[set0 + c][t] = channel c0 + c of amp[t]
__global__ void corr2d_scatter_kernel(const double *__restrict__ amp, int64_t R, int n_f, int set0, int c0,
                                      double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= R * 4) return;
    const int64_t t = i / 4;
    const int c = (int)(i % 4);
    if (set0 + c >= n_f || c0 + c >= 4) return;
    double *o = out + ((int64_t)(set0 + c) * R + t) * 2;
    o[0] = amp[t * 8 + 2 * (c0 + c)];
    o[1] = amp[t * 8 + 2 * (c0 + c) + 1];
}

static size_t al2(size_t b) { return (b + 255) & ~(size_t)255; }

// Bytes of split partial sums, whatever the channel set.
static size_t corr2d_partial_bytes(const Detector &rd, int64_t P)
{
    size_t b = 0;
    for (int ch : {4, 3, 1})
        b = std::max(b, rd.kind == NUMAG_GRID_CARTESIAN ? cart_partial_bytes(plan_direct_cartesian(rd, P, ch, true))
                                                        : polar_partial_bytes(plan_direct_polar(rd, P, ch, true)));
    return b;
}

size_t correlation_2d_workspace_bytes(const Detector &d, const Detector &rd)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    const int64_t R = (int64_t)rd.n0 * rd.n1;
    return al2((size_t)P * sizeof(PointRec)) + al2(corr2d_partial_bytes(rd, P)) + al2((size_t)R * 8 * sizeof(double));
}
int launch_correlation_2d(const Detector &d, const double *f, int n_f, const Detector &rd, double *C, void *ws,
                          size_t ws_bytes, hipStream_t s)
{
    const int64_t P = (int64_t)d.n0 * d.n1;
    const int64_t R = (int64_t)rd.n0 * rd.n1;
    if (ws_bytes < correlation_2d_workspace_bytes(d, rd)) {
        set_error("numag_correlation_2d: workspace too small");
        return NUMAG_E_WORKSPACE;
    }
    char *base = (char *)ws;
    PointRec *pts = (PointRec *)base;
    double *part = (double *)(base + al2((size_t)P * sizeof(PointRec)));
    double *amp = (double *)(base + al2((size_t)P * sizeof(PointRec)) + al2(corr2d_partial_bytes(rd, P)));
    for (int set0 = 0; set0 < n_f; set0 += 4) {
        // the sum kernels' channel set for this group: 1 (channel 0), 3 (channels 1-3) or 4
        const int m = std::min(4, n_f - set0);
        const int channels = m == 1 ? 1 : (m == 4 ? 4 : 3);
        const int c0 = channels == 3 ? 1 : 0;
        hipLaunchKernelGGL(corr2d_points_kernel, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, d, f, n_f, set0,
                           c0, pts);
        NUMAG_HIP_CHECK(hipGetLastError());
        const int rc =
            rd.kind == NUMAG_GRID_CARTESIAN
                ? launch_direct_cartesian(pts, P, plan_direct_cartesian(rd, P, channels, true), part, amp, 0, s)
                : launch_direct_polar(pts, P, plan_direct_polar(rd, P, channels, true), part, amp, 0, s);
        if (rc != NUMAG_OK) return rc;
        hipLaunchKernelGGL(corr2d_scatter_kernel, dim3((unsigned)((R * 4 + 255) / 256)), dim3(256), 0, s, amp, R, n_f,
                           set0, c0, C);
        NUMAG_HIP_CHECK(hipGetLastError());
    }
    return NUMAG_OK;
}

// ---------------------------------------------------------------------------
// Angular spectrum on the polar detector: periodic trapezoid over theta of
// f sin(k theta), f cos(k theta) with prefactor (2 - delta_k0) / (2 pi).
// One workgroup per (data set, q row); a wave takes every fourth order, its lanes the
// columns.  (The periodic trapezoid weights every column with h.)  One thread per order
// walked all columns with two sincos each: 2 data sets, 200 x 360 pixels, orders to 8
// 248 -> 9.3 us.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void angular_spectrum_kernel(Detector d, const double *__restrict__ f, int k_max,
                                                               double *__restrict__ Is, double *__restrict__ Ic)
{
    const int row = blockIdx.x, set = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t P = (int64_t)d.n0 * d.n1;
    const double *fr = f + (int64_t)set * P + (int64_t)row * d.n1;
    const double h = 2.0 * 3.141592653589793 / (double)d.n1;
    for (int k = wave; k <= k_max; k += 4) {
        double ss = 0.0, cc = 0.0;
        for (int m = lane; m < d.n1; m += 64) {
            double s0, c0;
            sincos_cw((double)k * (h * (double)m), &s0, &c0);
            ss += fr[m] * s0;
            cc += fr[m] * c0;
        }
        ss = wave_sum(ss);
        cc = wave_sum(cc);
        if (lane == 0) {
            const double pref = h * ((k == 0 ? 1.0 : 2.0) / (2.0 * 3.141592653589793));
            const int64_t o = ((int64_t)set * d.n0 + row) * (k_max + 1) + k;
            Is[o] = pref * ss;
            Ic[o] = pref * cc;
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
    hipLaunchKernelGGL(angular_spectrum_kernel, dim3(d.n0, n_f), dim3(256), 0, s, d, f, k_max, Is, Ic);
    NUMAG_HIP_CHECK(hipGetLastError());
    if (As != nullptr && Ac != nullptr) {
        hipLaunchKernelGGL(modal_amplitude_kernel, dim3(n_f), dim3(256), 0, s, Is, Ic, d.n0, k_max, As, Ac);
        NUMAG_HIP_CHECK(hipGetLastError());
    }
    return NUMAG_OK;
}

}  // namespace numag
