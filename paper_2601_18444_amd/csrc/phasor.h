// Small device helpers shared by the sum kernels: complex product, FP64 sine and
// cosine, the unit phasor exp(-i phi), and a detector axis value computed
// exactly as the detector is defined (one rounded product, one rounded sum,
// never fused).
#pragma once

#include <hip/hip_runtime.h>

#include "../../include/numag.h"
#include "types.h"

namespace numag {

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// v summed over the wave, in every lane (fixed order).
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
// LDS operations of a wave complete in order: this only keeps the compiler from
// moving reads and writes across.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// sin x and cos x in FP64 for single angles and phases (the separable tables, column angles,
// object phases; the sum kernels' tables take phasor_fast below).
// Cody-Waite reduction (Cody & Waite, Software Manual for the Elementary
// Functions, 1980): x = k pi/2 + r with pi/2 split into P1 + P2 + P3, P1 and P2
// holding 33 significant bits each, so k P1 and k P2 are exact for |k| < 2^20,
// and P3 the next 53 bits (the split reproduces pi/2 to 1e-37; derived from
// Machin's series for pi).  sin r and cos r on |r| <= pi/4 are the Taylor
// series through r^17 and r^16 (truncation below 0.05 ulp), evaluated by
// Horner's rule in r^2; the quadrant k mod 4 swaps and negates them.  Arguments
// beyond 2^19 take the library sincos.  Host-callable so that its accuracy can
// be checked without a GPU.
// The library call is kept out of line: inlined, its argument reduction takes enough
// registers to push the sum kernels' accumulators into scratch memory.
__host__ __device__ __attribute__((noinline)) static double2 sincos_library(double x)
{
    double s, c;
    sincos(x, &s, &c);
    return make_double2(s, c);
}

// |x| < 2^19 takes the fast path (false also for NaN and infinities).
__host__ __device__ __forceinline__ bool sincos_fast_range(double x) { return fabs(x) < 0x1p19; }

__host__ __device__ __forceinline__ void sincos_fast(double x, double *sp, double *cp)
{
    constexpr double kTwoOverPi = 0x1.45f306dc9c883p-1;
    constexpr double P1 = 0x1.921fb54400000p+0;
    constexpr double P2 = 0x1.0b4611a600000p-34;
    constexpr double P3 = 0x1.3198a2e037073p-69;
    const double k = rint(x * kTwoOverPi);
    const double r = fma(-k, P3, fma(-k, P2, fma(-k, P1, x)));
    const double z = r * r;
    // sin: r + r z (S3 + z (S5 + ... + z S17)),  S_n = (-1)^((n-1)/2) / n!
    double ps = 0x1.952c77030ad4ap-49;
    ps = fma(ps, z, -0x1.ae7f3e733b81fp-41);
    ps = fma(ps, z, 0x1.6124613a86d09p-33);
    ps = fma(ps, z, -0x1.ae64567f544e4p-26);
    ps = fma(ps, z, 0x1.71de3a556c734p-19);
    ps = fma(ps, z, -0x1.a01a01a01a01ap-13);
    ps = fma(ps, z, 0x1.1111111111111p-7);
    ps = fma(ps, z, -0x1.5555555555555p-3);
    const double sn = fma(r * z, ps, r);
    // cos: 1 + z (C2 + z (C4 + ... + z C16)),  C_n = (-1)^(n/2) / n!
    double pc = 0x1.ae7f3e733b81fp-45;
    pc = fma(pc, z, -0x1.93974a8c07c9dp-37);
    pc = fma(pc, z, 0x1.1eed8eff8d898p-29);
    pc = fma(pc, z, -0x1.27e4fb7789f5cp-22);
    pc = fma(pc, z, 0x1.a01a01a01a01ap-16);
    pc = fma(pc, z, -0x1.6c16c16c16c17p-10);
    pc = fma(pc, z, 0x1.5555555555555p-5);
    pc = fma(pc, z, -0x1.0000000000000p-1);
    const double cs = fma(z, pc, 1.0);
    // x = k pi/2 + r: quadrant n = k mod 4
    const int n = (int)k & 3;
    const double s0 = (n & 1) ? cs : sn;
    const double c0 = (n & 1) ? sn : cs;
    *sp = (n & 2) ? -s0 : s0;
    *cp = ((n + 1) & 2) ? -c0 : c0;
}

__host__ __device__ __forceinline__ void sincos_cw(double x, double *sp, double *cp)
{
    if (__builtin_expect(!sincos_fast_range(x), 0)) {
        const double2 r = sincos_library(x);
        *sp = r.x;
        *cp = r.y;
        return;
    }
    sincos_fast(x, sp, cp);
}

// exp(-i phi) = (cos phi, -sin phi)
__host__ __device__ __forceinline__ double2 twiddle(double phi)
{
    double s, c;
    sincos_cw(phi, &s, &c);
    return make_double2(c, -s);
}

// ---------------------------------------------------------------------------
// Unit phasors exp(-i q x) for a coefficient q that many x share (the sum kernels'
// generation phases, where on gfx950 every vector instruction takes time from the matrix
// instructions of its SIMD).  q is held in half turns, q / pi = hi + lo, so the reduction
// is k = rint(hi x), r = (hi x - k) + lo x with fused products: |r| <= 1/2, free of the
// rounding of the phase itself.  exp(-i q x) = (-1)^k (cos(pi r), -sin(pi r)), both by
// polynomials in r^2 (Chebyshev interpolants on [0, 1/4], truncation 3e-19 and 1.5e-17;
// the parity is one shift and two exclusive ors).  22 FP64 and 4 integer instructions,
// against 46 for a sine and cosine reduced to a quarter turn.  The Horner constants are
// scalar operands: left to itself the compiler keeps them in vector registers and copies
// each into the accumulating form of the FMA.  Measured against that sine and cosine
// (with the sum loops read by constant LDS offsets): 24,000 points, 1000 x 1000 polar
// 3.40 -> 3.30 ms; adjoint of 262,144 points, 256 x 256, 2.05 -> 2.01 ms.
// ---------------------------------------------------------------------------
struct HalfTurns {
    double hi, lo;
};

__host__ __device__ __forceinline__ HalfTurns half_turns(double q)
{
    constexpr double kHi = 0x1.45f306dc9c883p-2, kLo = -0x1.6b01ec5417056p-56;  // 1 / pi
    HalfTurns t;
    t.hi = q * kHi;
    t.lo = fma(q, kLo, fma(q, kHi, -t.hi));
    return t;
}

// a b + c with c a scalar constant
__host__ __device__ __forceinline__ double fma_const(double a, double b, double c)
{
#ifdef __HIP_DEVICE_COMPILE__
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
#else
    return fma(a, b, c);
#endif
}

// |hi x| < 2^30 (the parity of k is taken from its integer conversion).
__host__ __device__ __forceinline__ double2 phasor_fast(HalfTurns q, double x)
{
    const double t = q.hi * x;
    const double k = rint(t);
    const double r = fma(q.lo, x, fma(q.hi, x, -k));
    const double w = r * r;
    double s = fma_const(-0x1.9d462020fcc78p-21, w, 0x1.6f7acdb8f6580p-16);  // -sin(pi r) / r
    s = fma_const(s, w, -0x1.e8f3675ee37ddp-12);
    s = fma_const(s, w, 0x1.e3074dfaf87afp-8);
    s = fma_const(s, w, -0x1.5078348551854p-4);
    s = fma_const(s, w, 0x1.32d2cce627c86p-1);
    s = fma_const(s, w, -0x1.466bc6775aa7dp+1);
    s = fma_const(s, w, 0x1.4abbce625be52p+2);
    s = fma_const(s, w, -0x1.921fb54442d18p+1);
    s *= r;
    double c = fma_const(0x1.179a329ef4140p-18, w, -0x1.b6a6feabe52e9p-14);  // (cos(pi r) - 1) / r^2
    c = fma_const(c, w, 0x1.f9d2c1f3b2167p-10);
    c = fma_const(c, w, -0x1.a6d1f12b0bef2p-6);
    c = fma_const(c, w, 0x1.e1f5068620bcbp-3);
    c = fma_const(c, w, -0x1.55d3c7e3c9051p+0);
    c = fma_const(c, w, 0x1.03c1f081b5a9fp+2);
    c = fma_const(c, w, -0x1.3bd3cc9be45dep+2);
    c = fma(c, w, 1.0);
    const long long odd = (long long)((unsigned long long)(unsigned int)(int)k << 63);
#ifdef __HIP_DEVICE_COMPILE__
    return make_double2(__longlong_as_double(__double_as_longlong(c) ^ odd),
                        __longlong_as_double(__double_as_longlong(s) ^ odd));
#else
    return odd ? make_double2(-c, -s) : make_double2(c, s);
#endif
}

// Largest |x| the fast form takes for coefficients up to |q|.
__host__ __device__ __forceinline__ double phasor_range(double q) { return 0x1p30 / (fabs(q) * 0.3183098861837907 + 0x1p-900); }

// exp(-i q x) through the library (any x; NaN for NaN and infinities), out of line.
__host__ __device__ __attribute__((noinline)) static double2 phasor_library(HalfTurns q, double x)
{
    double s, c;
    sincos((q.hi * 3.141592653589793) * x, &s, &c);
    return make_double2(c, -s);
}

// Two phasors; `fast` is whether both arguments are in range.
__device__ __forceinline__ void phasor2(HalfTurns q0, double x0, HalfTurns q1, double x1, bool fast, double2 &e0,
                                        double2 &e1)
{
    if (__builtin_expect(!fast, 0)) {
        e0 = phasor_library(q0, x0);
        e1 = phasor_library(q1, x1);
    } else {
        e0 = phasor_fast(q0, x0);
        e1 = phasor_fast(q1, x1);
    }
}

__device__ __forceinline__ double2 phasor(HalfTurns q, double x, bool fast)
{
    return __builtin_expect(!fast, 0) ? phasor_library(q, x) : phasor_fast(q, x);
}

// origin + i * step
__device__ __forceinline__ double axis_value(double origin, int i, double step)
{
#pragma clang fp contract(off)
    double t = (double)i * step;
    return origin + t;
}

// Unit vector of pixel p of a full detector (Cartesian: q / |q| with q = 0 -> e_z,
// |q| without fused operations; polar: the column angle, also at q = 0):
// qhat = (0, s, c).
__device__ __forceinline__ void pixel_qhat(const Detector &d, int64_t p, double &s, double &c)
{
    // (a 64-bit division takes several times the instructions of the rest)
    const int row = p < ((int64_t)1 << 32) ? (int)((uint32_t)p / (uint32_t)d.n1) : (int)(p / d.n1);
    const int col = (int)(p - (int64_t)row * d.n1);
    if (d.kind == NUMAG_GRID_CARTESIAN) {
        const double qy = axis_value(d.origin0, row, d.step0);
        const double qz = axis_value(d.origin1, col, d.step1);
        if (qy == 0.0 && qz == 0.0) {
            s = 0.0;
            c = 1.0;
            return;
        }
        double qn;
        {
#pragma clang fp contract(off)
            double a2 = qy * qy;
            double b2 = qz * qz;
            qn = sqrt(a2 + b2);
        }
        s = qy / qn;
        c = qz / qn;
    } else {
        const double th = (2.0 * 3.141592653589793 * (double)col) / (double)d.n_theta;
        sincos(th, &s, &c);
    }
}

}  // namespace numag
