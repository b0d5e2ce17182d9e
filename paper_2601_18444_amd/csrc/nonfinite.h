// Sums with infinite weights.
//
// The matrix-core sums form a pixel from products of two phasors' parts, RR - II and so
// on, so a weight of infinity makes inf - inf, NaN, where the sum of the terms
// w cos(q.X), -w sin(q.X) is infinite.  A result that is NaN is therefore formed again from
// the terms that are not finite (the finite ones cannot change it any more), where it is
// written: rare and slow, so that the sum kernels only test for it.
#pragma once

#include "numag_internal.h"

namespace numag {

// The points of a sum: records, or a sample's arrays (pos != null) rotated by R.
struct PointSource {
    const PointRec *rec;
    const double *pos, *nuc, *mag;
    Rot R;
};

__device__ __forceinline__ bool is_nan(double2 v) { return v.x != v.x || v.y != v.y; }

// Signs of cos phi and -sin phi: all that a term of infinite weight needs (0 at a sine of
// zero and NaN at a phase that is not finite, as the product would have it).
__device__ __forceinline__ double2 phasor_signs(double phi)
{
    const double t = phi * 0.3183098861837907, k = rint(t), r = t - k;
    const double c = k - 2.0 * floor(0.5 * k) != 0.0 ? -1.0 : 1.0, none = r - r;
    return make_double2(c + none, (r == 0.0 ? 0.0 : r > 0.0 ? -c : c) + none);
}

// The sum over the points [j0, j1) at (q_y, q_z), which came out as v = NaN, from its terms
// that are not finite; v itself if all are.  get(j, Y, Z, w) reads point j.
template <class Get>
__device__ __forceinline__ double2 nonfinite_terms(const Get &get, int64_t j0, int64_t j1, double qy, double qz,
                                                   double2 v)
{
    double2 r = make_double2(0.0, 0.0);
    bool any = false;
#pragma unroll 1
    for (int64_t j = j0; j < j1; ++j) {
        double Y, Z, w;
        get(j, Y, Z, w);
        if (isfinite(w) && isfinite(Y) && isfinite(Z)) continue;
        const double2 e = phasor_signs(qy * Y + qz * Z);
        r.x += w * e.x;
        r.y += w * e.y;
        any = true;
        if (r.x != r.x && r.y != r.y) break;
    }
    return any ? r : v;
}

// Channel ch of point j of a sample (arrays may be null) rotated by R [9].
__device__ __forceinline__ void sample_point(const double *pos, const double *nuc, const double *mag, const double *R,
                                             int ch, int64_t j, double &Y, double &Z, double &w)
{
    auto row = [&](int i, const double *x) { return R[3 * i] * x[0] + R[3 * i + 1] * x[1] + R[3 * i + 2] * x[2]; };
    Y = row(1, pos + 3 * j);
    Z = row(2, pos + 3 * j);
    if (ch == 0)
        w = nuc != nullptr ? nuc[j] : 0.0;
    else if (mag == nullptr)
        w = 0.0;
    else
        w = ch == 1 ? row(0, mag + 3 * j) : ch == 2 ? row(1, mag + 3 * j) : row(2, mag + 3 * j);
}

// The same for channel ch of the points of s.
__device__ __forceinline__ double2 nonfinite_sum(const PointSource &s, int64_t j0, int64_t j1, int ch, double qy,
                                                 double qz, double2 v)
{
    return nonfinite_terms(
        [&](int64_t j, double &Y, double &Z, double &w) {
            if (s.pos != nullptr) {
                sample_point(s.pos, s.nuc, s.mag, s.R.m, ch, j, Y, Z, w);
            } else {
                Y = s.rec[j].Y;
                Z = s.rec[j].Z;
                w = s.rec[j].w[ch];
            }
        },
        j0, j1, qy, qz, v);
}

}  // namespace numag
