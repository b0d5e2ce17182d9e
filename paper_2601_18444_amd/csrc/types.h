// Plain types the kernels take as arguments or read from device memory: the
// detector descriptor, a rotation, and the per-point record of the direct sums.
#pragma once

#include <cstdint>

namespace numag {

// ---------------------------------------------------------------------------
// Detector descriptor passed by value to kernels.
// q(i) = -qmax + i * step on both Cartesian axes (step = 2 qmax / (n - 1));
// polar: q(i) = i * step with step = qmax / (n_q - 1), theta_m = m * dtheta.
// ---------------------------------------------------------------------------
struct Detector {
    int kind;
    int n0, n1;            // rows and columns evaluated
    int n_theta;           // polar: columns of the full detector (theta_m = 2 pi m / n_theta)
    double qmax;
    double step0, step1;   // Cartesian: axis steps (rows, cols); polar: q step, theta step
    double origin0, origin1;
};


// Work split of a Cartesian direct sum over cells |q_M|, |q_N| (cartesian_block.h).
// M is the axis packed into matrix rows (the detector rows unless swapped), N the
// other; A and B count the |q| values, nM and nN the detector's.  |q| value k of an
// axis is (k + first) step, first = 0 on an odd axis and 1/2 on an even one: the pixels
// n - K + k and K - 1 - k, K = ceil(n / 2), lie at +-|q| within the rounding of the
// detector's axis.
struct CartGeom {
    int A, B, nM, nN;
    int na;                 // |q_M| values per row block
    int nz;                 // column blocks (16 |q_N| values) per workgroup: 1, 2, 4 or 8
    int nrb, nzb;           // row blocks and column blocks of the detector
    int swapped;            // M is the column axis of the detector
    double firstM, stepM, firstN, stepN;
    int64_t strideM, strideN;  // pixels
};

// Work split of a polar direct sum (polar_block.h): theta columns [0, cols) of a detector
// of n_out columns are summed; nh = n_out / 2 when column m + nh is filled with the
// conjugate of column m, else 0.
struct PolGeom {
    int n0, n_out;          // q rows, theta columns of the detector
    int cols, nh;
    int na, nrg;            // row blocks (of 32 rows) per wave, row groups
    int mid;                // rows mid + b and mid - 1 - b of a block share offset b: 16; 8 in the block of a
                            // detector of up to 16 rows
    double dq;
};

// Row-major 3x3 rotation as a kernel argument.
struct Rot {
    double m[9];
};

// Per-point record written by the preparation kernel: lab-frame Y, Z (q has
// no x component) and lab-frame weights (n, m'x, m'y, m'z), padded to 64 bytes.
struct alignas(64) PointRec {
    double Y, Z;
    double w[4];
    double pad[2];
};

// A pair of points at (Y, Z) and (-Y, -Z): the sums (even) and differences (odd entries) of
// their weights, per channel.
struct PairRec {
    double Y, Z;
    double w[8];
};

}  // namespace numag
