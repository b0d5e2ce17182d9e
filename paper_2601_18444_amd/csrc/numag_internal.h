// Internal declarations of the numag HIP library (gfx950).  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <memory>
#include <string>
#include <vector>

#include "../../include/numag.h"
#include "types.h"

namespace numag {

// ---------------------------------------------------------------------------
// Error reporting (thread-local message behind numag_last_error()).
// ---------------------------------------------------------------------------
void set_error(const std::string &msg);
void clear_error();

#define NUMAG_HIP_CHECK(expr)                                                        \
    do {                                                                             \
        hipError_t err_ = (expr);                                                    \
        if (err_ != hipSuccess) {                                                    \
            ::numag::set_error(std::string(#expr) + ": " + hipGetErrorString(err_)); \
            return NUMAG_E_HIP;                                                      \
        }                                                                            \
    } while (0)

// ---------------------------------------------------------------------------
// Kernel timer: TimedLaunch brackets one kernel launch with a HIP event pair
// on its stream while numag_kernel_timer is enabled.
// ---------------------------------------------------------------------------
bool timer_enabled();
int timer_begin(int kernel, hipStream_t s);   // returns a record id, or -1
void timer_end(int id, hipStream_t s);

struct TimedLaunch {
    int id;
    hipStream_t s;
    TimedLaunch(int kernel, hipStream_t st) : id(timer_enabled() ? timer_begin(kernel, st) : -1), s(st) {}
    ~TimedLaunch()
    {
        if (id >= 0) timer_end(id, s);
    }
};

// Most workgroups of `threads` a launch takes along x: a grid of 2^32 threads or more is
// not refused but truncated to 32 bits, so kernels that may be asked for more loop.
constexpr int64_t max_workgroups(int threads) { return ((int64_t)1 << 31) / threads; }

Detector make_detector(const numag_qgrid &g);

// Validation of a numag_amplitudes request (sample, detector, rotations, path and
// mode); `fn` prefixes the error message.  NUMAG_OK or the status to return.
int validate_amplitudes_request(const numag_sample *sample, int64_t n_rot, const double *rot,
                                const numag_qgrid *grid, int32_t path, int32_t mode, const char *fn);

// ---------------------------------------------------------------------------
// Launchers (each enqueues on `stream`, returns NUMAG_OK or NUMAG_E_HIP).
// ---------------------------------------------------------------------------

// X_j = R (x_j + r^{k(j)}), w'_j = (n_j, R m_j) of the points j in [j_lo, j_hi),
// written to out[j - j_lo].  The object of a point follows from the HOST CSR
// offsets h_offsets [K+1] (read on the host and passed to the kernels by value,
// in groups of objects; unused when obj_pos is nullptr or K == 1).
int launch_prepare_points(const double *pos, const double *nuc, const double *mag, int64_t j_lo, int64_t j_hi,
                          const numag_regular *regular, const int64_t *h_offsets, int64_t K,
                          const double *obj_pos, const Rot &R, PointRec *out, hipStream_t s);

// Split of a Cartesian direct sum (cartesian_block.h).
struct CartPlan {
    CartGeom g;
    int mt;          // 16-row matrix tiles per wave
    int shape;       // launch shape (8, 64, 16, 32: 1, 2, 4, 8 column blocks per workgroup)
    int channels;
    int nsplit;
    int64_t per;     // points per split (a multiple of 4)
    int col_groups;  // workgroups along N
};
// The count NUMAG_TARGET_WGS asks for (0: not set).
int env_target();

// ---------------------------------------------------------------------------
// Launch-shape table (tune.hip): tuned shapes keyed by kernel, the evaluated
// detector and the point-count class; plans fall back to the defaults below.
// ---------------------------------------------------------------------------
enum { kTuneDirect = 0, kTuneAdjoint = 1, kTuneObjects = 2, kTuneKernelCount = 3 };
struct TuneShape {
    int shape;   // Cartesian: column blocks (cart_nz); polar: row blocks per wave; adjoint: 0
    int target;  // workgroups (objects: work items) a launch aims for
};
// An entry: a launch shape, or (untuned) the autotuner's finding that the library's own plan,
// which also knows the sample's channels and objects, is the fastest; `shape` then only names
// the default.
struct TuneEntry {
    TuneShape shape;
    double ms, default_ms;  // measured by numag_autotune (0 when set directly or unknown)
    bool untuned;
};
int tune_wclass(int64_t W);
bool tune_entry(int kernel, const Detector &d, int64_t W, TuneEntry *out);
// The shape a plan has to take: false without a valid one in the table.
bool tuned_shape(int kernel, const Detector &d, int64_t W, TuneShape *out);
void tune_store(int kernel, const Detector &d, int64_t W, const TuneEntry &e);
void tune_erase(int kernel, const Detector &d, int64_t W);
int tune_save();
void tune_clear();
bool valid_tune_shape(int kernel, const Detector &d, const TuneShape &s);
// The library's untuned shape for a kernel on the whole detector d and W points (four
// channels; the objects are not known).
TuneShape default_tune_shape(int kernel, const Detector &d, int64_t W);
// The shape in use: the tuned one if the table holds it under `key` (the evaluated part), else
// the default.
TuneShape current_tune_shape(int kernel, const Detector &d, const Detector &key, int64_t W);
// Plan of a Cartesian sum on the whole detector d.  The launch shape is looked up
// under the part of the detector that the caller's path stands for (hermitian: the
// first ceil(n0 / 2) rows); either way every pixel is written, the mirrored ones as
// conjugates.  max_partial > 0 caps the bytes of partial sums.
CartPlan plan_direct_cartesian(const Detector &d, int64_t W, int channels, bool hermitian, size_t max_partial = 0);
// Estimated cycles of that sum under the library's own launch shape.
double cart_default_cost(const Detector &d, int64_t W, int channels);
// Cells, row blocks and matrix tiles of detector d for `channels` (cartesian_block.h).
void cart_geometry(const Detector &d, int channels, CartGeom &g, int &mt);
// The geometry of the object sums (four channels, column blocks of `shape`) in the cheaper
// orientation; its cycles per chunk of points, and (group) those of a workgroup of all its
// column blocks and of the last, partial one.
double cart_objects_geometry(const Detector &d, int shape, CartGeom &g, int &mt, double *group);
// Column blocks per workgroup of a launch shape.
int cart_nz(int shape);
// Bytes of partial sums (0 when one split writes the sums directly).
size_t cart_partial_bytes(const CartPlan &p);
// Writes (accumulate: adds) the sums of all pixels of the detector to amp [P][8].
int launch_direct_cartesian(const PointRec *pts, int64_t W, const CartPlan &p, double *partial, double *amp,
                            int accumulate, hipStream_t s);
// The same from a sample's arrays, rotated by R as they are read (no object offsets; the
// arrays of channels outside the plan's set are not read).
int launch_sample_cartesian(const double *pos, const double *nuc, const double *mag, const Rot &R, int64_t W,
                            const CartPlan &p, double *partial, double *amp, hipStream_t s);

// Polar detector direct sum (polar_block.h).
constexpr int kPolarShapeCount = 5;
struct PolarPlan {
    PolGeom g;
    int mt;          // 16-row matrix tiles per wave; 0, -1: one, two of 4 rows; -2, -3: of 8 offsets
    int shape;       // launch shape: 1, 0, 2, 3, 4 for 1, 2, 4, 8 or 16 row blocks of 32 per wave
    int channels;    // channels summed: 4 (N, M), 3 (M only) or 1 (N only); the rest are written as 0
    int nsplit;      // point ranges summed by different workgroups
    int64_t per;     // points per split
};
int default_polar_shape(const Detector &d);
// Row groups, columns and tiles of detector d for `channels` under a launch shape.
void polar_geometry(const Detector &d, int channels, int shape, PolGeom &g, int &mt);
TuneShape default_polar_tune(const Detector &d, int64_t W);
// Plan on the whole detector d; the launch shape is looked up under the part the path
// stands for (hermitian: half of the columns).  Every pixel is written; columns
// theta + pi of an even detector as conjugates.  max_partial > 0 caps the partial sums.
PolarPlan plan_direct_polar(const Detector &d, int64_t W, int channels, bool hermitian, size_t max_partial = 0);
size_t polar_partial_bytes(const PolarPlan &p);
int launch_direct_polar(const PointRec *pts, int64_t W, const PolarPlan &p, double *partial, double *amp,
                        int accumulate, hipStream_t s);
// The same from a sample's arrays, as launch_sample_cartesian.
int launch_sample_polar(const double *pos, const double *nuc, const double *mag, const Rot &R, int64_t W,
                        const PolarPlan &p, double *partial, double *amp, hipStream_t s);
// Sums of 1 to 4 channels over pairs of points.
int launch_polar_pairs(const PairRec *pts, int64_t n, const PolarPlan &p, double *partial, double *amp, hipStream_t s);
// out[i] = value for i < n (a kernel, so that callers may capture it in a graph).
int launch_fill(double *out, int64_t n, double value, hipStream_t s);

// Work items (object slot, pixel block) of the object kernel; each sums complete objects
// and adds F F^H (and, in split mode, exp(-i q.R r^k) F) into accumulators no other item
// touches; slots are reduced in a fixed order.
struct ObjectsPlan {
    CartGeom cg;     // Cartesian detector
    PolGeom pg;      // polar detector
    int mt;          // matrix tiles per wave; -1, -3 (polar): two of 4 rows
    int64_t n_blocks;  // pixel blocks (items per slot)
    int64_t strips;  // accumulator strips of a slot (sixteen pixels each)
    int n_slots;     // accumulator slots (object set x rotation range)
    int n_out;       // spectral matrices written (K per object, or 1)
    int64_t n_items;
};

// An object-mode (DILUTE / SPLIT) plan: everything the kernels need that depends
// on the host arguments (object offsets, rotations, work tables), as an image the
// caller uploads to the start of its workspace.  The image begins with a tag
// unique to the plan; the kernels compare it with the plan's and write NaN
// instead of reading tables that another plan, or other data, left there.
constexpr size_t kPlanTagBytes = 256;
struct ObjPlanTables;  // the persistent kernel's work tables (objects.hip)
struct ObjPlan {
    unsigned long long tag;
    Detector d;                 // the whole detector
    int path, mode, spec_per_object;
    int64_t n_rot, K, W;
    std::vector<int64_t> off;   // [K+1] host copy of the object offsets
    std::vector<char> image;    // uploaded to workspace offset 0: the tag, then the tables
    size_t o_rot = 0;           // rotations [n_rot][9] (doubles) within the image
    size_t ws_bytes = 0;        // workspace bytes the plan's calls need
    std::shared_ptr<ObjPlanTables> tables;  // the persistent kernel's tables
};
// Detector part an object-mode path stands for (the key of its launch shape): all of d,
// or with `hermitian` the first ceil(n0 / 2) rows of a Cartesian detector or the theta
// columns [0, n_theta / 2) of a polar one.
Detector objects_detector(const Detector &d, bool hermitian);
// Fills pl.tables, pl.image (rotations excepted), pl.o_rot and pl.ws_bytes of a plan
// whose other fields are set (either detector kind).
void build_objects_plan(ObjPlan &pl);
// Enqueues the sums of a plan whose image is in `ws` (kernels only).
int launch_objects_plan(const ObjPlan &pl, const numag_sample &s, double *spec_out, double *amp_out, void *ws,
                        hipStream_t st);

// cross sections from amplitudes ([n_sets][P][8]) or spectra ([n_sets][P][16]).
int launch_cross_section(const Detector &d, int64_t n_sets, const double *amp, const double *spec,
                         const numag_consts &c, uint32_t mask, double *out, hipStream_t s);
// spec = scale A A^H per set and pixel (accumulate: spec += scale A A^H)
int launch_spectral_matrix(int64_t n_sets, int64_t P, const double *amp, double *spec, hipStream_t s,
                           double scale = 1.0, int accumulate = 0);

// a8
int launch_azimuthal(const Detector &d, const double *f, int n_f, int n_bins, double qmax_avg,
                     double *I, int64_t *count, hipStream_t s);

// a9
int launch_correlation(const double *q, const double *I, int n_q, int n_f, const double *r, int n_r,
                       double scale, double *c, double *p, hipStream_t s);

// residual weights, loss, adjoint sum (hermitian: which table entry sets the split; the
// adjoint always runs on residual weights folded onto the independent pixels).
int launch_grad(const PointRec *pts, int64_t W, const Detector &d, const numag_consts &c,
                const double *amp, const double *target, const double *weight, double *loss,
                double *dnuc, double *dmag, const Rot &R, void *ws, size_t ws_bytes, hipStream_t s,
                bool hermitian = false);
// Workspace bytes of launch_grad on detector d (whole), for the path it will run.
size_t grad_workspace_bytes(const Detector &d, int64_t W, bool hermitian);
int default_adjoint_target(const Detector &d, int64_t W);

// 2D correlation function (eq. crav2d) from data on detector d onto real-space grid rd.
size_t correlation_2d_workspace_bytes(const Detector &d, const Detector &rd);
int launch_correlation_2d(const Detector &d, const double *f, int n_f, const Detector &rd, double *C, void *ws,
                          size_t ws_bytes, hipStream_t s);

// Angular spectrum (eqs. CosineSinceIntensities, ModalAmplitudes) on a polar detector.
int launch_angular_spectrum(const Detector &d, const double *f, int n_f, int k_max, double *Is, double *Ic,
                            double *As, double *Ac, hipStream_t s);

// regular-grid separable path on the matrix cores, for n_snap weight snapshots
// (nuc [n_snap][W], mag [n_snap][W][3]; amp [n_snap][P][8]).  pixels: the points are the
// pixels of a detector, their coordinates rounded as its axes are.
int launch_separable(const double *nuc, const double *mag, const numag_regular &g, const Detector &d,
                     int path, int64_t n_snap, double *amp, void *ws, size_t ws_bytes, hipStream_t s,
                     bool pixels = false);
size_t separable_workspace_bytes(const numag_regular &g, const Detector &d, int path, int64_t n_snap);

}  // namespace numag
