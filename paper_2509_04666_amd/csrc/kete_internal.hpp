// Host-side internal interfaces between the C ABI layer and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "kete_device.hpp"
#include "kete_mi.h"

namespace kete {

// Gauss-Radau collocation constants (8 nodes including 0) for the
// increment form of the step: with D_m = F_m - F_0 (m = 1..7),
//   X(s) = x0 + s h v0 + h^2 (s^2/2 F0 + sum_m A_m(s) D_m)
//   V(s) = v0 + h (s F0 + sum_m B_m(s) D_m)
// and the highest monomial coefficient of the acceleration polynomial
//   b6 = sum_m E6[m] D_m.
// Row n = 0..7 is node s_n, row 8 is s = 1.
struct RadauConst {
    double s[9];
    double A[9][7];
    double B[9][7];
    double E6[7];
    double half_s2[9];
    // dense output at any sig in [0, 1]:
    //   A_m(sig) = sum_k Ap[m][k] sig^(k+2),  B_m(sig) = sum_k Bp[m][k] sig^(k+1)
    double Ap[7][8];
    double Bp[7][8];
    // Lagrange basis l_m on the nodes 0, s_1..s_7 (m = 1..7): 1 / prod_{k != m} (s_m - s_k)
    // and l_m(1), to extrapolate a step's increments into the next step
    double Lden[7];
    double L1[7];
};
// The constants the grouped kernels keep in LDS (GroupConst), as laid out by
// fill_group_const: Ap, Bp, then per lane gl = 0..7 of a group the row {s,
// s^2/2, A, B, 2 spare} of its node (gl + 1, and 7 for gl = 7), the nodes
// 1..7, Lden and L1 (7 each), and the step-end weights of D_1..D_7 and F_0 in
// the position and of D_1..D_7 in the velocity.
constexpr int kGroupConstDoubles = 2 * 56 + 8 * 18 + 3 * 7 + 8 + 7;
__host__ __device__ inline double group_const_at(const RadauConst& rc, int i) {
    if (i < 56) return rc.Ap[i / 8][i % 8];
    if (i < 112) return rc.Bp[(i - 56) / 8][i % 8];
    i -= 112;
    if (i < 144) {
        const int n = i / 18 < 7 ? i / 18 + 1 : 7, k = i % 18;
        return k == 0 ? rc.s[n] : k == 1 ? rc.half_s2[n] : k < 9 ? rc.A[n][k - 2] : k < 16 ? rc.B[n][k - 9] : 0.0;
    }
    i -= 144;
    if (i < 7) return rc.s[i + 1];
    if (i < 14) return rc.Lden[i - 7];
    if (i < 21) return rc.L1[i - 14];
    if (i < 28) return rc.A[8][i - 21];
    return i == 28 ? rc.half_s2[8] : rc.B[8][i - 29];
}

// One staged ephemeris window of the integration: [t_a, t_b] lies within
// Chebyshev segments [seg_lo, seg_hi]; out >= 0 marks an output epoch.
struct Window {
    double t_a, t_b;
    int32_t seg_lo, seg_hi;
    int32_t out, pad;
};

// Segment holding time t (floor rule, clamped to the table).
__host__ __device__ inline int seg_clamped(double t, double t_start, double inv_seg, int n_seg) {
    const double k = floor((t - t_start) * inv_seg);
    return k < 0.0 ? 0 : (k > (double)(n_seg - 1) ? n_seg - 1 : (int)k);
}

// The next integration window from t toward target: it ends at target or
// at the segment joint w segment lengths past the start of t's segment,
// whichever comes first (w <= 0: at target), and reads at most w + 1
// consecutive segments (seg_lo..seg_hi), the capacity of the staging buffers
// of the one-lane-per-body kernel.  Every path
// (host plans and the persistent kernel) uses this rule, so they window
// identically.  If t sits on a joint that rounding placed in the earlier
// segment, the limit moves one segment on so the window never has zero
// length.
__host__ __device__ inline Window next_window(double t, double target, double t_start, double seg_days,
                                              double inv_seg, int n_seg, int w) {
    const bool fwd = target > t;
    double tb;
    if (w <= 0) {
        tb = target;
    } else if (fwd) {
        const double kk = floor((t - t_start) * inv_seg);
        double limit = t_start + (kk + w) * seg_days;
        if (!(limit > t)) limit = t_start + (kk + w + 1) * seg_days;
        tb = limit < target ? limit : target;
    } else {
        const double kk = ceil((t - t_start) * inv_seg) - 1.0;
        double limit = t_start + (kk - w + 1) * seg_days;
        if (!(limit < t)) limit = t_start + (kk - w) * seg_days;
        tb = limit > target ? limit : target;
    }
    Window W;
    W.t_a = t;
    W.t_b = tb;
    int lo = seg_clamped(fwd ? t : tb, t_start, inv_seg, n_seg);
    int hi = seg_clamped(fwd ? tb : t, t_start, inv_seg, n_seg);
    if (w > 0 && hi - lo > w) {
        if (fwd) hi = lo + w; else lo = hi - w;
    }
    W.seg_lo = lo;
    W.seg_hi = hi;
    W.out = -1;
    W.pad = 0;
    return W;
}

// The end of the window from t, forward in time only, with the window ends on
// a fixed grid: multiples of w segments from t_start (or the target; w <= 0:
// the target alone).  A run that resumes inside a window (from a checkpoint)
// then ends its windows where the first run did, so both cut their steps at
// the same times.
__host__ __device__ inline double aligned_end(double t, double target, double t_start, double seg_days,
                                              double inv_seg, int w) {
    if (w <= 0) return target;
    const double kk = floor((t - t_start) * inv_seg);
    double limit = t_start + (floor(kk / w) + 1.0) * w * seg_days;
    if (!(limit > t)) limit += w * seg_days;
    return limit < target ? limit : target;
}

struct NbodyParams {
    EphemArgs eph;
    RadauConst rc;
    const double* state_in; // [N][6] states at the launch's start
    double* state;          // [N][6] working state, null when nothing follows the launch
    double* h_pref;         // [N] preferred step (days, > 0)
    const int32_t* perm;    // [N] object order (bucketed) or null
    int32_t* status;        // [N]
    double* x_out;          // [E][N][6]
    unsigned long long* stats;  // [8] or null
    const Window* win;      // windows of this launch
    const double* t_out;    // [E] output epochs (device)
    const double* group_const;  // [kGroupConstDoubles] (device)
    int32_t e_first;        // epochs e_first .. e_land - 1 are read off the step polynomials,
    int32_t e_land;         // epoch e_land ends the launch's last window (no dense epochs: e_first = e_land)
    int32_t n_win;
    int32_t n_obj;
    int32_t max_iter;
    int32_t max_steps;
    int32_t max_win_segs;   // LDS capacity in segments (one lane per object)
    int32_t first_launch;   // no status to read yet
    int32_t zero_start;     // corrector starts from zero increments (no extrapolation)
    int32_t pad_;
    int32_t solo_waves;     // wavefronts of one object each, ahead of the others (G8 kernels)
    int32_t wave_doubles;   // LDS of a wavefront in doubles (set by the launch)
    const int32_t* n_solo;  // device: objects that get one, or null (all of solo_waves do)
    double t_begin;         // start of the launch's first window
    double t_only;          // end of its window when n_win is 1
    double eps, h_min, h_max, h_init, safety;
};

const RadauConst& radau_const();
// The grouped kernels' constants (group_const_at) into device memory by a kernel.
hipError_t launch_group_const(const RadauConst& rc, double* out, hipStream_t s);

// Instantiation of the grouped kernels for a perturber table: 2 and 3 the
// default model's shape (10 bodies, 3 with Eq. A.3, 2 of them with Eq. A.4)
// and that of the Sun with two planets, whose force is unrolled; 1 any other
// count with 13 coefficients, 0 any, also tables of 2^32 values a body.
inline int group_shape(const EphemArgs& E) {
    if (E.deg1 != 13 || (uint64_t)E.n_seg * 3 * E.deg1 > UINT32_MAX) return 0;
    if (E.n_j2 != 2 || E.n_j2g != 2) return 1;
    return E.n_body == 10 && E.n_gr == 3 ? 2 : E.n_body == 3 && E.n_gr == 2 ? 3 : 1;
}

// lanes_per_body: 1 (one lane per object), 8 (an 8-lane group per object) or 7
// (see k_nbody_g8).
hipError_t launch_nbody(const NbodyParams& p, int block, int lanes_per_body, hipStream_t s);

// Stable counting sort of objects into step-size buckets.
// Buckets per octave of the predicted step (the batched jobs' sort), and
// the most buckets one counting-sort pass takes.
constexpr int kBucketSub = 8;
constexpr int kMaxBuckets = 256;

// Sort keys of the bodies of one integrator launch (k_hpref_init): the high
// 16 bits hold the step class, the low 16 the time class; bodies are
// ordered by class, then by time (two stable counting-sort passes).
//   step class 0: bodies for a wavefront of their own (see solo_waves_for and
//     solo_class_steps),
//     with more than kSoloSteps predicted steps shorter than kSoloMaxStep
//     days, the most steps first (16 classes an octave): the bodies of fast
//     orbits, not the slow ones of a long span;
//   step class 1: "critical" bodies, whose predicted step count over the
//     launch exceeds kCritSteps: they set the launch's longest wavefronts,
//     so they come next, ordered by the time of their smallest distance
//     alone (kCritTimeBins classes), which lines up their perihelion
//     passages inside a wavefront;
//   step class 2 + k: the others, kClassSub classes per octave of the
//     predicted step above h_ref, then kTimeBins classes of that time.
constexpr double kCritSteps = 100.0;
constexpr double kSoloSteps = 150.0, kSoloMaxStep = 5.0;
// lanes of an object that has a wavefront of its own, and the list length up
// to which every object has one: two wavefronts a SIMD
constexpr int kSoloAll = 2048;
constexpr int kSoloLanes = 56;
constexpr int kClassSub = 2;
constexpr int kTimeBins = 64;
constexpr int kCritTimeBins = 256;

// One counting-sort pass over a digit of the keys: item i of the input
// order (in_perm[i], or i when in_perm is null) goes to its digit's
// bucket, stably.
struct BucketParams {
    const uint32_t* keys;   // [N] packed keys
    const int32_t* in_perm; // [N] input order or null
    int32_t* perm;          // [N] out
    int32_t* counts;        // [n_buckets][n_blocks] scratch
    int32_t n_obj;
    int32_t n_buckets;      // digit range (<= kMaxBuckets)
    int32_t shift;          // digit = (key >> shift) & 0xffff
    int32_t pad;
};
hipError_t launch_bucket(const BucketParams& p, hipStream_t s);

// Optional live timing of kernel launches with HIP events (per thread).
// kTimeFov brackets every kernel of a field-of-view call (preparation,
// binning, join, exact test, pair sort); kTimeFovJoin the join alone.
enum TimedKernel {
    kTimeNbody = 0, kTimeFov = 1, kTimeAdjoint = 2, kTimeBatch = 3, kTimeFovJoin = 4, kTimeKinds = 8
};
struct TimedScope {
    TimedScope(int kind, hipStream_t s);
    ~TimedScope();
    int kind;
    hipStream_t stream;
    void* stop;
};

// Exclusive scan of int32 counts (n + 1 outputs); scratch >= scan_scratch(n).
size_t scan_scratch_bytes(int64_t n);
hipError_t exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, void* scratch, hipStream_t s);

}  // namespace kete
