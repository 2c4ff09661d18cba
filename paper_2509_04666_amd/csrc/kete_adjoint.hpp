// Adjoint (sky-residual gradient) stage: parameters shared by the host
// layer and kernels.
#pragma once

#include "kete_internal.hpp"

namespace kete {

// Checkpoint: x[3], v[3], wave step, failed flag, force F0[3], F0 valid, the last accepted step's increments
// at nodes 1..7 [7][3], that step (0: none), the checkpoint's time, steps accepted before it
constexpr int kCkptDoubles = 36;
constexpr int kAdjTabDoubles = 8 * (16 + 18);   // constant rows of the reverse sweep
// One accepted step of one object, eight slots of four doubles: slot m < 7
// the increment at node m + 1 and the m-th of x[3], v[3] and the step's
// start time, slot 7 the force at the start and the step size.
constexpr int kStepRec = 32;
// Room for step records: kRecSteps per object and step of a checkpoint
// segment (opts adj_seg_steps).  The steps of one segment, at most that
// number, have their place at the end of a wavefront's; the rest hold the
// forward's steps from the start on.
constexpr int kRecSteps = 9;

struct AdjParams {
    EphemArgs eph;
    RadauConst rc;
    const double* x0;           // [N][6]
    const int32_t* perm;        // [N] object order (bucketed), or null
    double t0;
    int32_t n_obj;
    int32_t k_obs;
    const double* t_obs;        // [N][K], ascending per object, in [t0, t_end]
    const double* obs_pos;      // [N][K][3]
    const double* dL_dsky;      // [N][K][2] (backward)
    double* sky_out;            // [N][K][2] (forward)
    double* grad;               // [N][6] (backward)
    int32_t* status;            // [N]
    double* h_pref;             // [N]
    double* ckpt;               // [C+1][N][kCkptDoubles]
    double t_end;
    double ckpt_days;           // checkpoint c: the first step start at or after t0 + c ckpt_days
    int32_t n_ckpt;             // C segments
    int32_t pad_;
    double* obs_state;          // [N][K][6] states at the observation times (forward)
    double* obs_grad;           // [N][K][6] dL/d(state) at the observation times (backward)
    double* obs_hop;            // [N][K][2] light time and final universal anomaly (forward)
    double* rec;                // [wavefronts][rec_fwd + s_max][objects of one][kStepRec]
    int32_t rec_fwd;            // steps of a wavefront that the forward records
    int32_t pad2_;
    double* adj_tab;            // [kAdjTabDoubles] constant rows of the reverse sweep, written by the forward launch
    double* group_const;        // [kGroupConstDoubles] written by the forward launch
    int32_t s_max;
    int32_t window_segs;        // segments between forced step ends (0: none)
    int32_t max_iter;
    int32_t max_steps;
    double eps, h_min, h_max, h_init, safety;
    double smu, c_light, lt_tol, cos_eps, sin_eps;
    int32_t lt_iter;
    int32_t kepler_iter;
    int32_t zero_start;         // correctors start from zero increments (no extrapolation)
};

// Objects of one adjoint wavefront.  They share their steps, and so also the
// limit on the steps of a checkpoint segment: all of them fail that one of
// them takes past it.
constexpr int kAdjBodies = 8;
inline int64_t adj_waves(int64_t n_obj) { return (n_obj + kAdjBodies - 1) / kAdjBodies; }
inline size_t adj_rec_doubles(int64_t n_obj, int s_max) {
    return (size_t)adj_waves(n_obj) * kAdjBodies * kStepRec * (size_t)(kRecSteps * s_max);
}
hipError_t launch_adjoint(const AdjParams& p, int mode, hipStream_t s);

}  // namespace kete
