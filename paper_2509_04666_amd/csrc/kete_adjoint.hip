// Gradient of sky-position residuals with respect to the initial state.
//
// Forward: the collocation integrator of the propagation kernels (8-lane
// group per object, wave-shared steps) takes its own steps; checkpoint c
// is the state at the first step start at or after t0 + c ckpt_days, and
// observations at per-object times are read off the step's collocation
// polynomial, hopped with light time to the emission point (Sect. 2) and
// turned into RA/Dec.
//
// Backward: the discrete adjoint of that forward map, swept over the steps
// last to first, a wavefront at a time.  A step's start and node increments
// were recorded by the forward (or, past its room for them, are recomputed
// checkpoint segment by segment, the same steps bit for bit); the force
// Jacobians at its 8 nodes follow from them, and the linear stage equations
// of the step's transpose are solved by fixed-point iteration, all in
// registers.  The light-time hop's
// Jacobian comes from one forward-mode (six-direction dual number)
// evaluation of the universal-variable solution at its converged anomaly
// plus the implicit light-time term.
#include <math.h>

#include "kete_adjoint.hpp"
#include "kete_radau.hpp"

namespace kete {
namespace {

// ---------------------------------------------------------------- duals
struct D6 {
    double v, d[6];
};
__device__ __forceinline__ D6 mk(double v) { D6 r; r.v = v; for (int i = 0; i < 6; ++i) r.d[i] = 0.0; return r; }
__device__ __forceinline__ D6 operator+(const D6& a, const D6& b) { D6 r; r.v = a.v + b.v; for (int i = 0; i < 6; ++i) r.d[i] = a.d[i] + b.d[i]; return r; }
__device__ __forceinline__ D6 operator-(const D6& a, const D6& b) { D6 r; r.v = a.v - b.v; for (int i = 0; i < 6; ++i) r.d[i] = a.d[i] - b.d[i]; return r; }
__device__ __forceinline__ D6 operator*(const D6& a, const D6& b) { D6 r; r.v = a.v * b.v; for (int i = 0; i < 6; ++i) r.d[i] = a.d[i] * b.v + a.v * b.d[i]; return r; }
__device__ __forceinline__ D6 operator*(double s, const D6& a) { D6 r; r.v = s * a.v; for (int i = 0; i < 6; ++i) r.d[i] = s * a.d[i]; return r; }
__device__ __forceinline__ D6 operator/(const D6& a, const D6& b) {
    D6 r; r.v = a.v / b.v;
    const double ib = 1.0 / b.v;
    for (int i = 0; i < 6; ++i) r.d[i] = (a.d[i] - r.v * b.d[i]) * ib;
    return r;
}
__device__ __forceinline__ D6 dsqrt(const D6& a) {
    D6 r; r.v = sqrt(a.v);
    const double k = 0.5 / r.v;
    for (int i = 0; i < 6; ++i) r.d[i] = a.d[i] * k;
    return r;
}

// Stumpff c0..c3 on dual arguments (series after quartering, then the
// quadrupling identities, as in the scalar version).
__device__ __forceinline__ void stumpff_d(D6 z, D6& c0, D6& c1, D6& c2, D6& c3) {
    int n = 0;
    while (fabs(z.v) > 0.1 && n < 64) { z = 0.25 * z; ++n; }
    const double a2[8] = {1.0 / 2.0, 1.0 / 24.0, 1.0 / 720.0, 1.0 / 40320.0, 1.0 / 3628800.0, 1.0 / 479001600.0,
                          1.0 / 87178291200.0, 1.0 / 20922789888000.0};
    const double a3[8] = {1.0 / 6.0, 1.0 / 120.0, 1.0 / 5040.0, 1.0 / 362880.0, 1.0 / 39916800.0, 1.0 / 6227020800.0,
                          1.0 / 1307674368000.0, 1.0 / 355687428096000.0};
    c2 = mk(a2[7]); c3 = mk(a3[7]);
    for (int k = 6; k >= 0; --k) {
        c2 = mk(a2[k]) - z * c2;
        c3 = mk(a3[k]) - z * c3;
    }
    c0 = mk(1.0) - z * c2;
    c1 = mk(1.0) - z * c3;
    for (; n > 0; --n) {
        D6 n0 = 2.0 * (c0 * c0) - mk(1.0);
        D6 n1 = c0 * c1;
        D6 n2 = 0.5 * (c1 * c1);
        D6 n3 = 0.25 * (c2 + c0 * c3);
        c0 = n0; c1 = n1; c2 = n2; c3 = n3;
    }
}

// P = d r(dt) / d(r0, v0) (3 x 6) of the two-body hop at fixed dt, given
// the converged universal anomaly chi: the implicit dependence of chi is
// one Newton correction evaluated in dual arithmetic.
__device__ void hop_jacobian(double mu, double smu, const double r0v[3], const double v0v[3], double dt, double chi,
                             double P[3][6]) {
    D6 r0[3], v0[3];
    for (int i = 0; i < 3; ++i) {
        r0[i] = mk(r0v[i]); r0[i].d[i] = 1.0;
        v0[i] = mk(v0v[i]); v0[i].d[3 + i] = 1.0;
    }
    const D6 r0n = dsqrt(r0[0] * r0[0] + r0[1] * r0[1] + r0[2] * r0[2]);
    const D6 s0 = (1.0 / smu) * (r0[0] * v0[0] + r0[1] * v0[1] + r0[2] * v0[2]);
    const D6 alpha = mk(2.0) / r0n - (1.0 / mu) * (v0[0] * v0[0] + v0[1] * v0[1] + v0[2] * v0[2]);
    D6 x = mk(chi);
    D6 c0, c1, c2, c3;
    stumpff_d(alpha * x * x, c0, c1, c2, c3);
    const D6 F = r0n * x * c1 + s0 * x * x * c2 + x * x * x * c3 - mk(smu * dt);
    const D6 Fp = r0n * c0 + s0 * x * c1 + x * x * c2;
    D6 xd = F;
    for (int i = 0; i < 6; ++i) xd.d[i] = -F.d[i] / Fp.v;
    xd.v = chi;
    stumpff_d(alpha * xd * xd, c0, c1, c2, c3);
    const D6 f = mk(1.0) - xd * xd * c2 / r0n;
    const D6 g = mk(dt) - (1.0 / smu) * (xd * xd * xd * c3);
    for (int i = 0; i < 3; ++i) {
        const D6 r = f * r0[i] + g * v0[i];
        for (int k = 0; k < 6; ++k) P[i][k] = r.d[k];
    }
}

// RA/Dec of an ecliptic direction (equator of J2000 by the obliquity) and
// d(ra, dec)/d(d_ecl).
__device__ __forceinline__ void radec(const double d[3], double ce, double se, double& ra, double& dec, double J[6]) {
    const double q[3] = {d[0], ce * d[1] - se * d[2], se * d[1] + ce * d[2]};
    const double rho2 = q[0] * q[0] + q[1] * q[1], rho = sqrt(rho2), n2 = rho2 + q[2] * q[2];
    ra = atan2(q[1], q[0]);
    if (ra < 0.0) ra += 6.283185307179586476925286766559;
    dec = atan2(q[2], rho);
    const double da[3] = {-q[1] / rho2, q[0] / rho2, 0.0};
    const double dd[3] = {-q[0] * q[2] / (n2 * rho), -q[1] * q[2] / (n2 * rho), rho / n2};
    J[0] = da[0]; J[1] = ce * da[1] + se * da[2]; J[2] = -se * da[1] + ce * da[2];
    J[3] = dd[0]; J[4] = ce * dd[1] + se * dd[2]; J[5] = -se * dd[1] + ce * dd[2];
}

struct SunGlobal {
    EphemArgs E;
    __device__ __forceinline__ void eval(double t, double pos[3], double vel[3]) const {
        cheb_body(E.coef, 0, E.deg1, t, E.t_start, E.seg_days, E.inv_seg, 0, E.n_seg - 1, pos, vel);
    }
    __device__ bool covers(double) const { return true; }
    __device__ void center(double) const {}
};

// Light-time hop of the state (x, v) at t_obs seen from o: direction d,
// light time, emission velocity, the heliocentric start (r0, v0) and the
// converged universal anomaly of the final hop.
__device__ __forceinline__ int hop(const AdjParams& p, const SunGlobal& sun, double t_obs, const double xs[3],
                                   const double vs[3], const double o[3], double d[3], double& tau, double ve[3],
                                   double r0[3], double v0[3], double& chi) {
    double S[3], Sd[3];
    sun.eval(t_obs, S, Sd);
    for (int i = 0; i < 3; ++i) { r0[i] = xs[i] - S[i]; v0[i] = vs[i] - Sd[i]; }
    return lighttime(sun, p.eph.gm[0], p.smu, p.c_light, p.lt_tol, p.lt_iter, t_obs, r0, v0, t_obs, o, d, tau, ve,
                     &chi, p.kepler_iter);
}

// The same hop from the light time and universal anomaly the forward
// converged to: one warm-started Kepler evaluation, no light-time loop.
__device__ __forceinline__ void hop_known(const AdjParams& p, const SunGlobal& sun, double t_obs, const double xs[3],
                                          const double vs[3], const double o[3], double tau, double& chi,
                                          double d[3], double ve[3], double r0[3], double v0[3]) {
    double S[3], Sd[3], r[3], v[3], Se[3], Sde[3];
    sun.eval(t_obs, S, Sd);
    for (int i = 0; i < 3; ++i) { r0[i] = xs[i] - S[i]; v0[i] = vs[i] - Sd[i]; }
    bool quick;
    kepler_uv(p.eph.gm[0], p.smu, r0, v0, -tau, chi, r, v, p.kepler_iter, quick);
    sun.eval(t_obs - tau, Se, Sde);
    for (int i = 0; i < 3; ++i) {
        d[i] = Se[i] + r[i] - o[i];
        ve[i] = Sde[i] + v[i];
    }
}

// dL/d(x, v) at t_obs from dL/d(ra, dec) through the sky projection and
// the light-time hop (implicit tau: dx_e = P dz - v_e (u . dx_e) / c),
// given the forward's light time and universal anomaly.
__device__ void hop_vjp(const AdjParams& p, const SunGlobal& sun, double t_obs, const double xs[3], const double vs[3],
                        const double o[3], double tau, double chi, double gra, double gdec, double lx[3],
                        double lv[3]) {
    double d[3], ve[3], r0[3], v0[3];
    hop_known(p, sun, t_obs, xs, vs, o, tau, chi, d, ve, r0, v0);
    double ra, dec, J[6];
    radec(d, p.cos_eps, p.sin_eps, ra, dec, J);
    double gd[3];
    for (int i = 0; i < 3; ++i) gd[i] = gra * J[i] + gdec * J[3 + i];
    const double dn = sqrt(dot3(d, d));
    const double u[3] = {d[0] / dn, d[1] / dn, d[2] / dn};
    const double cu = p.c_light + dot3(u, ve);
    const double vg = dot3(ve, gd);
    double gP[3];
    for (int i = 0; i < 3; ++i) gP[i] = gd[i] - u[i] * vg / cu;
    double P[3][6];
    hop_jacobian(p.eph.gm[0], p.smu, r0, v0, -tau, chi, P);
    for (int k = 0; k < 3; ++k) {
        lx[k] = gP[0] * P[0][k] + gP[1] * P[1][k] + gP[2] * P[2][k];
        lv[k] = gP[0] * P[0][3 + k] + gP[1] * P[1][3 + k] + gP[2] * P[2][3 + k];
    }
}

// ---------------------------------------------------------------- forward
// Both passes integrate each object as an 8-lane group (one lane per
// collocation node, 8 objects per wavefront, wave-shared steps) with the
// step loop of the propagation kernels.

// Checkpoint c of object j at time t: state, the step size to resume
// with, a failure flag, the force at the state (with whether it was
// evaluated yet), and the last accepted step with its node increments, so
// that a recompute repeats the forward's steps exactly (extrapolated
// corrector starts included).  Lanes 0..7 of the group write the first
// eight values, lanes 0..3 the force, lanes 0..6 their node's increment
// and lane 7 the step, the time and the number of steps before it.
__device__ __forceinline__ void save_ckpt_g8(const AdjParams& p, int c, int j, int gl, const G8State& S, double t,
                                             int n_steps) {
    double* ck = p.ckpt + ((size_t)c * p.n_obj + j) * kCkptDoubles;
    const double v = gl < 6 ? state_component(S.x0, S.v0, gl)
                            : gl == 6 ? S.hw : (S.active ? 0.0 : (double)(S.status ? S.status : 1));
    ck[gl] = v;
    const double f = gl < 3 ? vector_component(S.F0, gl) : (S.haveF0 ? 1.0 : 0.0);
    if (gl < 4) ck[8 + gl] = f;
    if (gl < 7) {
#pragma unroll
        for (int i = 0; i < 3; ++i) ck[12 + 3 * gl + i] = S.Dp[i];
    } else {
        ck[33] = S.hprev;
        ck[34] = t;
        ck[35] = (double)n_steps;
    }
}


__device__ __forceinline__ void init_lane_state(const AdjParams& p, bool valid, int j, G8State& S) {
    S.status = 0;
    S.active = valid;
    for (int i = 0; i < 3; ++i) {
        S.x0[i] = valid ? p.x0[6 * j + i] : (i == 0 ? 1.0 : 0.0);
        S.v0[i] = valid ? p.x0[6 * j + 3 + i] : 0.0;
        S.F0[i] = 0.0;
    }
    S.hp_new = kInf;
    S.haveF0 = false;
}

// One step of this lane's object into its slot of the record at rec (see
// kStepRec).
__device__ __forceinline__ void write_step(double* __restrict__ rec, int gl, double ts, double h, const double dn[3],
                                           const G8State& S) {
    const double q = gl < 6 ? state_component(S.x0, S.v0, gl) : ts;
    double2* w = reinterpret_cast<double2*>(rec + 4 * gl);
    w[0] = gl < 7 ? make_double2(dn[0], dn[1]) : make_double2(S.F0[0], S.F0[1]);
    w[1] = gl < 7 ? make_double2(dn[2], q) : make_double2(S.F0[2], h);
}

template <int NB, int NGR, int NJ2, int DEG1>
__global__ __launch_bounds__(64, 2) void k_adjoint_fwd(const AdjParams p) {
    extern __shared__ __align__(16) double smem[];
    const int lane = threadIdx.x;
    const GroupMap<kGroup> M(lane);
    const int gl = M.gl;
    const EphemArgs& E = p.eph;
    __shared__ __align__(16) GroupConst gc;
    __shared__ __align__(16) double wt_all[kAdjBodies * 16];
    load_group_const(p.group_const, &gc, lane, kWave);
    const G8Lds T = g8_lds<kGroup>(E, smem, M.grp);
    g8_table_init<kGroup>(E, lane, smem);
    __syncthreads();
    const long gi = (long)blockIdx.x * kAdjBodies + M.grp;
    const bool valid = gi < p.n_obj;
    const int j = valid ? (p.perm ? p.perm[gi] : (int)gi) : 0;
    double* rec = p.rec + ((size_t)blockIdx.x * (p.rec_fwd + p.s_max) * kAdjBodies + M.grp) * kStepRec;
    G8State S;
    init_lane_state(p, valid, j, S);
    S.hw = groups_min(valid ? p.h_pref[j] : kInf);
    if (!(S.hw < kInf)) S.hw = p.h_init;
    S.t = p.t0;
    G8Count C;
    const int K = p.k_obs;
    int kobs = 0;
    const double* tob = p.t_obs + (size_t)j * K;
    // The group's lanes hold the times of eight observations, k_buf .. k_buf
    // + 7, so that a step seldom loads: a load waits for the states stored
    // before it.
    int k_buf = 0;
    double t_buf = 0.0;
    auto load_times = [&]() {
        k_buf = kobs;
        t_buf = valid && kobs + gl < K ? tob[kobs + gl] : kInf;
    };
    auto next_time = [&]() { return __shfl(t_buf, kobs - k_buf, kGroup); };        // the whole group calls it
    auto advance = [&]() {
        if (++kobs - k_buf == kGroup) load_times();
    };
    load_times();
    auto store_obs = [&](double v) {
        if (gl < 6) p.obs_state[((size_t)j * K + kobs) * 6 + gl] = v;
    };
    // observations at the start epoch
    for (;;) {
        const bool at = valid && kobs < K && next_time() <= S.t;
        if (__ballot(at) == 0ull) break;
        const double v = state_component(S.x0, S.v0, gl < 6 ? gl : 5);
        if (at) { store_obs(v); advance(); }
    }
    double* wt = wt_all + 16 * M.grp;
    const bool vel = gl >= 3;
    const int comp = vel ? (gl < 6 ? gl - 3 : 2) : gl;
    // Checkpoint c (1 .. C - 1) is the state at the first accepted step
    // start at or after t0 + c ckpt_days (wave-uniform: the wavefront's
    // objects share their steps), so steps are not cut at checkpoints.
    int c_next = 1, n_steps = 0;
    // (te is the time the step lands on: ts + h may round below the last observation)
    auto visit = [&](double ts, double te, double h, const double dn[3], const G8State& St) {
        while (c_next < p.n_ckpt && ts >= p.t0 + c_next * p.ckpt_days) {
            if (valid) save_ckpt_g8(p, c_next, j, gl, St, ts, n_steps);
            ++c_next;
        }
        if (valid && n_steps < p.rec_fwd) write_step(rec + (size_t)n_steps * kAdjBodies * kStepRec, gl, ts, h, dn, St);
        ++n_steps;
        double tk = next_time();
        auto pending = [&]() { return valid && St.active && kobs < K && (h > 0 ? tk <= te : tk >= te); };
        bool pend = pending();
        if (__ballot(pend) == 0ull) return;
        double D[8];
        dense_increments(T.xg, gl, comp, dn, St.F0, D);
        const double xc = vector_component(St.x0, comp), vc = vector_component(St.v0, comp);
        do {
            const double v = dense_component8(gc, wt, gl, vel, pend ? (tk - ts) / h : 0.0, h, xc, vc, D);
            if (pend) { store_obs(v); advance(); }
            tk = next_time();
            pend = pending();
        } while (__ballot(pend) != 0ull);
    };
    if (valid) save_ckpt_g8(p, 0, j, gl, S, S.t, 0);
    // (windows, if asked for, end on the fixed grid of aligned_end, so a
    // recompute that starts at a checkpoint cuts its steps where this run did)
    while (S.t < p.t_end)
        g8_integrate<NB, NGR, NJ2, DEG1, kGroup>(
            p, gc, T, M, lane, aligned_end(S.t, p.t_end, E.t_start, E.seg_days, E.inv_seg, p.window_segs), S, C, visit);
    // checkpoints no step start reached: the end state
    for (; c_next <= p.n_ckpt; ++c_next)
        if (valid) save_ckpt_g8(p, c_next, j, gl, S, p.t_end, n_steps);
    if (valid && gl == 0) p.status[j] = S.status;
}

// Sky position of every observation from its stored state (forward), one
// lane per (object, observation); failed objects get NaN, and so does an
// observation whose hop ends on the Kepler iteration cap (its light time
// is stored as NaN for k_obs_status).
__global__ __launch_bounds__(256) void k_obs_sky(const AdjParams p) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)p.n_obj * p.k_obs) return;
    const int64_t j = i / p.k_obs;
    double* out = p.sky_out + 2 * i;
    if (p.status[j] != 0) { out[0] = out[1] = __builtin_nan(""); return; }
    const SunGlobal sun{p.eph};
    const double* st = p.obs_state + 6 * i;
    double d[3], tau, ve[3], r0[3], v0[3], chi;
    if (hop(p, sun, p.t_obs[i], st, st + 3, p.obs_pos + 3 * i, d, tau, ve, r0, v0, chi)) {
        out[0] = out[1] = __builtin_nan("");
        p.obs_hop[2 * i] = p.obs_hop[2 * i + 1] = __builtin_nan("");
        return;
    }
    double ra, dec, J[6];
    radec(d, p.cos_eps, p.sin_eps, ra, dec, J);
    out[0] = ra;
    out[1] = dec;
    p.obs_hop[2 * i] = tau;
    p.obs_hop[2 * i + 1] = chi;
}

// Objects with an observation whose hop failed (NaN light time) get
// KETE_ST_KEPLER_NOCONV, so the backward gives them a zero gradient.  A
// kernel of its own: k_obs_sky's lanes of one object read the status
// they would otherwise be writing.
__global__ void k_obs_status(const AdjParams p) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= p.n_obj || p.status[j] != 0) return;
    for (int k = 0; k < p.k_obs; ++k) {
        const double tau = p.obs_hop[2 * (j * p.k_obs + k)];
        if (!(tau == tau)) { p.status[j] = KETE_ST_KEPLER_NOCONV; return; }
    }
}

// dL/d(state) of every observation (backward), one lane per observation.
__global__ __launch_bounds__(256) void k_obs_vjp(const AdjParams p) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)p.n_obj * p.k_obs) return;
    const int64_t j = i / p.k_obs;
    double* g = p.obs_grad + 6 * i;
    if (p.status[j] != 0) { for (int c = 0; c < 6; ++c) g[c] = 0.0; return; }
    const SunGlobal sun{p.eph};
    const double* st = p.obs_state + 6 * i;
    double lX[3], lV[3];
    hop_vjp(p, sun, p.t_obs[i], st, st + 3, p.obs_pos + 3 * i, p.obs_hop[2 * i], p.obs_hop[2 * i + 1],
            p.dL_dsky[2 * i], p.dL_dsky[2 * i + 1], lX, lV);
    for (int c = 0; c < 3; ++c) { g[c] = lX[c]; g[3 + c] = lV[c]; }
}

// ---------------------------------------------------------------- backward
// Constants of the reverse sweep held by lane gl of a group.  Lane m - 1
// (m = 1..7) owns stage m: cA[n-1] = A_m(s_n), cB[n-1] = B_m(s_n) and the
// step-end weights gA = A_m(1), gB = B_m(1); lane 7 owns the step start:
// s_n^2/2 - sum_m A_m(s_n), s_n - sum_m B_m(s_n), and the same at s = 1.
struct AdjCols {
    double cA[7], cB[7], gA, gB;
};
constexpr int kAdjColDoubles = 16;
static_assert(sizeof(AdjCols) == kAdjColDoubles * sizeof(double), "AdjCols is 16 doubles");
static_assert(kAdjTabDoubles == kGroup * (kAdjColDoubles + 18), "table size");

__device__ __forceinline__ void load_adj_cols(const RadauConst& rc, int gl, AdjCols& c) {
#pragma unroll
    for (int n = 1; n <= 8; ++n) {
        double sA = 0.0, sB = 0.0, a = 0.0, b = 0.0;
#pragma unroll
        for (int m = 0; m < 7; ++m) {
            sA += rc.A[n][m];
            sB += rc.B[n][m];
            a = (gl == m) ? rc.A[n][m] : a;
            b = (gl == m) ? rc.B[n][m] : b;
        }
        if (gl == 7) { a = rc.half_s2[n] - sA; b = rc.s[n] - sB; }
        if (n < 8) { c.cA[n - 1] = a; c.cB[n - 1] = b; }
        else { c.gA = a; c.gB = b; }
    }
}

// Constant rows of the reverse sweep, for the 8 lanes of a group: the
// stage columns (AdjCols) and the dense-output rows alpha(sig) =
// sum_k dr[k] sig^(k+2) + dr[16] sig^2, beta(sig) = sum_k dr[8+k] sig^(k+1)
// + dr[17] sig of stage m = lane + 1 (lanes 0..6), and minus the sum over
// the stages for lane 7.  The first block writes the
// grouped kernels' constants, the second these.
__global__ __launch_bounds__(320) void k_adj_consts(const AdjParams p) {
    const int lane = threadIdx.x;
    if (blockIdx.x == 0) {
        if (lane < kGroupConstDoubles) p.group_const[lane] = group_const_at(p.rc, lane);
        return;
    }
    if (lane >= kGroup) return;
    const RadauConst& rc = p.rc;
    AdjCols q;
    load_adj_cols(rc, lane, q);
    double* col = p.adj_tab + lane * kAdjColDoubles;
    for (int n = 0; n < 7; ++n) { col[n] = q.cA[n]; col[7 + n] = q.cB[n]; }
    col[14] = q.gA;
    col[15] = q.gB;
    double* dr = p.adj_tab + kGroup * kAdjColDoubles + lane * 18;
    for (int k = 0; k < 8; ++k) {
        double a = 0.0, b = 0.0, sa = 0.0, sb = 0.0;
        for (int m = 0; m < 7; ++m) {
            sa += rc.Ap[m][k]; sb += rc.Bp[m][k];
            if (m == lane) { a = rc.Ap[m][k]; b = rc.Bp[m][k]; }
        }
        dr[k] = lane < 7 ? a : -sa;
        dr[8 + k] = lane < 7 ? b : -sb;
    }
    dr[16] = lane < 7 ? 0.0 : 0.5;
    dr[17] = lane < 7 ? 0.0 : 1.0;
}

// Backward: one wavefront goes through its objects' steps last to first.
// Lane m - 1 of an object holds the stage cotangent mu_m, lane 7 the step-start
// term; each forms the force Jacobians at its node (lane 7: the step start)
// from the step's record.
//   A wavefront waits on its own chain: the perturbers at the nodes, the
// Jacobians, and some eight passes of the stage equations of a step (two
// exchanges through LDS each).  With each checkpoint segment recomputed by
// one kernel into memory and swept by another, forward and backward of
// 100,000 objects x 20 observations over 60 d took 3.9 ms and of 20,000 2.6;
// from the forward's records 2.6 and 1.9.  (Objects of many steps alone in
// their wavefronts took it to 2.5 and 1.5, but the limit on a segment's steps,
// which the objects of a wavefront share, then failed others than before.)
template <int NB, int NGR, int NJ2, int DEG1>
__global__ __launch_bounds__(64, 2) void k_adj_back(const AdjParams p) {
    extern __shared__ __align__(16) double smem[];
    __shared__ __align__(16) GroupConst gc;
    __shared__ __align__(16) double srec_all[kAdjBodies * kStepRec];
    __shared__ __align__(16) double xw_all[kAdjBodies * kGroup * 6];    // exchange slots: [node lane][6] (W, U)
    __shared__ AdjCols cols[kGroup];
    __shared__ double drow[kGroup][18];             // dense-output rows
    const int lane = threadIdx.x;
    const GroupMap<kGroup> M(lane);
    const int gl = M.gl;
    const int jnode = gl < 7 ? gl + 1 : 0;          // node whose Jacobians this lane holds
    const EphemArgs& E = p.eph;
    const RadauConst& rc = p.rc;
    double* srec = srec_all + M.grp * kStepRec;
    double* xw = xw_all + M.grp * kGroup * 6;
    double* dst = &cols[0].cA[0];
    for (int i = lane; i < kAdjTabDoubles; i += kWave)
        (i < kGroup * kAdjColDoubles ? dst[i] : drow[0][i - kGroup * kAdjColDoubles]) = p.adj_tab[i];
    load_group_const(p.group_const, &gc, lane, kWave);
    const G8Lds T = g8_lds<kGroup>(E, smem, M.grp);
    g8_table_init<kGroup>(E, lane, smem);
    __syncthreads();
    const NodeRow& R = gc.row[gl];
    const AdjCols& Q = cols[gl];
    const double* dr = drow[gl];
    const size_t N = p.n_obj;
    const long first = (long)blockIdx.x * kAdjBodies, gi = first + M.grp;
    const bool valid = gi < p.n_obj;
    const int j = valid ? (p.perm ? p.perm[gi] : (int)gi) : 0;
    const int j_first = p.perm ? p.perm[first] : (int)first;
    const int K = p.k_obs;
    const double* tob = p.t_obs + (size_t)j * K;
    const bool ok_final = valid && p.status[j] == 0;
    // one step of every object of the wavefront, and this lane's slot of it
    constexpr size_t kStep = (size_t)kAdjBodies * kStepRec;
    double* rec_wave = p.rec + (size_t)blockIdx.x * (p.rec_fwd + p.s_max) * kStep;
    const int slot = M.grp * kStepRec + 4 * gl;
    double lx[3] = {0.0, 0.0, 0.0}, lv[3] = {0.0, 0.0, 0.0};
    int kb = K - 1;
    bool overflow_steps = false;

    // The reverse of one step, its record in srec.
    auto step_back = [&]() {
        // (the same in every object)
        const double ts = uniform(srec_all[4 * 6 + 3]), h = uniform(srec_all[4 * 7 + 3]);
        const double hh = h * h;
        double D[7][3], x0[3], v0[3], F0[3];
#pragma unroll
        for (int m = 0; m < 7; ++m) {
            const double2 a = *reinterpret_cast<const double2*>(srec + 4 * m);
            const double2 b = *reinterpret_cast<const double2*>(srec + 4 * m + 2);
            D[m][0] = a.x; D[m][1] = a.y; D[m][2] = b.x;
            if (m < 3) x0[m] = b.y;
            else if (m < 6) v0[m - 3] = b.y;
        }
        F0[0] = srec[28]; F0[1] = srec[29]; F0[2] = srec[30];
        node_ephemeris8<NB, NGR, DEG1>(E, gc, T, ts, h, ts + h, true, lane);
        double Jx[9], Jv[9];
        {
            // state at this lane's Jacobian node
            double X[3], V[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                double ax = R.hs2 * F0[i], av = R.s * F0[i];
#pragma unroll
                for (int m = 0; m < 7; ++m) { ax = fma(R.A[m], D[m][i], ax); av = fma(R.B[m], D[m][i], av); }
                X[i] = jnode == 0 ? x0[i] : fma(hh, ax, fma(R.s * h, v0[i], x0[i]));
                V[i] = jnode == 0 ? v0[i] : fma(h, av, v0[i]);
            }
            accel_jac8<NB, NGR>(T.e8 + jnode * T.row, E, X, V, Jx, Jv);
        }
        // output cotangents: the step end and the observations inside
        double G0[3], gx0[3], gv0[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            G0[i] = hh * Q.gA * lx[i] + h * Q.gB * lv[i];
            gx0[i] = lx[i];
            gv0[i] = h * lx[i] + lv[i];
        }
        auto pending = [&]() { return ok_final && kb >= 0 && (h > 0 ? tob[kb] > ts : tob[kb] < ts); };
        bool pend = pending();
        while (__ballot(pend) != 0ull) {
            if (pend) {
                const double sig = (tob[kb] - ts) / h;
                const double* og = p.obs_grad + ((size_t)j * K + kb) * 6;
                const double lX[3] = {og[0], og[1], og[2]}, lV[3] = {og[3], og[4], og[5]};
                // this lane's dense-output weights at sig
                double a = dr[7], b = dr[15];
#pragma unroll
                for (int k = 6; k >= 0; --k) { a = fma(a, sig, dr[k]); b = fma(b, sig, dr[8 + k]); }
                a = (a + dr[16]) * sig * sig;
                b = (b + dr[17]) * sig;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    G0[i] += hh * a * lX[i] + h * b * lV[i];
                    gx0[i] += lX[i];
                    gv0[i] += sig * h * lX[i] + lV[i];
                }
                --kb;
            }
            pend = pending();
        }
        // stage cotangents: mu_m = G_m + sum_n [h^2 A_m(s_n) Jx_n^T mu_n + h B_m(s_n) Jv_n^T mu_n],
        // lane m - 1 holding mu_m; lane 7 accumulates the step-start term m0
        double mu[3] = {G0[0], G0[1], G0[2]};
        double wsum[3], usum[3], m0[3] = {0.0, 0.0, 0.0};
        double pc = 1e300, pcl;
        int it = 0;
        do {
            pcl = pc;
            ++it;
            double W[3] = {0.0, 0.0, 0.0}, U[3] = {0.0, 0.0, 0.0};
            if (gl < 7) {
#pragma unroll
                for (int c2 = 0; c2 < 3; ++c2) {
                    double a = 0.0, b = 0.0;
#pragma unroll
                    for (int r = 0; r < 3; ++r) { a = fma(Jx[3 * r + c2], mu[r], a); b = fma(Jv[3 * r + c2], mu[r], b); }
                    W[c2] = a; U[c2] = b;
                }
            }
            *reinterpret_cast<double2*>(xw + 6 * gl) = make_double2(W[0], W[1]);
            *reinterpret_cast<double2*>(xw + 6 * gl + 2) = make_double2(W[2], U[0]);
            *reinterpret_cast<double2*>(xw + 6 * gl + 4) = make_double2(U[1], U[2]);
            wave_lds_sync();
            double nm[3] = {G0[0], G0[1], G0[2]};
#pragma unroll
            for (int i = 0; i < 3; ++i) { wsum[i] = 0.0; usum[i] = 0.0; }
#pragma unroll
            for (int n = 1; n <= 7; ++n) {
                const double* x = xw + 6 * (n - 1);
                const double2 w01 = *reinterpret_cast<const double2*>(x);
                const double2 w2u0 = *reinterpret_cast<const double2*>(x + 2);
                const double2 u12 = *reinterpret_cast<const double2*>(x + 4);
                const double wn[3] = {w01.x, w01.y, w2u0.x}, un[3] = {w2u0.y, u12.x, u12.y};
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    nm[i] += hh * Q.cA[n - 1] * wn[i] + h * Q.cB[n - 1] * un[i];
                    wsum[i] += wn[i];
                    usum[i] += rc.s[n] * h * wn[i] + un[i];
                }
            }
            wave_lds_sync();
            double dm = 0.0, mm = 0.0;
            if (gl < 7) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    dm = fmax(dm, fabs(nm[i] - mu[i]));
                    mm = fmax(mm, fabs(nm[i]));
                    mu[i] = nm[i];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i) m0[i] = nm[i];
            }
#pragma unroll
            for (int off = 1; off < kGroup; off <<= 1) {
                dm = fmax(dm, __shfl_xor(dm, off, kWave));
                mm = fmax(mm, __shfl_xor(mm, off, kWave));
            }
            // the ratio only steers the stopping rule: the reciprocal estimate suffices
            pc = groups_max((ok_final && mm > 0.0) ? dm * __builtin_amdgcn_rcp(mm) : 0.0);
        } while (!(pc < 1e-16) && !(it > 2 && pcl <= pc) && it < 2 * p.max_iter);
        // step-start Jacobians (lane 7) applied to m0, shared with the group
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            double a = 0.0, b = 0.0;
#pragma unroll
            for (int r = 0; r < 3; ++r) { a = fma(Jx[3 * r + i], m0[r], a); b = fma(Jv[3 * r + i], m0[r], b); }
            lx[i] = gx0[i] + wsum[i] + __shfl(a, 7, kGroup);
            lv[i] = gv0[i] + usum[i] + __shfl(b, 7, kGroup);
        }
    };
    // steps [a, b) of the records at `rec`, last first; the next one is read during a step
    auto sweep = [&](const double* rec, int a, int b) {
        const double* r = rec + slot;
        double2 q0 = make_double2(0.0, 0.0), q1 = q0;
        auto read = [&](int st) {
            if (!valid || st < a) return;
            const double2* s = reinterpret_cast<const double2*>(r + (size_t)st * kStep);
            q0 = s[0];
            q1 = s[1];
        };
        read(b - 1);
        for (int st = b - 1; st >= a; --st) {
            wave_lds_sync();                        // the previous record is read
            *reinterpret_cast<double2*>(srec + 4 * gl) = q0;
            *reinterpret_cast<double2*>(srec + 4 * gl + 2) = q1;
            wave_lds_sync();
            read(st - 1);
            step_back();
        }
    };
    auto ckpt = [&](int c, int obj) { return p.ckpt + ((size_t)c * N + obj) * kCkptDoubles; };

    for (int c = p.n_ckpt - 1; c >= 0; --c) {
        // the segment's steps, and the times of its checkpoint and the next
        // (the same for every object of the wavefront)
        const double *cf = ckpt(c, j_first), *cn = ckpt(c + 1, j_first);
        const int a = (int)uniform(cf[35]), b = (int)uniform(cn[35]);
        if (b <= a) continue;
        const int ns = min(b - a, p.s_max);
        overflow_steps = overflow_steps || b - a > p.s_max;
        if (b <= p.rec_fwd) {
            sweep(rec_wave, b - ns, b);
            continue;
        }
        // The forward's steps (and windows) again from the checkpoint on,
        // until the step start where it took the next one.
        const double t_c = uniform(cf[34]), t_stop = uniform(cn[34]);
        G8State S;
        init_lane_state(p, false, j, S);
        double hw = 0.0, hprev = -kInf;
        bool have_f0 = false;
        if (valid) {
            const double* ck = ckpt(c, j);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                S.x0[i] = ck[i]; S.v0[i] = ck[3 + i]; S.F0[i] = ck[8 + i];
                S.Dp[i] = gl < 7 ? ck[12 + 3 * gl + i] : 0.0;
            }
            hw = ck[6];
            S.active = ck[7] == 0.0;
            have_f0 = ck[11] != 0.0;
            hprev = ck[33];
        }
        S.hw = groups_max(valid ? hw : 0.0);     // the same value in every valid group
        S.hprev = groups_max(hprev);             // likewise (invalid groups give -inf)
        S.haveF0 = __ballot(have_f0) != 0ull;       // as in the forward at this checkpoint
        S.t = t_c;
        G8Count Cn;
        int n = 0;
        double* seg = rec_wave + (size_t)p.rec_fwd * kStep;
        auto store = [&](double ts, double, double h, const double dn[3], const G8State& St) {
            if (valid && n < ns) write_step(seg + (size_t)n * kStep + M.grp * kStepRec, gl, ts, h, dn, St);
            ++n;
        };
        while (S.t < t_stop)
            g8_integrate<NB, NGR, NJ2, DEG1, kGroup>(
                p, gc, T, M, lane, aligned_end(S.t, p.t_end, E.t_start, E.seg_days, E.inv_seg, p.window_segs), S, Cn,
                store, t_stop);
        sweep(seg, 0, min(n, ns));
    }
    // observations at the start epoch
    if (ok_final) {
        while (kb >= 0) {
            const double* og = p.obs_grad + ((size_t)j * K + kb) * 6;
#pragma unroll
            for (int i = 0; i < 3; ++i) { lx[i] += og[i]; lv[i] += og[3 + i]; }
            --kb;
        }
    }
    if (valid) {
        const bool good = ok_final && !overflow_steps;
        if (gl < 6) p.grad[6 * (size_t)j + gl] = good ? state_component(lx, lv, gl) : 0.0;
        if (gl == 0 && overflow_steps && ok_final) p.status[j] = KETE_ST_MAX_STEPS;
    }
}

}  // namespace

static hipError_t launch_adjoint_waves(const AdjParams& p, int mode, hipStream_t s) {
    const dim3 grid((unsigned)adj_waves(p.n_obj));
    const size_t lds = (size_t)g8_wave_doubles<kGroup>(p.eph) * sizeof(double);
    const int shape = group_shape(p.eph);
    if (mode == KETE_ADJ_FWD) {
        switch (shape) {
            case 2: hipLaunchKernelGGL((k_adjoint_fwd<10, 3, 2, 13>), grid, dim3(64), lds, s, p); break;
            case 3: hipLaunchKernelGGL((k_adjoint_fwd<3, 2, 2, 13>), grid, dim3(64), lds, s, p); break;
            case 1: hipLaunchKernelGGL((k_adjoint_fwd<0, 0, 0, 13>), grid, dim3(64), lds, s, p); break;
            default: hipLaunchKernelGGL((k_adjoint_fwd<0, 0, 0, 0>), grid, dim3(64), lds, s, p); break;
        }
    } else {
        switch (shape) {
            case 2: hipLaunchKernelGGL((k_adj_back<10, 3, 2, 13>), grid, dim3(64), lds, s, p); break;
            case 3: hipLaunchKernelGGL((k_adj_back<3, 2, 2, 13>), grid, dim3(64), lds, s, p); break;
            case 1: hipLaunchKernelGGL((k_adj_back<0, 0, 0, 13>), grid, dim3(64), lds, s, p); break;
            default: hipLaunchKernelGGL((k_adj_back<0, 0, 0, 0>), grid, dim3(64), lds, s, p); break;
        }
    }
    return hipGetLastError();
}

hipError_t launch_adjoint(const AdjParams& p, int mode, hipStream_t s) {
    if (p.n_obj <= 0) return hipSuccess;
    const int64_t n_o = (int64_t)p.n_obj * p.k_obs;
    const unsigned go = (unsigned)((n_o + 255) / 256);
    hipError_t e;
    if (mode == KETE_ADJ_FWD) {
        static_assert(kGroupConstDoubles <= 320, "one thread per constant");
        hipLaunchKernelGGL(k_adj_consts, dim3(2), dim3(320), 0, s, p);
        if ((e = launch_adjoint_waves(p, mode, s)) != hipSuccess) return e;
        if (n_o > 0) {
            hipLaunchKernelGGL(k_obs_sky, dim3(go), dim3(256), 0, s, p);
            hipLaunchKernelGGL(k_obs_status, dim3((unsigned)((p.n_obj + 255) / 256)), dim3(256), 0, s, p);
        }
        return hipGetLastError();
    }
    if (n_o > 0) hipLaunchKernelGGL(k_obs_vjp, dim3(go), dim3(256), 0, s, p);
    return launch_adjoint_waves(p, mode, s);
}


}  // namespace kete
