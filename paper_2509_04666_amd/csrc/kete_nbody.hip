// n-body propagation of massless bodies on gfx950 (App. A force model,
// Gauss-Radau collocation with the predictor removed, App. A.6).
//
// Two layouts share the force and the step control.  k_nbody_g8 (the
// default) spreads each object over a group of lanes, one or more per
// collocation node: 7 lanes, 9 objects a wavefront, in long lists; 14 lanes,
// 4 objects, in short ones; 56 lanes for an object that has a wavefront of its
// own; or, on request, 8 lanes, 8 objects.  k_nbody keeps one object per lane
// (64 per wavefront).  The objects of a wavefront share the time grid: the
// step size is the smallest one any of them asks for, so the perturber states
// at the node times of a step are evaluated once per wavefront and read from
// LDS.
// k_nbody stages the Chebyshev coefficients of the segments a window needs
// in LDS once per workgroup; k_nbody_g8 reads them from L2 (see
// node_ephemeris8).  Objects are sorted by predicted step size
// before a launch so that the objects of one wavefront want similar steps.
#include <math.h>

#include "kete_radau.hpp"

namespace kete {
hipError_t launch_bucket(const BucketParams& p, hipStream_t s);

namespace {


template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_nbody(const NbodyParams p) {
    extern __shared__ double smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const EphemArgs& E = p.eph;
    const RadauConst& rc = p.rc;
    const int nb = E.n_body, deg1 = E.deg1;
    const int cps = 3 * deg1;                         // doubles per segment
    const int bstride = p.max_win_segs * cps;         // doubles per body in LDS
    double* coefL = smem;
    double* ephW = smem + (size_t)nb * bstride + (size_t)wid * kNodes * nb * 6;

    const long gi = (long)blockIdx.x * BLOCK + tid;
    const bool valid = gi < p.n_obj;
    const int j = valid ? (p.perm ? p.perm[gi] : (int)gi) : 0;
    int my_status = valid && !p.first_launch ? p.status[j] : 0;
    bool active = valid && my_status == 0;

    double x0[3] = {1.0, 0.0, 0.0}, v0[3] = {0.0, 0.0, 0.0};
    double hin = kInf;
    if (valid) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            x0[i] = p.state_in[6 * (size_t)j + i];
            v0[i] = p.state_in[6 * (size_t)j + 3 + i];
        }
        hin = p.h_pref[j];
    }
    double hw = wave_min(active ? hin : kInf);
    if (!(hw < kInf)) hw = p.h_init;
    double hp_new = kInf;

    unsigned long long c_steps = 0, c_iter = 0, c_rej = 0, c_lsteps = 0, c_liter = 0, c_chain = 0;
    double t = p.win[0].t_a;
    double F0[3] = {0.0, 0.0, 0.0};
    bool haveF0 = false;

    for (int w = 0; w < p.n_win; ++w) {
        const Window W = p.win[w];
        __syncthreads();
        stage_window(E, W.seg_lo, W.seg_hi, bstride, tid, BLOCK, coefL);
        __syncthreads();
        const double tb = W.t_b;
        if (__ballot(active) == 0ull) {
            t = tb;
        }
        while (t != tb) {
            const double dir = tb > t ? 1.0 : -1.0;
            double hmag = hw;
            if (p.h_max > 0.0 && hmag > p.h_max) hmag = p.h_max;
            double h = dir * hmag;
            bool landed = false;
            if (fabs(h) >= fabs(tb - t)) { h = tb - t; landed = true; }
            if ((long)c_steps >= p.max_steps) {
                if (active) { my_status = KETE_ST_MAX_STEPS; active = false; }
                t = tb;
                break;
            }
            const double t_end = landed ? tb : t + h;
            const double hh = h * h;

            // perturbers at the 9 node times, one Clenshaw chain per lane
            node_ephemeris(coefL, bstride, E, rc, W.seg_lo, W.seg_hi, t, h, t_end, lane, ephW);
            c_chain += kNodes * nb * 3;

            if (!haveF0) { accel(ephW, E, x0, v0, F0); haveF0 = true; }

            double D[7][3], b6p[3];
            const int it = corrector(rc, E, ephW, x0, v0, F0, h, active, p.max_iter, D, b6p, c_liter);
            c_iter += it;

            // IAS15-style control on |b6| / |a| at the last node
            double fm = 0.0, bm = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) { fm = fmax(fm, fabs(D[6][c] + F0[c])); bm = fmax(bm, fabs(b6p[c])); }
            const double ebl = fm > 0.0 ? bm / fm : 0.0;
            double hl = (ebl > 0.0 && ebl < kInf) ? fabs(h) * step_factor(p.eps / ebl) : fabs(h) / p.safety;
            if (!active) hl = kInf;
            if (active && hl < p.h_min) { my_status = KETE_ST_STEP_UNDERFLOW; active = false; hl = kInf; }
            const double hn = wave_min(hl);
            if (!(hn < kInf)) { t = tb; break; }
            if (hn < p.safety * fabs(h)) {       // reject and retry from the same state
                hw = hn;
                ++c_rej;
                continue;
            }
            // accept: step end from the collocation polynomial
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                double ax = rc.half_s2[8] * F0[c], av = F0[c];
#pragma unroll
                for (int m = 0; m < 7; ++m) {
                    ax = fma(rc.A[8][m], D[m][c], ax);
                    av = fma(rc.B[8][m], D[m][c], av);
                }
                x0[c] = fma(hh, ax, fma(h, v0[c], x0[c]));
                v0[c] = fma(h, av, v0[c]);
            }
            t = t_end;
            ++c_steps;
            c_lsteps += __popcll(__ballot(active));
            if (active && !(isfinite(x0[0]) && isfinite(x0[1]) && isfinite(x0[2]) &&
                            isfinite(v0[0]) && isfinite(v0[1]) && isfinite(v0[2]))) {
                my_status = KETE_ST_NONFINITE; active = false;
            }
            accel(ephW + 8 * nb * 6, E, x0, v0, F0);
            if (landed) {
                hw = fmin(hw, hn);
            } else {
                hw = fmin(hn, fabs(h) / p.safety);
                hp_new = fmin(hp_new, fmin(hl, fabs(h) / p.safety));
            }
        }
        if (W.out >= 0 && valid) {
            double* dst = p.x_out + ((size_t)W.out * p.n_obj + j) * 6;
            const bool ok = active && my_status == 0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                dst[i] = ok ? x0[i] : __builtin_nan("");
                dst[3 + i] = ok ? v0[i] : __builtin_nan("");
            }
        }
    }
    if (valid) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (p.state) { p.state[6 * (size_t)j + i] = x0[i]; p.state[6 * (size_t)j + 3 + i] = v0[i]; }
        if (p.state && hp_new < kInf) p.h_pref[j] = hp_new;
        p.status[j] = my_status;
    }
    if (p.stats && lane == 0 && __ballot(valid) != 0ull) {
        atomicAdd(p.stats + 0, c_steps);
        atomicAdd(p.stats + 1, c_iter);
        atomicAdd(p.stats + 2, c_rej);
        atomicAdd(p.stats + 3, c_lsteps);
        atomicAdd(p.stats + 4, c_liter);
        atomicAdd(p.stats + 5, c_chain);
    }
}

// One wavefront of the grouped kernel, G lanes per object (see GroupMap): 9
// objects (or 8, 4, 1) from place `first` of the order on, each spread over a
// group whose lanes own the collocation nodes.  The objects of a wavefront
// share the time grid and the perturber table as above; each sweep evaluates
// the force at all 7 nodes of an object at once.  Output and counters are
// per object, as in k_nbody.  wt: the wavefront's dense-output weights, base:
// its other LDS.
template <int G, int NB, int NGR, int NJ2, int DEG1>
__device__ __forceinline__ void nbody_wave(const NbodyParams& p, const GroupConst& K, long first, double* wt,
                                           double* base) {
    const int lane = threadIdx.x & (kWave - 1);
    const GroupMap<G> M(lane);
    const int gl = M.gl;
    const EphemArgs& E = p.eph;
    const long gi = first + M.grp;
    const bool valid = gi < p.n_obj;
    const int j = valid ? (p.perm ? p.perm[gi] : (int)gi) : 0;
    const G8Lds T = g8_lds<G>(E, base, M.grp);
    g8_table_init<G>(E, lane, base);

    G8State S;
    S.status = valid && !p.first_launch ? p.status[j] : 0;
    S.active = valid && S.status == 0;
    S.x0[0] = 1.0; S.x0[1] = S.x0[2] = 0.0;
    S.v0[0] = S.v0[1] = S.v0[2] = 0.0;
    S.F0[0] = S.F0[1] = S.F0[2] = 0.0;
    double hin = kInf;
    if (valid) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            S.x0[i] = p.state_in[6 * (size_t)j + i];
            S.v0[i] = p.state_in[6 * (size_t)j + 3 + i];
        }
        hin = p.h_pref[j];
    }
    // Epochs e_first .. e_land - 1 come off the collocation polynomial of
    // the accepted step that spans them (the cursor is wave-uniform: the
    // wavefront's objects share every step).
    EpochCursor ec(p.t_out, p.e_first, p.e_land, lane);
    S.hw = groups_min<G>(S.active ? hin : kInf);
    if (!(S.hw < kInf)) S.hw = p.h_init;
    S.hp_new = kInf;
    S.t = p.t_begin;
    S.haveF0 = false;
    G8Count C;

    const bool writer = valid && gl < 6 && M.sub == 0;
    auto put = [&](int e, double v, bool ok) {      // node lane gl writes component gl
        if (writer) p.x_out[((size_t)e * p.n_obj + j) * 6 + gl] = ok ? v : __builtin_nan("");
    };
    while (ec.next < ec.end && ec.time() == S.t) {              // epochs at the start time
        put(ec.next, state_component(S.x0, S.v0, gl < 6 ? gl : 5), S.active && S.status == 0);
        ec.advance(1, lane);
    }
    auto dense_out = [&](double ts, double te, double h, const double dn[3], const G8State& St) {
        const bool ok = St.active && St.status == 0;
        dense_epochs(K, wt, T.xg, gl, lane, ts, te, h, dn, St.x0, St.v0, St.F0, ec,
                     [&](int e, double v) { put(e, v, ok); });
    };

    for (int w = 0; w < p.n_win; ++w) {
        // the only window of a launch comes with the arguments
        const double t_b = p.n_win == 1 ? p.t_only : p.win[w].t_b;
        const int out = p.n_win == 1 ? p.e_land : p.win[w].out;
        g8_integrate<NB, NGR, NJ2, DEG1, G>(p, K, T, M, lane, t_b, S, C, dense_out);
        if (out >= 0) put(out, state_component(S.x0, S.v0, gl < 6 ? gl : 5), S.active && S.status == 0);
    }
    // a wavefront whose objects have all failed ends its steps before their epochs
    while (ec.next < ec.end) put(ec.next++, 0.0, false);
    if (writer && p.state) p.state[6 * (size_t)j + gl] = state_component(S.x0, S.v0, gl);
    if (valid && gl == 0 && M.sub == 0) {
        if (p.state && S.hp_new < kInf) p.h_pref[j] = S.hp_new;
        p.status[j] = S.status;
    }
    const unsigned long long c_steps = C.steps, c_iter = C.iter, c_rej = C.rej, c_lsteps = C.lsteps,
                             c_liter = C.liter, c_chain = C.chain, c_vchain = C.vchain, c_lpred = C.lpred;
    if (p.stats && __ballot(valid) != 0ull && lane == 0) {
        atomicAdd(p.stats + 0, c_steps);
        atomicAdd(p.stats + 1, c_iter);
        atomicAdd(p.stats + 2, c_rej);
        atomicAdd(p.stats + 3, c_lsteps);
        atomicAdd(p.stats + 4, c_liter);
        atomicAdd(p.stats + 5, c_chain);
        atomicAdd(p.stats + 6, c_vchain);
        atomicAdd(p.stats + 7, c_lpred);
    }
}

// The launch's wavefronts: the first p.solo_waves take one object each, 56
// lanes of it, the rest G lanes per object.  With p.n_solo (device) only as
// many of the first as it says have an object, and the others begin behind
// those; without, every one does.
//   A lone object takes its own steps (the shared step of nine objects on
// fast orbits, each at another place of its own, is near the shortest any of
// them ever needs) and its sweep is short, the force of a node summed by
// eight lanes.  It uses the chip less well than nine objects a wavefront, so
// it is for launches with fewer objects than keep the chip busy, and for the
// objects whose wavefronts would end the launch (see solo_waves_for).
template <int G, int NB, int NGR, int NJ2, int DEG1>
__global__ __launch_bounds__(256, 2) void k_nbody_g8(const NbodyParams p) {
    extern __shared__ __align__(16) double smem[];
    __shared__ __align__(16) GroupConst K;
    const int wid = threadIdx.x / kWave, n_waves = blockDim.x / kWave;
    load_group_const(p.group_const, &K, threadIdx.x, (int)blockDim.x);
    __syncthreads();
    const long wave = (long)blockIdx.x * n_waves + wid;
    double* wt = smem + (size_t)wid * p.wave_doubles;
    if constexpr (G != 8) {
        const int solo = p.n_solo ? min(*p.n_solo, p.solo_waves) : p.solo_waves;
        if (wave < p.solo_waves) {
            if (wave < solo) nbody_wave<kSoloLanes, NB, NGR, NJ2, DEG1>(p, K, wave, wt, wt + kDenseWeights);
            return;
        }
        const long first = solo + (wave - p.solo_waves) * GroupMap<G>::kBodies;
        if (first < p.n_obj) nbody_wave<G, NB, NGR, NJ2, DEG1>(p, K, first, wt, wt + kDenseWeights);
    } else {
        nbody_wave<G, NB, NGR, NJ2, DEG1>(p, K, wave * GroupMap<G>::kBodies, wt, wt + kDenseWeights);
    }
}

// ---------------------------------------------------------------- buckets
__device__ __forceinline__ int bucket_digit(const BucketParams& p, long i, int& item) {
    item = p.in_perm ? p.in_perm[i] : (int)i;
    const int d = (int)((p.keys[item] >> p.shift) & 0xffffu);
    return d < p.n_buckets ? d : p.n_buckets - 1;
}

__global__ __launch_bounds__(256) void k_bucket_count(const BucketParams p) {
    __shared__ int hist[kMaxBuckets];
    const int tid = threadIdx.x;
    for (int k = tid; k < p.n_buckets; k += 256) hist[k] = 0;
    __syncthreads();
    const long i = (long)blockIdx.x * 256 + tid;
    int item;
    if (i < p.n_obj) atomicAdd(&hist[bucket_digit(p, i, item)], 1);
    __syncthreads();
    for (int k = tid; k < p.n_buckets; k += 256) p.counts[(size_t)k * gridDim.x + blockIdx.x] = hist[k];
}

// Stable scatter: the rank inside a block follows the object index.
__global__ __launch_bounds__(256) void k_bucket_scatter(const BucketParams p, const int32_t* __restrict__ offs) {
    __shared__ int wcount[4][kMaxBuckets];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const long i = (long)blockIdx.x * 256 + tid;
    const bool valid = i < p.n_obj;
    int item = 0;
    const int key = valid ? bucket_digit(p, i, item) : -1;
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int rank = 0;
    for (int k = 0; k < p.n_buckets; ++k) {
        const unsigned long long m = __ballot(key == k);
        if (key == k) rank = __popcll(m & lt);
        if (lane == 0) wcount[wid][k] = __popcll(m);
    }
    __syncthreads();
    if (valid) {
        int before = 0;
        for (int w = 0; w < wid; ++w) before += wcount[w][key];
        const int pos = offs[(size_t)key * gridDim.x + blockIdx.x] + before + rank;
        p.perm[pos] = (int32_t)item;
    }
}

// Predicted step and sort key (see BucketParams) of every body over the
// launch's time span [dt_lo, dt_hi] from its start state (taken as
// heliocentric: the Sun is within 0.01 au of the barycentre, which only
// blurs the ordering).
__global__ void k_hpref_init(const double* __restrict__ x0, double* __restrict__ h_pref, uint32_t* __restrict__ keys,
                             int n, double mu, double dt_lo, double dt_hi, int n_class, double h_ref,
                             int keep_order, double solo_steps) {
    const long j = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    double tm = 0.0;
    const double h = predicted_step(x0 + 6 * j, x0 + 6 * j + 3, mu, dt_lo, dt_hi, &tm);
    h_pref[j] = h;
    if (!keys) return;
    const double span = dt_hi - dt_lo;
    const double frac = span > 0.0 ? fmin(fmax((tm - dt_lo) / span, 0.0), 1.0) : 0.0;
    uint32_t hi, lo;
    const double steps = h > 0.0 ? span / h : 0.0;
    if (steps > solo_steps && h < kSoloMaxStep) {
        hi = 0;
        lo = (uint32_t)fmin(fmax(kCritTimeBins - 1.0 - 16.0 * log2(steps / solo_steps), 0.0), kCritTimeBins - 1.0);
    } else if (steps > kCritSteps) {
        hi = 1;
        lo = (uint32_t)fmin(frac * kCritTimeBins, kCritTimeBins - 1.0);
    } else {
        // With keep_order the bodies that cross the span in one step stay in
        // the order of their index, so that their states at the epochs inside
        // it are written next to each other (the 1,368 epochs of a day for
        // 100,000 bodies: 7.8 -> 2.8 ms).
        const bool one = keep_order && h >= span;
        const double hs = one ? span : h;
        const double c = (hs > 0.0 && hs < kInf) ? floor(kClassSub * log2(hs / h_ref)) : (double)(n_class - 3);
        hi = 2u + (uint32_t)fmin(fmax(c, 0.0), (double)(n_class - 3));
        lo = one ? 0u : (uint32_t)fmin(frac * kTimeBins, kTimeBins - 1.0);
    }
    keys[j] = hi << 16 | lo;
}

}  // namespace

// Wavefronts of one object each, for a launch of n objects of which the
// device may name the heaviest (`classes`: they are sorted by predicted step).
// Up to kSoloAll objects, two wavefronts a SIMD, all of them (63 objects over
// a month: 55 -> 43 us).  Up to kSoloSomeObj, twelve rounds of wavefronts on
// the chip, the heaviest kSoloSome: the fast orbits' wavefronts end a launch
// of few rounds (5% fast orbits: 20,000 objects for a quarter of a year 0.99 ->
// 0.84 ms, for five years 10.0 -> 6.7; 100,000 for five years 14.4 -> 12.2).
// For a year, over which sharing wavefronts lines up their perihelion passages
// (see solo_class_steps), it gains up to 50,000 objects (2.33 -> 1.79 ms) and
// costs behind (100,000 2.55 -> 2.79, 220,000 4.72 -> 5.12).  In longer lists
// it costs at either span (400,000: a year 8.3 -> 8.9 ms, five 41.5 -> 43.0).
constexpr int kSoloSome = 1024, kSoloSomeObj = 220000;
// Two lanes per node (4 objects a wavefront) up to here: at most two
// wavefronts a SIMD, whose sweeps are half as long (a quarter of a year: 3,000
// objects 0.87 -> 0.73 ms, 9,000 1.10 -> 0.74; five years with 30% fast
// orbits: 9,000 8.6 -> 7.0 ms, 3,000 6.06 either way).  Beyond it depends on
// the orbits: 16,000 objects for a year would take 1.48 -> 1.52 ms with 5% fast
// ones and 2.20 -> 1.69 with 30%.
constexpr int kPairLanesObj = 8192;
int solo_waves_for(int n, bool classes) {
    if (n <= kSoloAll) return n;
    return classes && n <= kSoloSomeObj ? kSoloSome : 0;
}

// Predicted steps from which a body is in the solo class, ordered by their
// number: kSoloSteps where the first of them get wavefronts of their own.
// Elsewhere its bodies share wavefronts, and whether to line up their numbers
// of steps or (as critical bodies, no solo class) their perihelion passages
// goes by the launch:
//   its longest wavefronts end it: the passages (eight lanes a body, 20,000
//     bodies 2.0 ms for a year and 9.0 for five, by steps 3.6 and 18.3; one
//     lane a body 30 and 123, by steps 49 and 244);
//   many rounds of wavefronts on the chip and a span of several passages: the
//     steps (400,000 bodies, seven lanes: one and a half years 12.5 ms either
//     way, two years 16.5, by passages 17.8, five 41.5 and 53.3).
constexpr double kManyPassages = 650.0;             // days
double solo_class_steps(int n, int solo_waves, int lanes_per_body, double span) {
    const bool rounds = lanes_per_body != 1 && n > kSoloSomeObj;
    return solo_waves || (rounds && span > kManyPassages) ? kSoloSteps : HUGE_VAL;
}

// The grouped kernel with G lanes per object; the usual shapes of the
// perturber table (bodies, bodies with the Eq. A.3 and A.4 terms) get an
// unrolled force.
template <int G>
static hipError_t launch_groups(NbodyParams p, int block, hipStream_t s) {
    const int wpb = block / kWave;
    const EphemArgs& E = p.eph;
    // with n_solo the objects not taken alone may be all of them
    const long rest = p.n_solo ? p.n_obj : std::max(0, p.n_obj - p.solo_waves);
    const long waves = p.solo_waves + (rest + GroupMap<G>::kBodies - 1) / GroupMap<G>::kBodies;
    const dim3 grid((unsigned)((waves + wpb - 1) / wpb));
    if (grid.x == 0) return hipSuccess;
    p.wave_doubles = kDenseWeights + (p.solo_waves ? std::max(g8_wave_doubles<G>(E), g8_wave_doubles<kSoloLanes>(E))
                                                   : g8_wave_doubles<G>(E));
    const size_t lds = (size_t)wpb * p.wave_doubles * sizeof(double);
    switch (group_shape(E)) {
        case 2: hipLaunchKernelGGL((k_nbody_g8<G, 10, 3, 2, 13>), grid, dim3(block), lds, s, p); break;
        case 3: hipLaunchKernelGGL((k_nbody_g8<G, 3, 2, 2, 13>), grid, dim3(block), lds, s, p); break;
        case 1: hipLaunchKernelGGL((k_nbody_g8<G, 0, 0, 0, 13>), grid, dim3(block), lds, s, p); break;
        default: hipLaunchKernelGGL((k_nbody_g8<G, 0, 0, 0, 0>), grid, dim3(block), lds, s, p); break;
    }
    return hipGetLastError();
}

hipError_t launch_nbody(const NbodyParams& p, int block, int lanes_per_body, hipStream_t s) {
    const size_t lds = ((size_t)p.eph.n_body * p.max_win_segs * 3 * p.eph.deg1 +
                        (size_t)(block / kWave) * kNodes * p.eph.n_body * 6) * sizeof(double);
    if (lanes_per_body == 7 || lanes_per_body == 8) {
        if (block != 64 && block != 128 && block != 256) return hipErrorInvalidValue;
        if (lanes_per_body == 8) return launch_groups<8>(p, block, s);
        return p.n_obj - p.solo_waves <= kPairLanesObj ? launch_groups<14>(p, block, s)
                                                       : launch_groups<7>(p, block, s);
    }
    if (lanes_per_body != 1) return hipErrorInvalidValue;
    const int grid = (int)((p.n_obj + block - 1) / block);
    if (grid == 0) return hipSuccess;
    switch (block) {
        case 64: hipLaunchKernelGGL(k_nbody<64>, dim3(grid), dim3(64), lds, s, p); break;
        case 128: hipLaunchKernelGGL(k_nbody<128>, dim3(grid), dim3(128), lds, s, p); break;
        case 256: hipLaunchKernelGGL(k_nbody<256>, dim3(grid), dim3(256), lds, s, p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Epochs from which bodies of one step keep their order: an epoch of 100,000
// of them costs 3.6 us less to write in order, and their wavefronts 3 us more
// where near orbits, whose corrector takes more sweeps, are not kept apart.
constexpr int kOrderEpochs = 4;
hipError_t launch_hpref_init(const double* x0, double* h_pref, uint32_t* keys, int n, double mu, double dt_lo,
                             double dt_hi, int n_class, int n_epochs, double solo_steps, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_hpref_init, dim3((n + 255) / 256), dim3(256), 0, s, x0, h_pref, keys, n, mu, dt_lo, dt_hi,
                       n_class, 1.0 / 64.0, n_epochs >= kOrderEpochs, solo_steps);
    return hipGetLastError();
}

// Bodies ordered by their keys: the time class first, then (stably) the
// step class, into perm; tmp [n] holds the first pass's order.  Afterwards
// body_sort_first gives the device address of the number of bodies in step
// class 0: the class-major offsets of the second pass, where class 1 starts.
const int32_t* body_sort_first(const int32_t* counts, int n, int n_class) {
    const int nblk = (n + 255) / 256;
    return counts + (size_t)n_class * nblk + nblk;
}
hipError_t launch_body_sort(const uint32_t* keys, int n, int n_class, int32_t* perm, int32_t* tmp, int32_t* counts,
                            hipStream_t s) {
    BucketParams B;
    B.keys = keys;
    B.counts = counts;
    B.n_obj = n;
    B.pad = 0;
    B.in_perm = nullptr;
    B.perm = tmp;
    B.n_buckets = kCritTimeBins;
    B.shift = 0;
    hipError_t e = launch_bucket(B, s);
    if (e != hipSuccess) return e;
    B.in_perm = tmp;
    B.perm = perm;
    B.n_buckets = n_class;
    B.shift = 16;
    return launch_bucket(B, s);
}

hipError_t launch_bucket(const BucketParams& p, hipStream_t s) {
    const int nblk = (p.n_obj + 255) / 256;
    if (nblk == 0) return hipSuccess;
    hipLaunchKernelGGL(k_bucket_count, dim3(nblk), dim3(256), 0, s, p);
    // offsets are written after the counts (bucket-major), total at the end
    int32_t* offs = p.counts + (size_t)p.n_buckets * nblk;
    void* scratch = offs + (size_t)p.n_buckets * nblk + 1;
    hipError_t e = exclusive_scan_i32(p.counts, offs, (int64_t)p.n_buckets * nblk, scratch, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bucket_scatter, dim3(nblk), dim3(256), 0, s, p, (const int32_t*)offs);
    return hipGetLastError();
}

size_t bucket_scratch_ints(int64_t n_obj, int n_buckets) {
    const int64_t nblk = (n_obj + 255) / 256;
    return (size_t)(2 * n_buckets * nblk + 1) + scan_scratch_bytes(n_buckets * nblk) / sizeof(int32_t) + 64;
}

}  // namespace kete
