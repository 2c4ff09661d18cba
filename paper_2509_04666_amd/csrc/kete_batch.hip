// Many independent propagation jobs of uneven size in one persistent
// launch.  A job is a set of bodies with a common start epoch and its own
// list of output epochs.  Its bodies are sorted by predicted step size
// (stable, per job) and cut into tiles of 9; the bodies of most predicted
// steps over the batch are taken out and get a wavefront each.  A grid sized
// to the device pops these, then the tiles by predicted steps, from a queue,
// one wavefront per entry.
#include <math.h>

#include "kete_batch.hpp"
#include "kete_radau.hpp"

namespace kete {
namespace {

// The time extent of each job around its start, for the predicted steps.
__global__ __launch_bounds__(64) void k_job_extent(const BatchParams p) {
    const kete_job_t job = p.jobs[blockIdx.x];
    double lo = 0.0, hi = 0.0;
    for (int64_t e = threadIdx.x; e < job.n_epoch; e += 64) {
        const double dt = p.epochs[job.epoch_off + e] - job.t0;
        lo = fmin(lo, dt);
        hi = fmax(hi, dt);
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if (threadIdx.x == 0) { p.job_ext[2 * blockIdx.x] = lo; p.job_ext[2 * blockIdx.x + 1] = hi; }
}

// Every body's bucket of predicted step, and for the bodies of many short
// steps (as in the propagation's body sort) a bin of their number, 1 .. 64 by
// powers of 2^(1/8), 0 for the others.  The bins are counted over the batch.
// One thread per body of the tiles' list.
__global__ __launch_bounds__(256) void k_job_keys(const BatchParams p) {
    __shared__ int hist[kSoloBins];
    const int tid = threadIdx.x;
    if (tid < kSoloBins) hist[tid] = 0;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + tid;
    const int64_t tile = i / KETE_BATCH_TILE;
    if (tile < p.n_tiles) {
        const int2 tj = p.tiles[tile];
        const kete_job_t job = p.jobs[tj.x];
        const int64_t k = (int64_t)tj.y * KETE_BATCH_TILE + (i - tile * KETE_BATCH_TILE);
        if (k < job.n_obj) {
            const double lo = p.job_ext[2 * tj.x], hi = p.job_ext[2 * tj.x + 1];
            const double* x = p.x0 + 6 * (job.obj_off + k);
            const double h = predicted_step(x, x + 3, p.eph.gm[0], lo, hi);
            const int nbk = p.n_buckets;
            int b = nbk - 1, bin = 0;
            if (h < kInf) {
                b = (int)floor(kBucketSub * log2(h * 64.0));
                b = b < 0 ? 0 : (b >= nbk ? nbk - 1 : b);
            }
            const double steps = h > 0.0 ? (hi - lo) / h : 0.0;
            if (steps > kSoloSteps && h < kSoloMaxStep)
                bin = 1 + (int)fmin(8.0 * log2(steps / kSoloSteps), kSoloBins - 1.0);
            p.keys[job.obj_off + k] = (uint32_t)b | (uint32_t)bin << 16;
            if (bin) atomicAdd(&hist[bin - 1], 1);
        }
    }
    __syncthreads();
    if (tid < kSoloBins && hist[tid]) atomicAdd(p.solo_hist + tid, hist[tid]);
}

// Order of each job's bodies: the lone ones first, then (stably) by step
// bucket; one block per job, two passes over its bodies' keys in chunks of
// 256.  The lone ones are the bodies of the highest solo bins, as many whole
// bins as hold kBatchSolo bodies at most over the batch; they are also put on
// the batch's list, higher bins first.
__global__ __launch_bounds__(256) void k_job_bucket(const BatchParams p) {
    __shared__ int hist[kMaxBuckets + 1], base[kMaxBuckets + 1], run[kMaxBuckets + 1], wcount[4][kMaxBuckets + 1];
    __shared__ int s_above[kSoloBins], s_bin;
    const int J = blockIdx.x;
    const kete_job_t job = p.jobs[J];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int nbk = p.n_buckets + 1;              // bucket 0: the lone bodies
    for (int b = tid; b < nbk; b += 256) { hist[b] = 0; run[b] = 0; }
    if (tid < kWave) {
        // bodies of bins above this one, and the lowest bin that is lone
        const int n = p.solo_hist[kSoloBins - 1 - lane];
        int incl = n;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int v = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += v;
        }
        s_above[kSoloBins - 1 - lane] = incl - n;
        const unsigned long long fit = __ballot(incl <= kBatchSolo);
        const int bins = fit == ~0ull ? kWave : __ffsll((long long)~fit) - 1;
        if (lane == 0) s_bin = kSoloBins - bins + 1;          // bins of 1 .. 64; 65: none
        if (J == 0 && lane == (bins ? bins - 1 : 0)) p.solo_hist[kSoloBins] = bins ? incl : 0;
    }
    __syncthreads();
    const int bin0 = s_bin;
    auto bucket_of = [&](uint32_t key) { return (int)(key >> 16) >= bin0 ? 0 : 1 + (int)(key & 0xffffu); };
    for (int64_t k = tid; k < job.n_obj; k += 256) {
        const uint32_t key = p.keys[job.obj_off + k];
        const int b = bucket_of(key);
        atomicAdd(&hist[b], 1);
        if (b == 0) {
            const int bin = (int)(key >> 16) - 1;
            const int at = s_above[bin] + atomicAdd(p.solo_hist + kSoloBins + 1 + bin, 1);
            p.solo[at] = make_int2(J, (int)k);
        }
    }
    __syncthreads();
    if (tid == 0) {
        p.job_solo[J] = hist[0];
        int acc = 0;
        for (int b = 0; b < nbk; ++b) { base[b] = acc; acc += hist[b]; }
    }
    __syncthreads();
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    constexpr int kKeyBits = 9;
    static_assert(kMaxBuckets + 1 < (1 << kKeyBits), "a bucket fits its bits");
    for (int64_t c0 = 0; c0 < job.n_obj; c0 += 256) {
        const int64_t k = c0 + tid;
        const bool in = k < job.n_obj;
        const int b = in ? bucket_of(p.keys[job.obj_off + k]) : 0;
        for (int q = lane; q < nbk; q += kWave) wcount[wid][q] = 0;
        // lanes of the wavefront with the same bucket
        unsigned long long m = __ballot(in);
#pragma unroll
        for (int i = 0; i < kKeyBits; ++i) {
            const unsigned long long v = __ballot((b >> i) & 1);
            m &= (b >> i) & 1 ? v : ~v;
        }
        const int rank = __popcll(m & lt);
        wave_lds_sync();
        if (in && rank == 0) wcount[wid][b] = __popcll(m);
        __syncthreads();
        if (in) {
            int before = run[b];
            for (int w = 0; w < wid; ++w) before += wcount[w][b];
            p.perm[job.obj_off + base[b] + before + rank] = (int32_t)k;
        }
        __syncthreads();
        for (int q = tid; q < nbk; q += 256)
            run[q] += wcount[0][q] + wcount[1][q] + wcount[2][q] + wcount[3][q];
        __syncthreads();
    }
}


// The tiles in order of their predicted steps, from the step bucket of the
// first body of each (the shortest of its job's order) and the job's extent:
// a pass that counts the bins, and one that places the tiles, whole bins in
// order and any order inside them.
template <bool kPlace>
__global__ __launch_bounds__(256) void k_tile_order(const BatchParams p) {
    __shared__ int hist[kTileBins], base[kTileBins];
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < kTileBins) hist[tid] = 0;
    __syncthreads();
    const int64_t tile = (int64_t)blockIdx.x * 256 + tid;
    int bin = -1, rank = 0;
    if (tile < p.n_tiles) {
        const int2 tj = p.tiles[tile];
        const kete_job_t job = p.jobs[tj.x];
        const int64_t k = (int64_t)tj.y * KETE_BATCH_TILE + p.job_solo[tj.x];
        if (k < job.n_obj) {
            const uint32_t key = p.keys[job.obj_off + p.perm[job.obj_off + k]];
            const float oct = (float)(key & 0xffffu) * (1.0f / kBucketSub);    // log2 of the step, in 1/64 d
            const float len = (float)(p.job_ext[2 * tj.x + 1] - p.job_ext[2 * tj.x]);
            const float steps = len * 64.0f * exp2f(-oct) + 1.0f;
            bin = kTileBins - 1 - (int)fminf(4.0f * log2f(steps), kTileBins - 1.0f);     // most steps first
            rank = atomicAdd(&hist[bin], 1);
        }
    }
    __syncthreads();
    if constexpr (!kPlace) {
        if (tid < kTileBins && hist[tid]) atomicAdd(p.tile_hist + tid, hist[tid]);
    } else {
        if (tid < kWave) {
            const int n = p.tile_hist[lane];
            int incl = n;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const int v = __shfl_up(incl, off, kWave);
                if (lane >= off) incl += v;
            }
            base[lane] = incl - n + (hist[lane] ? atomicAdd(p.tile_hist + kTileBins + lane, hist[lane]) : 0);
            if (blockIdx.x == 0 && lane == kTileBins - 1) p.tile_counter[1] = (unsigned)incl;
        }
        __syncthreads();
        if (bin >= 0) p.tile_order[base[bin] + rank] = (int32_t)tile;
    }
}
static_assert(kTileBins == kWave, "a wavefront scans the bins");

// One wavefront's bodies of a job, from place `first` of its order on (the
// one body `first` itself if lone), G lanes each (see GroupMap), through the
// job's epochs.
template <int G, int NB, int NGR, int NJ2, int DEG1>
__device__ __forceinline__ void batch_wave(const BatchParams& p, const GroupConst& K, const kete_job_t& job,
                                           int64_t first, bool lone, double* dwts, double* base) {
    const int lane = threadIdx.x;
    const GroupMap<G> M(lane);
    const int gl = M.gl;
    const EphemArgs& E = p.eph;
    const G8Lds T = g8_lds<G>(E, base, M.grp);
    g8_table_init<G>(E, lane, base);
    {
        const int64_t k = first + M.grp;
        const bool valid = k < job.n_obj;
        const int64_t local = valid ? (p.n_buckets > 1 && !lone ? p.perm[job.obj_off + k] : k) : 0;
        const int64_t gobj = job.obj_off + local;
        G8State S;
        S.status = 0;
        S.active = valid;
        for (int i = 0; i < 3; ++i) {
            S.x0[i] = valid ? p.x0[6 * gobj + i] : (i == 0 ? 1.0 : 0.0);
            S.v0[i] = valid ? p.x0[6 * gobj + 3 + i] : 0.0;
            S.F0[i] = 0.0;
        }
        double hp = kInf;
        if (valid) {
            const double r = sqrt(dot3(S.x0, S.x0));
            hp = 0.05 * sqrt(r * r * r / E.gm[0]);
        }
        S.hw = groups_min<G>(S.active ? hp : kInf);
        if (!(S.hw < kInf)) S.hw = p.h_init;
        S.hp_new = kInf;
        S.t = job.t0;
        S.haveF0 = false;
        G8Count C;
        const double* ep = p.epochs + job.epoch_off;
        auto put = [&](int e, double v, bool ok) {       // lane gl writes component gl
            if (valid && gl < 6 && M.sub == 0)
                p.x_out[job.xout_off + ((int64_t)e * job.n_obj + local) * 6 + gl] = ok ? v : __builtin_nan("");
        };
        // The epochs run away from t0 (later ones ascending, then earlier
        // ones descending).  Each run of epochs in one direction lands on
        // its last epoch; the others come off the collocation polynomial
        // of the step that spans them (unless every epoch is landed on).
        int e = 0;
        while (e < job.n_epoch) {
            if (ep[e] == S.t) {
                put(e, state_component(S.x0, S.v0, gl < 6 ? gl : 5), S.active && S.status == 0);
                ++e;
                continue;
            }
            const bool fwd = ep[e] > S.t;
            int e_end = e;
            if (!p.land_epochs)
                while (e_end + 1 < job.n_epoch && (fwd ? ep[e_end + 1] > ep[e_end] : ep[e_end + 1] < ep[e_end]))
                    ++e_end;
            const double target = ep[e_end];
            EpochCursor ec(ep, e, e_end, lane);          // wave-uniform cursor over e .. e_end - 1
            auto dense_out = [&](double ts, double te, double h, const double dn[3], const G8State& St) {
                const bool ok = St.active && St.status == 0;
                dense_epochs(K, dwts, T.xg, gl, lane, ts, te, h, dn, St.x0, St.v0, St.F0, ec,
                             [&](int k, double v) { put(k, v, ok); });
            };
            while (S.t != target) {
                const Window Wn = next_window(S.t, target, E.t_start, E.seg_days, E.inv_seg, E.n_seg, p.window_segs);
                g8_integrate<NB, NGR, NJ2, DEG1, G>(p, K, T, M, lane, Wn.t_b, S, C, dense_out);
                S.t = Wn.t_b;
            }
            // a wavefront whose objects have all failed ends its steps before their epochs
            while (ec.next < ec.end) put(ec.next++, 0.0, false);
            put(e_end, state_component(S.x0, S.v0, gl < 6 ? gl : 5), S.active && S.status == 0);
            e = e_end + 1;
        }
        if (valid && gl == 0 && M.sub == 0) p.status[gobj] = S.status;
    }
}

// One wavefront per block.  It pops the lone bodies, longest first, then
// tiles of KETE_BATCH_TILE bodies of one job's others.  A tile's bodies share
// the shortest step of any of them, so the tiles of the fast orbits of a long
// job ended the launch: of 256 uneven jobs (500,000 bodies, up to ten years)
// all but a hundred wavefronts were done in 9 ms and the last in 31.  With
// the lone bodies 12.5 ms, and with the tiles by their steps instead of their
// jobs' time spans 10.8.
template <int NB, int NGR, int NJ2, int DEG1>
__global__ __launch_bounds__(64, 2) void k_batch_g8(const BatchParams p) {
    constexpr int G = KETE_BATCH_LANES;
    static_assert(GroupMap<G>::kBodies == KETE_BATCH_TILE, "tile = bodies per wavefront");
    extern __shared__ __align__(16) double smem[];
    const int lane = threadIdx.x;
    __shared__ __align__(16) GroupConst K;
    __shared__ __align__(16) double dwts[kDenseWeights];
    load_group_const(p.group_const, &K, lane, kWave);
    __syncthreads();
    const bool sorted = p.n_buckets > 1 && !p.all_solo;
    const int n_solo = sorted ? p.solo_hist[kSoloBins] : 0;
    const int n_tiles = sorted ? (int)p.tile_counter[1] : p.n_tiles * (p.all_solo ? KETE_BATCH_TILE : 1);
    for (;;) {
        int at = 0;
        if (first_lane(lane)) at = (int)atomicAdd(p.tile_counter, 1u);
        at = __builtin_amdgcn_readfirstlane(at);
        if (at < n_solo) {
            const int2 jk = p.solo[at];
            batch_wave<kSoloLanes, NB, NGR, NJ2, DEG1>(p, K, p.jobs[jk.x], jk.y, true, dwts, smem);
            continue;
        }
        if (at - n_solo >= n_tiles) break;
        if (p.all_solo) {
            const int2 tj = p.tiles[at / KETE_BATCH_TILE];
            const kete_job_t job = p.jobs[tj.x];
            const int k = tj.y * KETE_BATCH_TILE + at % KETE_BATCH_TILE;
            if (k < job.n_obj) batch_wave<kSoloLanes, NB, NGR, NJ2, DEG1>(p, K, job, k, true, dwts, smem);
            continue;
        }
        const int2 tj = p.tiles[sorted ? p.tile_order[at - n_solo] : at];
        const kete_job_t job = p.jobs[tj.x];
        const int64_t first = (int64_t)tj.y * KETE_BATCH_TILE + (sorted ? p.job_solo[tj.x] : 0);
        batch_wave<G, NB, NGR, NJ2, DEG1>(p, K, job, first, false, dwts, smem);
    }
}

}  // namespace

size_t batch_lds_bytes(const BatchParams& p) {
    return (size_t)std::max(g8_wave_doubles<KETE_BATCH_LANES>(p.eph), g8_wave_doubles<kSoloLanes>(p.eph)) *
           sizeof(double);
}

// The grouped kernels' constants into device memory (a tiny kernel, so the
// copy is part of a captured graph too).
__global__ void k_group_const(const RadauConst rc, double* __restrict__ out) {
    const int i = threadIdx.x;
    if (i < kGroupConstDoubles) out[i] = group_const_at(rc, i);
}

hipError_t launch_group_const(const RadauConst& rc, double* out, hipStream_t s) {
    static_assert(kGroupConstDoubles <= 320, "one thread per constant");
    hipLaunchKernelGGL(k_group_const, dim3(1), dim3(320), 0, s, rc, out);
    return hipGetLastError();
}

hipError_t launch_batch(const BatchParams& p, int waves_per_cu, hipStream_t s) {
    int dev = 0, ncu = 256;
    if (hipGetDevice(&dev) == hipSuccess) hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    hipError_t e;
    if ((e = fill_zero(p.tile_counter, sizeof(unsigned int), s)) != hipSuccess) return e;
    if ((e = launch_group_const(p.rc, p.group_const, s)) != hipSuccess) return e;
    if (p.n_jobs > 0 && p.n_buckets > 1 && !p.all_solo) {
        if ((e = fill_zero(p.solo_hist, (2 * (kSoloBins + 1) + 2 * kTileBins) * sizeof(int32_t), s)) != hipSuccess) return e;
        hipLaunchKernelGGL(k_job_extent, dim3((unsigned)p.n_jobs), dim3(64), 0, s, p);
        const int64_t n = (int64_t)p.n_tiles * KETE_BATCH_TILE;
        if (n > 0) hipLaunchKernelGGL(k_job_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p);
        hipLaunchKernelGGL(k_job_bucket, dim3((unsigned)p.n_jobs), dim3(256), 0, s, p);
        const dim3 gt((unsigned)std::max(1, (p.n_tiles + 255) / 256));
        hipLaunchKernelGGL(k_tile_order<false>, gt, dim3(256), 0, s, p);
        hipLaunchKernelGGL(k_tile_order<true>, gt, dim3(256), 0, s, p);
    }
    const int items = p.all_solo ? p.n_tiles * KETE_BATCH_TILE : p.n_tiles + kBatchSolo;
    const int grid = std::max(1, std::min(ncu * waves_per_cu, items));
    const size_t lds = batch_lds_bytes(p);
    switch (group_shape(p.eph)) {
        case 2: hipLaunchKernelGGL((k_batch_g8<10, 3, 2, 13>), dim3(grid), dim3(64), lds, s, p); break;
        case 3: hipLaunchKernelGGL((k_batch_g8<3, 2, 2, 13>), dim3(grid), dim3(64), lds, s, p); break;
        case 1: hipLaunchKernelGGL((k_batch_g8<0, 0, 0, 13>), dim3(grid), dim3(64), lds, s, p); break;
        default: hipLaunchKernelGGL((k_batch_g8<0, 0, 0, 0>), dim3(grid), dim3(64), lds, s, p); break;
    }
    return hipGetLastError();
}

}  // namespace kete
