// Batched uneven propagation jobs: parameters shared by the host layer
// and the persistent kernel.
#pragma once

#include "kete_fov.hpp"
#include "kete_internal.hpp"

// lanes per body of the persistent kernel (7: 9 bodies per wavefront,
// 8: 8 bodies) and bodies per tile, one wavefront each
#define KETE_BATCH_LANES 7
#define KETE_BATCH_TILE (KETE_BATCH_LANES == 7 ? 9 : 8)

namespace kete {

struct BatchParams {
    EphemArgs eph;
    RadauConst rc;
    const kete_job_t* jobs;     // [n_jobs]
    int32_t n_jobs;
    int32_t n_tiles;
    int32_t all_solo;           // every body has a wavefront of its own (no order needed)
    int32_t pad_;
    const int2* tiles;          // [n_tiles] (job, tile of KETE_BATCH_TILE bodies), longest jobs first;
                                // taken in this order only where the bodies are not sorted (else tile_order)
    unsigned int* tile_counter;
    const double* x0;           // [bodies][6]
    const double* epochs;       // concatenated epochs of all jobs
    double* x_out;              // per-job blocks [n_epoch][n_obj][6]
    int32_t* status;            // [bodies]
    int32_t* perm;              // [bodies] job-local order of each job's bodies, its lone ones first
    uint32_t* keys;             // [bodies] step bucket | solo bin << 16 (see k_job_keys)
    double* job_ext;            // [n_jobs][2] epochs relative to the start: the earliest, the latest
    int32_t* job_solo;          // [n_jobs] lone bodies of each job
    int32_t* tile_order;        // [n_tiles] the tiles that have bodies, most predicted steps first
    int32_t* tile_hist;         // [2][kTileBins] tiles per bin, then places taken
    int2* solo;                 // [kBatchSolo] (job, body), most predicted steps first
    int32_t* solo_hist;         // [2][kSoloBins + 1] bodies per bin, then places taken; last of the first row: their total
    int32_t n_buckets;
    int32_t window_segs;        // segments between forced step ends (0: none)
    int32_t max_iter;
    int32_t max_steps;
    int32_t zero_start;         // corrector starts from zero increments (no extrapolation)
    int32_t land_epochs;        // land on every epoch (else epochs inside a step come off its polynomial)
    double* group_const;        // [kGroupConstDoubles] written by the launch
    double eps, h_min, h_max, h_init, safety;
};

// Bodies that get a wavefront of their own: all of a batch of up to kSoloAll
// (no order, no tiles), else the kBatchSolo of most steps at most (512, 1,024 or 2,048 of 500,000: 13.0,
// 12.8 and 12.8 ms).  The bins of their predicted steps go by powers of
// 2^(1/8) above kSoloSteps.
constexpr int kBatchSolo = 1024;
constexpr int kSoloBins = 64;
// Bins of a tile's predicted steps, four an octave from one step on.
constexpr int kTileBins = 64;

size_t batch_lds_bytes(const BatchParams& p);
hipError_t launch_batch(const BatchParams& p, int waves_per_cu, hipStream_t s);

}  // namespace kete
