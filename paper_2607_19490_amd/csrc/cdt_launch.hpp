// Internal launch interface between the C ABI layer and the kernel files.
// Arguments reaching these functions have been validated by the ABI layer.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "cdt_device.hpp"
#include "cdt_reduce.hpp"

namespace cdt {

// Elementwise kernels: a thread owns groups of 8 consecutive elements (one
// 16-byte fp16 vector, two 16-byte fp32 vectors); a workgroup covers up to
// kGenItems groups per thread of one block per chunk (the next group's
// reference is always loaded before the current one is generated, so only
// the first load of a chunk is exposed).  The single-run Gaussian live pass
// of a large array takes 1024 threads, everything else 256 (gen_shape).
constexpr int kGenThreads = 1024;
constexpr int kGenThreadsSmall = 256;
constexpr int kGenItems = 8;
constexpr uint32_t kGenChunkGroups = kGenThreads * kGenItems;
// Most jobs of a batch unit (BatchGroupDev), for the live pass and Eq. 4.
constexpr uint32_t kSimJobsPerIter = 4;
constexpr uint32_t kDriftJobsPerIter = 8;

struct SimLaunch {
    uint32_t S, C, T, H;
    uint64_t seed;
    uint32_t cfg_id;
    uint32_t benign_mode, benign_dist, tamper, tamper_base, redraw;
    uint64_t mal_mask;
    float sigma_b;       // fp32(sigma_b)
    uint32_t flip_thr;   // floor(p 2^32) (p < 1)
    uint32_t flip_all;   // p >= 1
    float scale;         // fp32(scale)
    float carry;         // fp32(carry): propagation gain (0: independent stages)
    uint32_t canary_base;  // global index of canary 0 (RNG counters)
    const float* bscale;
    const float* tscale;
};

struct AurocCfgDev {
    uint32_t S, C;
    uint64_t score_off;
    uint64_t pos_mask;
    uint32_t cfg_id;
    uint32_t canary_base;
};
static_assert(sizeof(AurocCfgDev) == 32, "cfg layout must match cdt_auroc_cfg");

hipError_t launch_outlier_gain(uint32_t H, uint32_t n_out, float big, uint64_t seed,
                               uint32_t ref_set_id, float* gain, hipStream_t st);
hipError_t launch_ref_synth(uint32_t S, uint32_t C, uint32_t T, uint32_t H, uint64_t seed,
                            uint32_t ref_set_id, uint32_t canary_base, const float* gain,
                            float* ref, hipStream_t st);
hipError_t launch_block_scales(uint64_t nblocks, uint32_t T, uint32_t H, const double* sumsq,
                               const double* sumabs, double eps, double sigma_b, float* tscale,
                               float* bscale, hipStream_t st);
hipError_t launch_canary_sim(const SimLaunch& p, const float* ref, uint16_t* h, hipStream_t st);

// A run of consecutive jobs of a batched launch that read one reference
// array in one layout.  An iteration is one chunk of up to `jobs_per_iter` of
// the group's jobs (a unit), and an XCD takes a chunk's units one after
// another, so that all but the first read of the reference chunk are served
// by its L2.
struct BatchGroupDev {
    uint64_t iter_begin;  // first iteration of the group (a multiple of 8)
    uint64_t chunks;      // chunks of one of its jobs
    uint32_t first_job, n_jobs;
    uint32_t units, jobs_per_iter;
};

// Iteration `it` of a grouped batch -> (first job of its unit, jobs in the
// unit, chunk); false for the padding that rounds each group's chunks up to a
// multiple of 8.  The group is found by a binary search (workgroup-uniform).
// Iteration it runs on XCD it % 8 (a grid stride that is a multiple of 8),
// and so does the group-local index, since every group starts on a multiple
// of 8.  kContiguous: each XCD walks one contiguous eighth of the chunks;
// else the chunks go round the XCDs one by one.
template <bool kContiguous>
__device__ __forceinline__ bool batch_iter(const BatchGroupDev* __restrict__ groups,
                                           uint32_t n_groups, uint64_t it, uint32_t* job,
                                           uint32_t* unit_jobs, uint64_t* chunk) {
    uint32_t lo = 0, hi = n_groups;  // last group whose first iteration <= it
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (groups[mid].iter_begin <= it) lo = mid; else hi = mid;
    }
    const BatchGroupDev& G = groups[lo];
    const uint64_t local = it - G.iter_begin;
    const uint64_t l = local / kXcds, lc = l / G.units;
    const uint64_t c = lc * kXcds + local % kXcds;
    if (c >= G.chunks) return false;
    *chunk = kContiguous ? xcd_contiguous(c, G.chunks) : c;
    const uint32_t first = static_cast<uint32_t>(l - lc * G.units) * G.jobs_per_iter;
    *job = G.first_job + first;
    *unit_jobs = G.n_jobs - first < G.jobs_per_iter ? G.n_jobs - first : G.jobs_per_iter;
    return true;
}

// What decides whether two jobs of a batch can share their reference reads:
// the same reference array in the same layout (blocks, elements per block,
// chunks), so that a chunk index means the same elements for both.
struct BatchKey {
    const void* ref;
    uint64_t chunks;
    uint32_t S, C, n8;
    uint64_t seed;         // live pass: what the random counters are keyed by
    uint32_t canary_base;
    bool operator==(const BatchKey& o) const {
        return ref == o.ref && chunks == o.chunks && S == o.S && C == o.C && n8 == o.n8;
    }
};

// Host side: the groups of a batch whose job j (jobs without chunks left
// out by the caller) has key keys[j]; consecutive jobs with equal keys form
// a group (the kernels may then read one job's reference layout for all of
// them), cut into units of up to max_jobs jobs, as even as they can be: a
// launch whose units alternate between 4 jobs and 2 keeps some CUs on the
// long ones (six runs of the 12 x 100 x 48 x 768 shape: 427 us for the live
// pass, Eq. 4 and the ranking with 4 + 2, 377 us with 3 + 3).  Jobs whose
// random counters differ in more than the tag are not put into one unit: a
// group that holds another seed or canary range than its first job's is taken
// apart, every job a unit of its own.  Fills groups[0 .. *n_groups) but for
// their iterations (place_batch_groups).
inline void group_batch_jobs(uint32_t n_jobs, const BatchKey* keys, uint32_t max_jobs,
                             BatchGroupDev* groups, uint32_t* n_groups) {
    *n_groups = 0;
    for (uint32_t j = 0; j < n_jobs; ++j) {
        if (*n_groups) {
            BatchGroupDev& last = groups[*n_groups - 1];
            const BatchKey& k = keys[last.first_job];
            if (k == keys[j]) {
                ++last.n_jobs;
                if (k.seed != keys[j].seed || k.canary_base != keys[j].canary_base)
                    last.jobs_per_iter = 1;
                continue;
            }
        }
        BatchGroupDev g;
        g.iter_begin = 0;
        g.chunks = keys[j].chunks;
        g.first_job = j;
        g.n_jobs = 1;
        g.units = 1;
        g.jobs_per_iter = max_jobs;
        groups[(*n_groups)++] = g;
    }
    for (uint32_t k = 0; k < *n_groups; ++k) {
        BatchGroupDev& g = groups[k];
        g.units = (g.n_jobs + g.jobs_per_iter - 1) / g.jobs_per_iter;
        g.jobs_per_iter = (g.n_jobs + g.units - 1) / g.units;
    }
}

// The groups' iterations one after another; returns the padded iteration count.
inline uint64_t place_batch_groups(BatchGroupDev* groups, uint32_t n_groups) {
    uint64_t total = 0;
    for (uint32_t k = 0; k < n_groups; ++k) {
        BatchGroupDev& g = groups[k];
        g.iter_begin = total;
        total += (g.chunks + kXcds - 1) / kXcds * kXcds * g.units;
    }
    return total;
}

// How a live pass's work is cut: threads per workgroup and 8-element groups
// per chunk.
struct GenShape {
    uint32_t threads, chunk_groups;
    uint64_t cpb;  // chunks per block
};

// The number of chunks from cpb on, below twice as many, that leaves the fewest
// rounds of a block's chunks idle.
inline uint64_t evenest_cut(uint64_t rounds, uint64_t cpb) {
    uint64_t best = cpb, least_idle = ~0ull;
    for (uint64_t c = cpb; c < 2 * cpb && c <= rounds; ++c) {
        const uint64_t idle = (rounds + c - 1) / c * c - rounds;
        if (idle < least_idle) {
            least_idle = idle;
            best = c;
        }
    }
    return best;
}

// 256-thread chunks of as many groups per thread (up to kGenItems) as leave
// 4096 workgroups, cut evenly within a block of n8 groups.  Fewer groups
// where the launch is small fill the chip (Student-t, 12 x 30 x 48 x 768:
// 88 us with Eq. 4 and the ranking, 102 us in 8192-group chunks).  Where a
// workgroup generates `runs` = 3 or 4 runs over its chunk, 2048 of them will do,
// and the chunks of a block are the evenest of up to twice as many: a unit of
// four 12 x 30 x 48 x 768 runs takes 46 us Gaussian and 155 us Student-t, 55
// and 181 us in the chunks of a single run (six rounds, not three); leaving 4096
// is faster there (146 us) and slower on 12 x 100 (512 against 482 us).
inline GenShape gen_shape(uint64_t n8, uint64_t all_groups, uint32_t runs = 1) {
    constexpr uint64_t kT = kGenThreadsSmall;
    uint64_t items = all_groups / (kT * (runs > 2 ? 2048u * runs : 4096u));
    items = items < 1 ? 1 : items > kGenItems ? kGenItems : items;
    uint64_t cpb = (n8 + kT * items - 1) / (kT * items);
    if (runs > 2) cpb = evenest_cut((n8 + kT - 1) / kT, cpb);
    const uint64_t per = (n8 + cpb - 1) / cpb;
    GenShape g;
    g.threads = kT;
    g.chunk_groups = static_cast<uint32_t>((per + kT - 1) / kT * kT);
    g.cpb = (n8 + g.chunk_groups - 1) / g.chunk_groups;
    return g;
}

// Most runs of a unit of a batched live pass over all_groups groups (of all
// jobs): as many as leave 1024 workgroups of one group per thread.  The runs of
// a unit share loads and the first rounds of their draws, but follow one
// another in its threads: four 4 x 8 x 16 x 256 runs (256 workgroups apart) take
// 6.8 us apart and 11.8 us together, Student-t 8.5 and 17.6 us; six of 4 x 32 x
// 16 x 512 (3072) 13.0 and 11.8 us, Student-t 24.6 and 23.7 us.
inline uint32_t sim_unit_runs(uint64_t all_groups) {
    const uint64_t fill = all_groups / (kGenThreadsSmall * 1024u);
    return fill < 1 ? 1 : fill > kSimJobsPerIter ? kSimJobsPerIter : static_cast<uint32_t>(fill);
}

// Batched live pass over runs of one noise distribution and mode, carry 0:
// the device table (sim_batch_table_bytes(n_jobs) bytes: jobs, then groups)
// is filled from `runs` on the stream, then one grid generates every run's
// chunks.
size_t sim_batch_table_bytes(uint32_t n_jobs);
hipError_t launch_canary_sim_batch(uint32_t n_jobs, const SimLaunch* runs,
                                   const float* const* refs, uint16_t* const* hs, void* table,
                                   hipStream_t st);

// The live pass's loads and stores with h = fp16(a): its memory bound.
hipError_t launch_canary_sim_stream(uint32_t S, uint32_t C, uint32_t T, uint32_t H,
                                    const float* ref, uint16_t* h, hipStream_t st);

hipError_t launch_ref_stats(uint32_t S, uint32_t C, uint32_t T, uint32_t H, const float* ref,
                            double* sumsq, double* sumabs, void* ws, hipStream_t st);
// Eq. 4 (or its cosine variant) per block: partial sums per chunk into ws,
// then the combine.
hipError_t launch_drift(DriftMetric metric, uint32_t S, uint32_t C, uint32_t T, uint32_t H,
                        const uint16_t* h, const void* ref, float* score, double* sums, void* ws,
                        hipStream_t st);

// One array of a batched Eq. 4 launch, as the kernels read it from the
// device table: its arrays, shape, chunking and place in the batch's block
// index range.
struct DriftJobDev {
    const uint16_t* h;
    const float* ref;
    float* score;
    double* sums;     // [C][S][2] or null
    double* partial;  // its per-chunk partial sums (unused with one chunk per block)
    uint64_t cpb;     // chunks per block (ReduceShape)
    uint64_t block_begin;
    uint32_t n8, S, C, chunk_groups;
};

hipError_t launch_drift_batch(const DriftJobDev* jobs_dev, uint32_t n_jobs,
                              const BatchGroupDev* groups_dev, uint32_t n_groups,
                              uint64_t total_iters, uint64_t total_blocks, hipStream_t st);

// The batched Eq. 4's reads (same iterations, chunks, loads, lane exchange
// and order) with no arithmetic; nothing is written in practice.
hipError_t launch_drift_batch_read_stream(const DriftJobDev* jobs_dev,
                                          const BatchGroupDev* groups_dev, uint32_t n_groups,
                                          uint64_t total_iters, hipStream_t st);

// drift_score's reads (same chunks, loads and order) with no arithmetic; ws
// is drift_score's workspace and may be overwritten.
hipError_t launch_drift_read_stream(uint32_t S, uint32_t C, uint32_t T, uint32_t H,
                                   const uint16_t* h, const float* ref, void* ws, hipStream_t st);

// The combine step alone, over partial sums laid out as drift_score's.
hipError_t launch_drift_combine(DriftMetric metric, const double* partial, uint64_t cpb,
                                uint64_t nblocks, uint32_t S, uint32_t C, float* score,
                                double* sums, hipStream_t st);

// Live pass and Eq. 4 in one kernel (h may be NULL: not stored).
hipError_t launch_sim_score(const SimLaunch& p, const float* ref, uint16_t* h, float* score,
                            double* num_den, void* ws, hipStream_t st);

// Per-block scale of the exact-norm Gaussian tamper (and its two norms).
hipError_t launch_tamper_scale_exact(const SimLaunch& p, const float* ref, double eps,
                                     float* tscale, double* norms, void* ws, hipStream_t st);

// The same under the propagation model (p.carry > 0): the malicious stages'
// scales in pipeline order, benign entries cleared to 0.
hipError_t launch_tamper_scale_exact_chain(const SimLaunch& p, const float* ref, double eps,
                                           float* tscale, double* norms, void* ws,
                                           hipStream_t st);

// Eqs. 5-6 over a device table of configurations; a configuration whose
// table lies outside [0, n_scores) (or, pooled, exceeds the LDS sort) gets
// counts of all ones instead of being read.
hipError_t launch_auroc(uint32_t n_cfg, const AurocCfgDev* cfgs_dev, const float* scores,
                        uint64_t n_scores, uint64_t seed, uint32_t flags, uint64_t* counts,
                        uint64_t* pooled, uint64_t* baseline, hipStream_t st);

// The same from a host table small enough to travel in the launch's arguments
// (auroc_in_args); the device table is written by the launch as well.
bool auroc_in_args(uint32_t n_cfg);
hipError_t launch_auroc_args(uint32_t n_cfg, const AurocCfgDev* cfgs, AurocCfgDev* table,
                             const float* scores, uint64_t n_scores, uint64_t seed,
                             uint32_t flags, uint64_t* counts, uint64_t* pooled,
                             uint64_t* baseline, hipStream_t st);

// Eq. 6 (strict and Mann-Whitney) from the counts of launch_auroc.
hipError_t launch_auroc_values(uint32_t n_cfg, const uint64_t* counts, const uint64_t* pooled,
                               const uint64_t* baseline, double* values, hipStream_t st);

}  // namespace cdt
