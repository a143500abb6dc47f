// Shared pieces of the block reductions (Eq. 4, its fused form with the
// live pass, the exact-norm tamper and the reference statistics): the
// chunking constants, the workgroup sum and the per-element accumulation
// of Eq. 4 and its cosine variant.  A block (shard, canary) of n = T*H
// elements is cut into even chunks of at most kReduceChunkElems (reduce_shape);
// kReduceThreads threads reduce a chunk to fp64 partial sums in a fixed order (no
// atomics), in a workgroup of their own or beside a block's other chunk; a combine
// kernel, or a workgroup that holds all of a block's chunks, adds them in
// chunk order.
#pragma once

#include <stdint.h>

#include "cdt_device.hpp"

#pragma clang fp contract(off)

namespace cdt {

// Threads per workgroup and 8-element groups in flight per thread.  On the
// 16 x 256 x 256 x 8192 stream, with the fp32 reference read in contiguous
// runs, 256 x 8 reaches 89.4-89.6% of the HBM peak against 87.3-88.1% for
// 512 x 4, 89.1-89.3% for 256 x 4 and 89.8-90.2% for 256 x 16 and 128 x 16;
// over the 216-configuration sweep's smaller blocks 256 x 8 is the fastest
// of these, and the fused live-pass-and-score kernel, which shares this
// thread-to-group mapping, runs 3-4% faster than at 512 x 4.
constexpr int kReduceThreads = 256;
constexpr int kReduceUnroll = 8;
constexpr uint64_t kReduceChunkElems = 32768;

// Most chunks of a block of n elements (what workspaces are sized for).
inline uint64_t reduce_chunks_per_block(uint64_t n) {
    return (n + kReduceChunkElems - 1) / kReduceChunkElems;
}

// How a block of n8 8-element groups is cut: into the fewest chunks of at most
// kReduceChunkElems elements, as even as whole rounds of the workgroup (one
// group per thread) allow.  It depends on the block's size alone, so that a
// canary's score is the same bits in every slice of a run.  Even chunks
// matter for blocks just above a chunk: 12 x 100 blocks of 48 x 768 elements
// are 9 + 9 rounds, and 16 + 2 left half of the workgroups nearly idle
// (kernel times: Eq. 4 44 us against 58 us, cosine 49 against 71, exact-norm
// scales 75 against 114 us).
struct ReduceShape {
    uint64_t cpb;           // chunks per block
    uint32_t chunk_groups;  // groups of a chunk
};

inline ReduceShape reduce_shape(uint64_t n8) {
    if (n8 == 0) return ReduceShape{0, 0};
    const uint64_t most = reduce_chunks_per_block(n8 * 8), per = (n8 + most - 1) / most;
    ReduceShape r;
    r.chunk_groups =
        static_cast<uint32_t>((per + kReduceThreads - 1) / kReduceThreads * kReduceThreads);
    r.cpb = (n8 + r.chunk_groups - 1) / r.chunk_groups;
    return r;
}

// Reduction variants of Eq. 4: the relative-L2 mismatch (the detector) and
// the cosine mismatch (the metric ablation), each against an fp32 reference
// or an fp16 reference (a second live pass).
enum class DriftMetric { kL2, kL2HalfRef, kCosine, kCosineHalfRef };

// Partial sums per chunk: (D, R) for the L2 metrics, (D, A, P) for cosine.
constexpr int kReduceMaxSums = 3;

namespace {

constexpr int kWavesPerGroup = kReduceThreads / kWave;

// Blocks of kReduceTeam chunks can be reduced by one workgroup of as many times
// kReduceThreads threads, which does the combine's addition too: a launch less,
// the same bits.  Eq. 4 takes it up to kTeamMostBlocks blocks (8 x 64 x 64 x 1024
// 30.7 us, 33.2 us with the combine; 12 x 100 x 48 x 768 39.6 against 41.9 us, its
// fp16 reference 27.1 against 29.0 us; 16 x 256 x 8 x 8192 230 against 235 us,
// 32 x 200 x 40 x 1024 226 against 229 us): beyond, the launch is a small part and
// workgroups that wait for their slower half cost as much (32 x 256 x 64 x 1024
// 464 against 462 us).  The exact-norm sums, which are bound by arithmetic, take
// it from kTeamLeastBlocks on (12 x 100 x 48 x 768 62 against 64 us): fewer blocks
// do not fill the CUs with workgroups twice the size (4 x 16 x 48 x 768 15.3
// against 11.5 us).
constexpr int kReduceTeam = 2;
constexpr uint64_t kTeamMostBlocks = 6400, kTeamLeastBlocks = 512;

// Sum kN per-thread values over a workgroup of kTeam chunks, kReduceThreads
// threads each: every chunk's total as block_sum forms it, then the totals
// from 0 in chunk order, as the combine kernels add them.  Thread 0 gets the
// result.
template <int kN, int kTeam>
__device__ __forceinline__ void team_sum(double (&v)[kN]) {
    __shared__ double lds[kN][kTeam * kWavesPerGroup];
#pragma unroll
    for (int k = 0; k < kN; ++k) v[k] = wave_sum(v[k]);
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kN; ++k) lds[k][wave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            double all = 0.0;
            for (int m = 0; m < kTeam; ++m) {
                double t = 0.0;
                for (int w = 0; w < kWavesPerGroup; ++w) t += lds[k][m * kWavesPerGroup + w];
                all = kTeam == 1 ? t : all + t;
            }
            v[k] = all;
        }
    }
    __syncthreads();
}

// One chunk per workgroup.
template <int kN>
__device__ __forceinline__ void block_sum(double (&v)[kN]) {
    team_sum<kN, 1>(v);
}

// Per-metric element step.  h and the reference are widened exactly to
// fp64, so d = h - a is exact and the sums carry no cancellation.
template <DriftMetric kM>
struct DriftTraits {
    static constexpr bool kHalfRef =
        kM == DriftMetric::kL2HalfRef || kM == DriftMetric::kCosineHalfRef;
    static constexpr bool kCos = kM == DriftMetric::kCosine || kM == DriftMetric::kCosineHalfRef;
    static constexpr int kSums = kCos ? 3 : 2;

    __device__ static __forceinline__ void add(double hv, double av, double (&acc)[kSums]) {
        const double d = hv - av;
        acc[0] = fma(d, d, acc[0]);      // D = sum d^2
        acc[1] = fma(av, av, acc[1]);    // R = A = sum a^2
        if constexpr (kSums == 3) acc[2] = fma(av, d, acc[2]);  // P = sum a d
    }
};

template <DriftMetric kM>
__device__ __forceinline__ void accumulate8(const u32x4& hv, const u32x4& r_half,
                                            const f32x4& a0, const f32x4& a1,
                                            double (&acc)[DriftTraits<kM>::kSums]) {
    const uint32_t hw[4] = {hv.x, hv.y, hv.z, hv.w};
    const uint32_t rw[4] = {r_half.x, r_half.y, r_half.z, r_half.w};
    const float av[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double h_lo = static_cast<double>(half_bits_to_float(hw[k] & 0xFFFFu));
        const double h_hi = static_cast<double>(half_bits_to_float(hw[k] >> 16));
        double a_lo, a_hi;
        if constexpr (DriftTraits<kM>::kHalfRef) {
            a_lo = static_cast<double>(half_bits_to_float(rw[k] & 0xFFFFu));
            a_hi = static_cast<double>(half_bits_to_float(rw[k] >> 16));
        } else {
            a_lo = static_cast<double>(av[2 * k]);
            a_hi = static_cast<double>(av[2 * k + 1]);
        }
        DriftTraits<kM>::add(h_lo, a_lo, acc);
        DriftTraits<kM>::add(h_hi, a_hi, acc);
    }
}

// One workgroup per chunk up to 2^20 chunks, then a grid-stride walk whose
// stride (2^20) is a multiple of the XCD count, as xcd_contiguous needs.
inline uint32_t reduce_grid(uint64_t total_chunks) {
    const uint64_t cap = 1ull << 20;
    return static_cast<uint32_t>(total_chunks < cap ? total_chunks : cap);
}

}  // namespace

}  // namespace cdt
