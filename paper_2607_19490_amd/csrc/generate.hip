// Generator kernels: synthetic fp32 references (stand-in for the verifier's
// offline pass of Eq. 1), per-block scales, and the simulated live pass of
// Eqs. 2-3 (benign hardware noise, tampering, fp16 hand-off).
//
// Every random number comes from Philox4x32-10 evaluated in registers from
// its counter, so noise and tamper directions never touch HBM: a thread
// reads 8 fp32 references (two 16-byte loads) and writes 8 fp16 activations
// (one 16-byte store).  All fp32 arithmetic is written one operation per
// step with FMA contraction off, so results are reproducible bit for bit.
#include <math.h>
#include <string.h>

#include <vector>

#include "cdt_device.hpp"
#include "cdt_launch.hpp"
#include "cdt_sim.hpp"

#pragma clang fp contract(off)

namespace cdt {
namespace {

constexpr uint32_t kMaxOutlierH = 32768;

// ---------------------------------------------------------------------------
// Outlier channels: one workgroup draws all H channel words into LDS, finds
// the n_out-th smallest by four 8-bit digits (a histogram of the words that
// share the digits found so far, scanned by one wave), and writes every gain.
// Words equal to it count in channel order.  9 us at H = 4096, where ranking
// every channel against all others took 118 us.
// ---------------------------------------------------------------------------
constexpr int kOutlierThreads = 1024;
__global__ __launch_bounds__(kOutlierThreads) void outlier_gain_kernel(uint32_t H, uint32_t n_out,
                                                                      float big, Key key,
                                                                      uint32_t tag,
                                                                      float* __restrict__ gain) {
    __shared__ uint32_t words[kMaxOutlierH];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t found[2];
    const BlockDraw bd = block_draw(key, 0, 0);
    for (uint32_t j = threadIdx.x; j < H; j += kOutlierThreads)
        words[j] = finish_draw(bd, draw_base(bd, j), tag ^ key.k1).x;
    uint32_t digits = 0, mask = 0, rank = n_out;  // the rank-th smallest (from 1) is sought
    for (int shift = 24; n_out > 0 && shift >= 0; shift -= 8) {  // uniform
        if (threadIdx.x < 256) hist[threadIdx.x] = 0;
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < H; j += kOutlierThreads) {
            const uint32_t w = words[j];
            if ((w & mask) == digits) atomicAdd(&hist[(w >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (threadIdx.x < kWave) {  // four bins per lane
            uint32_t bin[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                bin[k] = hist[4 * threadIdx.x + k];
                sum += bin[k];
            }
            uint32_t upto = sum;
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t left = __shfl_up(upto, off, kWave);
                upto += static_cast<int>(threadIdx.x) >= off ? left : 0u;
            }
            uint32_t below = upto - sum;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (below < rank && rank <= below + bin[k]) {
                    found[0] = 4 * threadIdx.x + k;
                    found[1] = rank - below;
                }
                below += bin[k];
            }
        }
        __syncthreads();
        digits |= found[0] << shift;
        mask |= 255u << shift;
        rank = found[1];
    }
    // `rank` of the words equal to `digits` are outliers; all, unless words tie
    const bool all_equal = n_out > 0 && hist[digits & 255u] == rank;
    for (uint32_t j = threadIdx.x; j < H; j += kOutlierThreads) {
        const uint32_t w = words[j];
        bool out = n_out > 0 && w < digits;
        if (n_out > 0 && w == digits) {
            uint32_t before = 0;
            if (!all_equal)
                for (uint32_t i = 0; i < j; ++i) before += words[i] == digits;
            out = before < rank;
        }
        gain[j] = out ? big : 1.0f;
    }
}

// ---------------------------------------------------------------------------
// Streamed loads and stores of the elementwise kernels (each byte is touched
// once per launch).  The output is stored nontemporally: it leaves no
// dirty lines behind in L2 / the Infinity Cache for the next kernel to evict.
// ---------------------------------------------------------------------------
template <typename P>
__device__ __forceinline__ f32x4 load_stream(P p) { return *p; }
template <typename P, typename V>
__device__ __forceinline__ void store_stream(P p, V v) {
    __builtin_nontemporal_store(v, p);
}

// ---------------------------------------------------------------------------
// Chunk walk shared by the elementwise kernels: chunk -> (block, first group).
// ---------------------------------------------------------------------------
struct ChunkPos {
    uint64_t block;
    uint32_t s, c;
    uint32_t g0;  // first 8-element group of this chunk inside the block
};

__device__ __forceinline__ ChunkPos chunk_pos(uint64_t chunk, uint64_t chunks_per_block,
                                              uint32_t C, uint32_t chunk_groups) {
    ChunkPos p;
    p.block = chunk / chunks_per_block;
    p.g0 = static_cast<uint32_t>(chunk - p.block * chunks_per_block) * chunk_groups;
    p.s = static_cast<uint32_t>(p.block / C);
    p.c = static_cast<uint32_t>(p.block - static_cast<uint64_t>(p.s) * C);
    return p;
}

// ---------------------------------------------------------------------------
// Synthetic references: ref = fp32(z_REF * gain[j]).  A wave's 64 groups of 8
// elements are 128 quads of 4; lane L makes quads L and 64 + L, so that each
// store instruction covers one contiguous 1 KB run, and a quad's channel moves
// by a constant from round to round.  Together with ref_stats on the 8 x 64 x
// 128 x 4096 shape (nontemporal stores move the write-back of dirty lines from
// its reads to these writes): 367 us, 380 us with ordinary stores; 16 x 64 x
// 256 x 8192 2.88 ms (3.00 ms with whole groups per lane and a division per
// group).  kLines: every block starts on a 64-byte boundary.  Where one does
// not, the runs end inside lines, and nontemporal stores write those in parts:
// 10 x 75 x 97 x 1288 98 us with them, 82 us with ordinary stores, 16 x 64 x 255
// x 8200 2.16 against 1.76 ms; at 64 bytes (10 x 75 x 97 x 1296) 79.8 against
// 81.6 us.  The chunks of a block are even: 12 x 100 x 48 x 768 39.0 us, 41.0 us
// with two of eight rounds and one of two; 16 x 64 x 33 x 1048 30.3 against 33.1
// us.
// ---------------------------------------------------------------------------
__device__ __forceinline__ f32x4 synth_quad(const BlockDraw& bd, uint32_t tag_key, uint32_t quad,
                                            const f32x4& g) {
    const Words4 u = finish_draw(bd, draw_base(bd, 2 * quad), tag_key);
    const Words4 v = finish_draw(bd, draw_base(bd, 2 * quad + 1), tag_key);
    return f32x4{irwin_hall4(u.x, u.y) * g.x, irwin_hall4(u.z, u.w) * g.y,
                 irwin_hall4(v.x, v.y) * g.z, irwin_hall4(v.z, v.w) * g.w};
}

constexpr int kSynthThreads = 256, kSynthItems = 8;
constexpr uint32_t kSynthChunkGroups = kSynthThreads * kSynthItems;
template <bool kLines, typename P, typename V>
__device__ __forceinline__ void store_synth(P p, V v) {
    if constexpr (kLines)
        store_stream(p, v);
    else
        *p = v;
}

template <bool kLines>
__global__ __launch_bounds__(kSynthThreads) void ref_synth_kernel(
    uint32_t C, uint32_t canary_base, uint32_t H, uint32_t n8, uint64_t chunks_per_block,
    uint32_t chunk_groups, uint64_t total_chunks, Key key, uint32_t tag,
    const float* __restrict__ gain, float* __restrict__ ref) {
    const uint64_t n = static_cast<uint64_t>(n8) * 8;
    const uint32_t h4 = H / 4, step = 2 * kSynthThreads % h4;  // quads of a row, of a round
    const uint32_t lane = threadIdx.x % kWave, wave0 = threadIdx.x - lane;
    const f32x4* gq = reinterpret_cast<const f32x4*>(gain);
    for (uint64_t it = blockIdx.x; it < total_chunks; it += gridDim.x) {
        const ChunkPos p = chunk_pos(xcd_contiguous(it, total_chunks), chunks_per_block, C,
                                     chunk_groups);
        f32x4* out = reinterpret_cast<f32x4*>(ref + p.block * n);
        const BlockDraw bd = block_draw(key, canary_base + p.c, p.s);
        const uint32_t n4 = 2 * n8, q_end = min(2 * (p.g0 + chunk_groups), n4);
        uint32_t q0 = 2 * (p.g0 + wave0) + lane;
        uint32_t j0 = q0 % h4, j1 = (q0 + kWave) % h4;
#pragma unroll 1
        for (; q0 < q_end; q0 += 2 * kSynthThreads) {
            const uint32_t q1 = q0 + kWave;
            store_synth<kLines>(out + q0, synth_quad(bd, tag ^ key.k1, q0, gq[j0]));
            if (q1 < q_end)
                store_synth<kLines>(out + q1, synth_quad(bd, tag ^ key.k1, q1, gq[j1]));
            j0 += step;
            j0 -= j0 >= h4 ? h4 : 0u;
            j1 += step;
            j1 -= j1 >= h4 ? h4 : 0u;
        }
    }
}

// ---------------------------------------------------------------------------
// Per-block scales (fp64, rounded once to fp32).
// ---------------------------------------------------------------------------
__global__ void block_scales_kernel(uint64_t nblocks, double n, const double* __restrict__ sumsq,
                                    const double* __restrict__ sumabs, double eps, double sigma_b,
                                    float* __restrict__ tscale, float* __restrict__ bscale) {
    const uint64_t b = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (b >= nblocks) return;
    if (tscale) {
        const double rms = n > 0 ? sqrt(sumsq[b] / n) : 0.0;
        tscale[b] = static_cast<float>(eps * rms);
    }
    if (bscale) {
        const double mu = n > 0 ? sumabs[b] / n : 0.0;
        bscale[b] = static_cast<float>(sigma_b * mu);
    }
}

// ---------------------------------------------------------------------------
// Live pass (Eqs. 2-3) -> fp16.
// ---------------------------------------------------------------------------
// Specialised on the two launch-uniform noise modes so that the common
// (Gaussian, elementwise) path carries no Student-t or block-scale code, and
// on the threads per workgroup (GenShape).
//
// kStream: the same chunks, loads, prefetch and stores with the live pass
// replaced by h = fp16(a) (no random numbers): the memory bound of the live
// pass's access pattern, against which the live pass is judged.
template <bool kT3, bool kBlock, bool kStream, int kThreads>
__device__ __forceinline__ void sim_chunk(const SimArgs& A, uint64_t chunk,
                                          const float* __restrict__ ref,
                                          uint16_t* __restrict__ h) {
    const uint64_t n = static_cast<uint64_t>(A.n8) * 8;
    const ChunkPos p = chunk_pos(chunk, A.chunks_per_block, A.C, A.chunk_groups);
    const SimBlock B = sim_block<kBlock>(A, p.block, p.s, p.c);
    const gptr<const f32x4> in = global_ptr(reinterpret_cast<const f32x4*>(ref + p.block * n));
    const gptr<u32x4> out = global_ptr(reinterpret_cast<u32x4*>(h + p.block * n));
    const uint32_t g_end = min(p.g0 + A.chunk_groups, A.n8);
    // Double buffer: the next group's reference loads are issued before
    // the Philox work on the current group, so loads overlap the ALU work.
    uint32_t g = p.g0 + threadIdx.x;
    f32x4 nxt_lo = f32x4{0.f, 0.f, 0.f, 0.f}, nxt_hi = nxt_lo;
    if (g < g_end) {
        nxt_lo = load_stream(in + 2 * g);
        nxt_hi = load_stream(in + 2 * g + 1);
    }
#pragma unroll 1
    while (g < g_end) {
        const f32x4 a_lo = nxt_lo, a_hi = nxt_hi;
        const uint32_t g_next = g + kThreads;
        if (g_next < g_end) {
            nxt_lo = load_stream(in + 2 * g_next);
            nxt_hi = load_stream(in + 2 * g_next + 1);
        }
        if constexpr (kStream) {
            const float a[8] = {a_lo.x, a_lo.y, a_lo.z, a_lo.w, a_hi.x, a_hi.y, a_hi.z, a_hi.w};
            store_stream(out + g, pack_half8(a));
        } else {
            store_stream(out + g, sim_group8<kT3, kBlock>(A, B, g * 8, a_lo, a_hi));
        }
        g = g_next;
    }
}

// Chunks go round the XCDs one by one (see canary_sim_batch_kernel; with five
// shards, one of them under all three tampers, 1.42 ms against 1.69 ms for a
// 5 x 64 x 256 x 8192 run and its Eq. 4).  Over the largest arrays each XCD is
// better off in one place (walks_shard_eighths), with kEighths in its own
// instantiation: the index arithmetic takes eight more VGPRs.
template <bool kT3, bool kBlock, bool kStream, int kThreads, bool kEighths>
__global__ __launch_bounds__(kThreads) void canary_sim_kernel(
    SimArgs A, const float* __restrict__ ref, uint16_t* __restrict__ h) {
    for (uint64_t it = blockIdx.x; it < A.total_chunks; it += gridDim.x) {
        uint64_t chunk = it;
        if constexpr (kEighths)
            chunk = shard_eighths(it, A.total_chunks, A.chunks_per_block * A.C);
        sim_chunk<kT3, kBlock, kStream, kThreads>(A, chunk, ref, h);
    }
}

// One chunk of a unit of kJ Gaussian runs over one reference, in a block that
// none of them tampers with: each group of 8 references is loaded once, and the
// part of its Philox calls that no run enters (normal_base: 2 of the 18
// multiplies of a call) is formed once for all of them.  The runs share one
// seed and canary range (group_batch_jobs).  What every group of a run needs
// is held in scalar registers from the chunk's start (read from the table per
// group, 24 runs of 16 x 32 x 64 x 4096 take 6.0 ms against 3.3 ms).
template <bool kBlock, int kJ>
__device__ __forceinline__ void benign_chunk_jobs(const SimJobDev* __restrict__ unit,
                                                  const ChunkPos& p) {
    const SimArgs& A0 = unit[0].A;
    const uint64_t n = static_cast<uint64_t>(A0.n8) * 8;
    const uint32_t g_end = min(p.g0 + A0.chunk_groups, A0.n8);
    const gptr<const f32x4> in =
        global_ptr(reinterpret_cast<const f32x4*>(unit[0].ref + p.block * n));
    const BlockDraw bd = block_draw(A0.key, A0.canary_base + p.c, p.s);
    BenignRun run[kJ];
    gptr<u32x4> out[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
        run[j] = benign_run<kBlock>(unit[j].A, p.block);
        out[j] = global_ptr(reinterpret_cast<u32x4*>(unit[j].h + p.block * n));
    }
    uint32_t g = p.g0 + threadIdx.x;
    f32x4 nxt_lo = f32x4{0.f, 0.f, 0.f, 0.f}, nxt_hi = nxt_lo;
    if (g < g_end) {
        nxt_lo = load_stream(in + 2 * g);
        nxt_hi = load_stream(in + 2 * g + 1);
    }
#pragma unroll 1
    while (g < g_end) {
        const f32x4 a_lo = nxt_lo, a_hi = nxt_hi;
        const uint32_t g_next = g + kGenThreadsSmall;
        if (g_next < g_end) {
            nxt_lo = load_stream(in + 2 * g_next);
            nxt_hi = load_stream(in + 2 * g_next + 1);
        }
        const float a[8] = {a_lo.x, a_lo.y, a_lo.z, a_lo.w, a_hi.x, a_hi.y, a_hi.z, a_hi.w};
        const NormalBase nb = normal_base(bd, g * 8);
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
            float v[8];
            benign8<false, kBlock>(run[j], bd, nb, g * 8, a, a, v);
            store_stream(out[j] + g, pack_half8(v));
            __builtin_amdgcn_sched_barrier(0);  // one run's temporaries at a time
        }
        g = g_next;
    }
}

// One chunk of a unit of runs over one reference, the runs one after another
// within each group of 8 elements: one body for every run count, with the
// tampering of the runs that tamper.  What a run needs comes from the table each
// time.
//
// Student-t: a group of a run is about 1000 instructions; unrolled over four
// runs that was 62 KB of code, which the compiler unrolled by two only and kept
// the runs' values in LDS.  12 KB, no LDS, 106 VGPRs (the runs share the first
// rounds of all their draws but the flips'; 74 VGPRs, sharing those of the
// one-normal streams alone, are up to 2% slower at large shapes).  Four runs
// with one malicious shard, against the unrolled form: 4 x 32 x 16 x 512 21.7
// against 35.1 us, 12 x 100 x 48 x 768 484 against 493 us, 16 x 64 x 128 x 8192
// 10.9 against 11.5 ms.
//
// Gaussian, where a run of the unit tampers with the block, against run by run
// over the chunk: four runs with every shard malicious, 8 x 32 x 32 x 512 31.3
// against 34.9 us, 16 x 64 x 128 x 8192 6.38 against 6.87 ms; with one shard in
// eight 18.8 against 18.9 us.  A unit of one run is better off with sim_chunk,
// which keeps its values in registers (24 runs of 16 x 32 x 64 x 4096 that share
// no unit 2.56 against 2.67 ms).
template <bool kT3, bool kBlock>
__device__ __forceinline__ void sim_chunk_jobs(const SimJobDev* __restrict__ unit,
                                               uint32_t unit_jobs, const ChunkPos& p) {
    const SimArgs& A0 = unit[0].A;
    const uint64_t n = static_cast<uint64_t>(A0.n8) * 8;
    const uint32_t g_end = min(p.g0 + A0.chunk_groups, A0.n8);
    const gptr<const f32x4> in =
        global_ptr(reinterpret_cast<const f32x4*>(unit[0].ref + p.block * n));
    const BlockDraw bd = block_draw(A0.key, A0.canary_base + p.c, p.s);
    uint32_t g = p.g0 + threadIdx.x;
    f32x4 nxt_lo = f32x4{0.f, 0.f, 0.f, 0.f}, nxt_hi = nxt_lo;
    if (g < g_end) {
        nxt_lo = load_stream(in + 2 * g);
        nxt_hi = load_stream(in + 2 * g + 1);
    }
#pragma unroll 1
    while (g < g_end) {
        const f32x4 a_lo = nxt_lo, a_hi = nxt_hi;
        const uint32_t g_next = g + kGenThreadsSmall;
        if (g_next < g_end) {
            nxt_lo = load_stream(in + 2 * g_next);
            nxt_hi = load_stream(in + 2 * g_next + 1);
        }
        const float a[8] = {a_lo.x, a_lo.y, a_lo.z, a_lo.w, a_hi.x, a_hi.y, a_hi.z, a_hi.w};
        const NormalBase nb = normal_base(bd, g * 8);
#pragma unroll 1
        for (uint32_t j = 0; j < unit_jobs; ++j) {
            const SimArgs& A = unit[j].A;
            SimBlock B;
            B.s = p.s;
            B.c = A.canary_base + p.c;
            B.mal = (A.mal_mask >> p.s) & 1u;
            B.benign = benign_run<kBlock>(A, p.block);
            B.tsc = (B.mal && (A.tamper & 1u)) ? A.tscale[p.block] : 0.0f;
            B.draw = bd;
            float v[8];
            benign8<kT3, kBlock>(B.benign, bd, nb, g * 8, a, a, v);
            uint32_t e0 = g * 8;
            asm volatile("" : "+v"(e0));  // the flip draws are formed here, not kept for all runs
            if (B.mal) tamper8<true>(A, B, nb, e0, a, v);
            store_stream(global_ptr(reinterpret_cast<u32x4*>(unit[j].h + p.block * n)) + g,
                         pack_half8(v));
        }
        g = g_next;
    }
}

// Batched live pass: the jobs' chunks form one iteration range walked by
// one grid, group by group (batch_iter).  An iteration is one chunk of a unit
// of the group's runs: Gaussian ones together where none of them tampers with
// the block (benign_chunk_jobs), else run by run within a group of elements
// (sim_chunk_jobs), each exactly as the single-run launch generates it.  The
// units of a larger group are walked chunk-major, so its later units find the
// chunk in L2.  A malicious block costs up to 2.5 times a benign one, so the
// chunks go round the XCDs one by one: with a contiguous eighth per XCD, the
// XCD that holds the malicious shard of 16 finishes last (three 16 x 128 x 256
// x 8192 runs with their scales and Eq. 4: 16.0 ms against 18.1 ms; 18.5 ms
// with the runs generated apart, 19.3 ms at 18 multiplies a call).  24 runs of
// 16 x 32 x 64 x 4096 so take 3.3 ms (3.75 ms).
template <bool kT3, bool kBlock>
__global__ __launch_bounds__(kGenThreadsSmall) void canary_sim_batch_kernel(
    const SimJobDev* __restrict__ jobs, const BatchGroupDev* __restrict__ groups,
    uint32_t n_groups, uint64_t total_iters) {
    for (uint64_t it = blockIdx.x; it < total_iters; it += gridDim.x) {
        uint32_t first, unit_jobs;
        uint64_t chunk;
        if (!batch_iter<false>(groups, n_groups, it, &first, &unit_jobs, &chunk)) continue;
        const SimJobDev* __restrict__ unit = jobs + first;
        const SimArgs& A0 = unit[0].A;
        const ChunkPos p = chunk_pos(chunk, A0.chunks_per_block, A0.C, A0.chunk_groups);
        if constexpr (kT3) {
            sim_chunk_jobs<kT3, kBlock>(unit, unit_jobs, p);
        } else {
            bool together = true;
            for (uint32_t j = 0; j < unit_jobs; ++j)
                together = together && !((unit[j].A.mal_mask >> p.s) & 1u);
            static_assert(kSimJobsPerIter <= 4, "one case per unit size");
            if (unit_jobs == 1) {
                sim_chunk<kT3, kBlock, false, kGenThreadsSmall>(unit[0].A, chunk, unit[0].ref,
                                                                unit[0].h);
            } else if (!together) {
                sim_chunk_jobs<kT3, kBlock>(unit, unit_jobs, p);
            } else if (unit_jobs == 4) {
                benign_chunk_jobs<kBlock, 4>(unit, p);
            } else if (unit_jobs == 3) {
                benign_chunk_jobs<kBlock, 3>(unit, p);
            } else {
                benign_chunk_jobs<kBlock, 2>(unit, p);
            }
        }
    }
}

// Propagation model: a thread walks one group of 8 elements of one canary
// through all S stages in order, carrying the live error in registers; a
// workgroup chunk covers groups of one canary, so the per-stage block state is
// workgroup-uniform (and formed from s and c: found from the block index, its
// division cost a seventh of a stage's instructions; 8 x 128 x 16 x 4096 58 us,
// 62 us with it).  Same bytes as the live pass (4 B read, 2 B written per
// element); nothing is re-read.  Loading the next stage's reference before the
// current one is generated costs more registers than it hides (8 x 64 x 128 x
// 4096 with its scales and Eq. 4: 740 against 729 us).
template <bool kT3, bool kBlock, int kThreads>
__global__ __launch_bounds__(kThreads) void canary_chain_kernel(SimArgs A, uint32_t S, float gain,
                                                                const float* __restrict__ ref,
                                                                uint16_t* __restrict__ h) {
    const uint64_t n = static_cast<uint64_t>(A.n8) * 8;
    const uint64_t stage4 = static_cast<uint64_t>(A.C) * n / 4;  // 4-element quads of a stage
    for (uint64_t it = blockIdx.x; it < A.total_chunks; it += gridDim.x) {
        const uint64_t chunk = xcd_contiguous(it, A.total_chunks);
        const uint32_t c = static_cast<uint32_t>(chunk / A.chunks_per_block);
        const uint32_t g0 =
            static_cast<uint32_t>(chunk - static_cast<uint64_t>(c) * A.chunks_per_block) *
            A.chunk_groups;
        const uint32_t g_end = min(g0 + A.chunk_groups, A.n8);
#pragma unroll 1
        for (uint32_t g = g0 + threadIdx.x; g < g_end; g += kThreads) {
            float d[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            const f32x4* in = reinterpret_cast<const f32x4*>(ref + c * n) + 2 * g;
            u32x4* out = reinterpret_cast<u32x4*>(h + c * n) + g;
#pragma unroll 1
            for (uint32_t s = 0; s < S; ++s) {
                const f32x4 a_lo = load_stream(in), a_hi = load_stream(in + 1);
                in += stage4;
                const SimBlock B = sim_block<kBlock>(A, static_cast<uint64_t>(s) * A.C + c, s, c);
                store_stream(out,
                             chain_group8<kT3, kBlock>(A, B, g * 8, s == 0, gain, a_lo, a_hi, d));
                out += stage4 / 2;
            }
        }
    }
}

// 1024-thread chunks of up to kGenItems groups per thread, cut evenly (16 x 40 x
// 2048-element blocks of a 64-canary run, 10 rounds: 83 us, 105 us as 8 and 2).
inline GenShape gen_shape_large(uint64_t n8) {
    GenShape g;
    g.threads = kGenThreads;
    const uint64_t cpb = evenest_cut((n8 + kGenThreads - 1) / kGenThreads,
                                     (n8 + kGenChunkGroups - 1) / kGenChunkGroups);
    const uint64_t per = (n8 + cpb - 1) / cpb;
    g.chunk_groups =
        static_cast<uint32_t>((per + kGenThreads - 1) / kGenThreads * kGenThreads);
    g.cpb = (n8 + g.chunk_groups - 1) / g.chunk_groups;
    return g;
}

// The single-run Gaussian pass is half bound by its mixed read and write
// stream, which longer chunks serve better once the array is large, and fills
// the chip worse below that (8 x 16 x 47 x 1032: 57 against 54 us).  256 against
// 1024 threads, live pass alone:
//   without tampering  2^22 groups in blocks of 8192  32.7  31.6 us
//                      2^22.4 in blocks of 4608       43.9  41.8 us
//                      2^22 in blocks of 512          34.0  50.4 us
//                      2^26 in blocks of 131072       592   571 us
//                      2^25 in blocks of 4096         293   301 us
//   one shard of 8 under all three tampers, whose chunks cost up to 2.5 times
//   the others'        2^22 in blocks of 8192         35.3  44.5 us
//                      2^23 in blocks of 16384        69.5  72.2 us
//                      2^24 in blocks of 16384        155   157 us
//                      2^26 in blocks of 131072       629   621 us
// The Student-t pass and the batched passes are bound by their arithmetic and
// take 256 threads at every size (four Student-t runs of the 8 x 64 x 128 x 4096
// shape: 3.25 against 3.51 ms).
inline GenShape gen_shape_single(uint64_t n8, uint64_t nblocks, bool t3, bool tampers) {
    const uint64_t all = n8 * nblocks, large = 1ull << 24;
    if (t3 || all < (tampers ? large : large / 4) || n8 < kGenChunkGroups / (all < large ? 2 : 1))
        return gen_shape(n8, all);
    return gen_shape_large(n8);
}

// Above 2^28 groups (8 GiB of references) the single-run pass takes the chunks
// in each shard's eighths, one to an XCD: 16 x 256 x 256 x 8192 9.7 ms benign and
// 9.8 ms with a shard under all three tampers, 9.9 and 10.1 ms with the chunks
// round the XCDs (the XCDs' one eighth of the array each, which leaves the
// malicious shard to two of them: 9.6 and 10.9 ms).  Below, the chunks round the
// XCDs are as good or better: 16 x 64 x 128 x 4096 577 against 591 us.
inline bool walks_shard_eighths(uint64_t all_groups) { return all_groups > (1ull << 28); }

// The propagation pass has C canaries of n8 groups (S stages each) to spread:
// 256 threads until that fills 1024-thread chunks well, and where blocks are no
// whole number of them (live pass alone, 256 against 1024 threads: 8 x 128 x 128
// x 1024 188 against 163 us, 16 x 64 x 64 x 4096 346 against 329 us; 8 x 64 x 257
// x 1024 179 against 186 us, 32 x 256 x 65 x 2048 1.35 against 1.60 ms).
// The Student-t variant needs more than the 128 registers that 1024 threads leave.
inline GenShape gen_shape_chain(uint64_t n8, uint64_t C, bool t3) {
    if (t3 || n8 % kGenChunkGroups || n8 * C < (1ull << 21)) return gen_shape(n8, n8 * C);
    return gen_shape_large(n8);
}

// Grid for a chunked elementwise walk: 64 workgroups per CU; larger jobs
// loop with a stride (16384) that is a multiple of the XCD count, as
// xcd_contiguous needs.
inline uint32_t gen_grid(uint64_t total_chunks) {
    const uint64_t cap = 256ull * 64;
    return static_cast<uint32_t>(total_chunks < cap ? total_chunks : cap);
}

}  // namespace

hipError_t launch_outlier_gain(uint32_t H, uint32_t n_out, float big, uint64_t seed,
                               uint32_t ref_set_id, float* gain, hipStream_t st) {
    if (H == 0) return hipSuccess;
    hipLaunchKernelGGL(outlier_gain_kernel, dim3(1), dim3(kOutlierThreads), 0, st, H, n_out, big,
                       Key{static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32)},
                       stream_tag(kStreamOutlier, ref_set_id), gain);
    return hipGetLastError();
}

hipError_t launch_ref_synth(uint32_t S, uint32_t C, uint32_t T, uint32_t H, uint64_t seed,
                            uint32_t ref_set_id, uint32_t canary_base, const float* gain,
                            float* ref, hipStream_t st) {
    const uint64_t n = static_cast<uint64_t>(T) * H;
    const uint64_t nblocks = static_cast<uint64_t>(S) * C;
    if (n == 0 || nblocks == 0) return hipSuccess;
    const uint32_t n8 = static_cast<uint32_t>(n / 8);
    const uint64_t cpb = (n8 + kSynthChunkGroups - 1) / kSynthChunkGroups;
    const uint64_t total = cpb * nblocks;
    const uint32_t chunk_groups = static_cast<uint32_t>(
        ((n8 + cpb - 1) / cpb + kSynthThreads - 1) / kSynthThreads * kSynthThreads);
    const Key key{static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32)};
    const dim3 grid(gen_grid(total)), block(kSynthThreads);
    const uint32_t tag = stream_tag(kStreamRef, ref_set_id);
    if (n8 % 2 == 0 && reinterpret_cast<uintptr_t>(ref) % 64 == 0)
        hipLaunchKernelGGL(ref_synth_kernel<true>, grid, block, 0, st, C, canary_base, H, n8, cpb,
                           chunk_groups, total, key, tag, gain, ref);
    else
        hipLaunchKernelGGL(ref_synth_kernel<false>, grid, block, 0, st, C, canary_base, H, n8,
                           cpb, chunk_groups, total, key, tag, gain, ref);
    return hipGetLastError();
}

hipError_t launch_block_scales(uint64_t nblocks, uint32_t T, uint32_t H, const double* sumsq,
                               const double* sumabs, double eps, double sigma_b, float* tscale,
                               float* bscale, hipStream_t st) {
    if (nblocks == 0) return hipSuccess;
    const uint64_t grid = (nblocks + 255) / 256;
    hipLaunchKernelGGL(block_scales_kernel, dim3(static_cast<uint32_t>(grid)), dim3(256), 0, st,
                       nblocks, static_cast<double>(T) * static_cast<double>(H), sumsq, sumabs,
                       eps, sigma_b, tscale, bscale);
    return hipGetLastError();
}

template <bool kT3, bool kBlock>
hipError_t launch_chain_t(const SimLaunch& p, const float* ref, uint16_t* h, hipStream_t st) {
    const uint64_t n8 = static_cast<uint64_t>(p.T) * p.H / 8;
    const GenShape g = gen_shape_chain(n8, p.C, kT3);  // chunks per canary
    const SimArgs A = make_sim_args(p, g.chunk_groups, g.cpb, g.cpb * p.C);
    const dim3 grid(gen_grid(A.total_chunks));
    if constexpr (!kT3) {
        if (g.threads == kGenThreads) {
            hipLaunchKernelGGL((canary_chain_kernel<kT3, kBlock, kGenThreads>), grid,
                               dim3(kGenThreads), 0, st, A, p.S, p.carry, ref, h);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((canary_chain_kernel<kT3, kBlock, kGenThreadsSmall>), grid,
                       dim3(kGenThreadsSmall), 0, st, A, p.S, p.carry, ref, h);
    return hipGetLastError();
}

hipError_t launch_canary_chain(const SimLaunch& p, const float* ref, uint16_t* h,
                               hipStream_t st) {
    const bool t3 = p.benign_dist == 1, block_mode = p.benign_mode == 1;
    if (t3 && block_mode) return launch_chain_t<true, true>(p, ref, h, st);
    if (t3) return launch_chain_t<true, false>(p, ref, h, st);
    if (block_mode) return launch_chain_t<false, true>(p, ref, h, st);
    return launch_chain_t<false, false>(p, ref, h, st);
}

template <bool kT3, bool kBlock, bool kStream, int kThreads, bool kEighths>
void launch_sim_k(const SimArgs& A, const float* ref, uint16_t* h, hipStream_t st) {
    hipLaunchKernelGGL((canary_sim_kernel<kT3, kBlock, kStream, kThreads, kEighths>),
                       dim3(gen_grid(A.total_chunks)), dim3(kThreads), 0, st, A, ref, h);
}

template <bool kT3, bool kBlock, bool kStream = false>
hipError_t launch_sim_t(const SimLaunch& p, const float* ref, uint16_t* h, hipStream_t st) {
    const uint64_t n8 = static_cast<uint64_t>(p.T) * p.H / 8;
    const uint64_t nblocks = static_cast<uint64_t>(p.S) * p.C;
    const uint64_t shards = p.S >= 64 ? ~0ull : (1ull << p.S) - 1;
    const GenShape g = gen_shape_single(n8, nblocks, kT3, p.tamper && (p.mal_mask & shards));
    const SimArgs A = make_sim_args(p, g.chunk_groups, g.cpb, g.cpb * nblocks);
    if constexpr (!kT3) {
        if (g.threads == kGenThreads) {
            if (walks_shard_eighths(n8 * nblocks))
                launch_sim_k<kT3, kBlock, kStream, kGenThreads, true>(A, ref, h, st);
            else
                launch_sim_k<kT3, kBlock, kStream, kGenThreads, false>(A, ref, h, st);
            return hipGetLastError();
        }
    }
    launch_sim_k<kT3, kBlock, kStream, kGenThreadsSmall, false>(A, ref, h, st);
    return hipGetLastError();
}

hipError_t launch_canary_sim(const SimLaunch& p, const float* ref, uint16_t* h, hipStream_t st) {
    const uint64_t n = static_cast<uint64_t>(p.T) * p.H;
    const uint64_t nblocks = static_cast<uint64_t>(p.S) * p.C;
    if (n == 0 || nblocks == 0) return hipSuccess;
    if (p.carry != 0.0f) return launch_canary_chain(p, ref, h, st);
    const bool t3 = p.benign_dist == 1, block_mode = p.benign_mode == 1;
    if (t3 && block_mode) return launch_sim_t<true, true>(p, ref, h, st);
    if (t3) return launch_sim_t<true, false>(p, ref, h, st);
    if (block_mode) return launch_sim_t<false, true>(p, ref, h, st);
    return launch_sim_t<false, false>(p, ref, h, st);
}

// Table layout: n_jobs SimJobDev, then (256-byte aligned) up to n_jobs
// BatchGroupDev.
size_t sim_batch_groups_offset(uint32_t n_jobs) {
    return (static_cast<size_t>(n_jobs) * sizeof(SimJobDev) + 255) & ~static_cast<size_t>(255);
}

size_t sim_batch_table_bytes(uint32_t n_jobs) {
    return sim_batch_groups_offset(n_jobs) + static_cast<size_t>(n_jobs) * sizeof(BatchGroupDev);
}

template <bool kT3, bool kBlock>
void launch_sim_batch_t(const SimJobDev* jobs, const BatchGroupDev* groups, uint32_t n_groups,
                        uint64_t total, hipStream_t st) {
    hipLaunchKernelGGL((canary_sim_batch_kernel<kT3, kBlock>), dim3(gen_grid(total)),
                       dim3(kGenThreadsSmall), 0, st, jobs, groups, n_groups, total);
}

hipError_t launch_canary_sim_batch(uint32_t n_jobs, const SimLaunch* runs,
                                   const float* const* refs, uint16_t* const* hs, void* table,
                                   hipStream_t st) {
    std::vector<SimJobDev> jobs;
    std::vector<BatchKey> keys;
    jobs.reserve(n_jobs);
    bool t3 = false, block_mode = false;
    uint64_t all_groups = 0;
    for (uint32_t j = 0; j < n_jobs; ++j)
        all_groups += static_cast<uint64_t>(runs[j].T) * runs[j].H / 8 * runs[j].S * runs[j].C;
    for (uint32_t j = 0; j < n_jobs; ++j) {
        const SimLaunch& p = runs[j];
        const uint64_t n8 = static_cast<uint64_t>(p.T) * p.H / 8;
        const uint64_t nblocks = static_cast<uint64_t>(p.S) * p.C;
        if (n8 == 0 || nblocks == 0) continue;
        t3 = p.benign_dist == 1;
        block_mode = p.benign_mode == 1;
        SimJobDev d;
        d.A = make_sim_args(p, 0, 0, 0);  // its chunks: below, from its group's units
        d.ref = refs[j];
        d.h = hs[j];
        jobs.push_back(d);
        keys.push_back(BatchKey{refs[j], 0, p.S, p.C, static_cast<uint32_t>(n8), p.seed,
                                p.canary_base});
    }
    if (jobs.empty()) return hipSuccess;
    const uint32_t n = static_cast<uint32_t>(jobs.size());
    const size_t goff = sim_batch_groups_offset(n);
    std::vector<char> staged(goff + n * sizeof(BatchGroupDev), 0);
    BatchGroupDev* groups = reinterpret_cast<BatchGroupDev*>(staged.data() + goff);
    uint32_t n_groups = 0;
    group_batch_jobs(n, keys.data(), sim_unit_runs(all_groups), groups, &n_groups);
    for (uint32_t k = 0; k < n_groups; ++k) {
        BatchGroupDev& G = groups[k];
        const BatchKey& key = keys[G.first_job];
        const GenShape g = gen_shape(key.n8, all_groups, G.jobs_per_iter);
        G.chunks = g.cpb * key.S * key.C;
        for (uint32_t j = G.first_job; j < G.first_job + G.n_jobs; ++j) {
            jobs[j].A.chunk_groups = g.chunk_groups;
            jobs[j].A.chunks_per_block = g.cpb;
            jobs[j].A.total_chunks = G.chunks;
        }
    }
    const uint64_t total = place_batch_groups(groups, n_groups);
    memcpy(staged.data(), jobs.data(), n * sizeof(SimJobDev));
    const size_t bytes = goff + n_groups * sizeof(BatchGroupDev);
    hipError_t e = hipMemcpyAsync(table, staged.data(), bytes, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return e;
    const SimJobDev* dev = static_cast<const SimJobDev*>(table);
    const BatchGroupDev* gdev =
        reinterpret_cast<const BatchGroupDev*>(static_cast<const char*>(table) + goff);
    if (t3 && block_mode)
        launch_sim_batch_t<true, true>(dev, gdev, n_groups, total, st);
    else if (t3)
        launch_sim_batch_t<true, false>(dev, gdev, n_groups, total, st);
    else if (block_mode)
        launch_sim_batch_t<false, true>(dev, gdev, n_groups, total, st);
    else
        launch_sim_batch_t<false, false>(dev, gdev, n_groups, total, st);
    return hipGetLastError();
}

hipError_t launch_canary_sim_stream(uint32_t S, uint32_t C, uint32_t T, uint32_t H,
                                    const float* ref, uint16_t* h, hipStream_t st) {
    const uint64_t n8 = static_cast<uint64_t>(T) * H / 8;
    const uint64_t nblocks = static_cast<uint64_t>(S) * C;
    if (n8 == 0 || nblocks == 0) return hipSuccess;
    SimLaunch p{};
    p.S = S;
    p.C = C;
    p.T = T;
    p.H = H;
    return launch_sim_t<false, false, true>(p, ref, h, st);
}

}  // namespace cdt
