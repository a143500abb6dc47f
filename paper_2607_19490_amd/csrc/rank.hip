// Detection AUROC (Eqs. 5-6), its Mann-Whitney form and the scrambled-label
// control of Section 4.5, batched over configurations.  All of it is bound by
// latency: a configuration holds a few thousand scores.
//
// Per-canary counts: one workgroup per configuration; a wave takes as many
// canaries at a time as fit its 64 lanes with one lane per shard (four of 16
// shards), and loads its next ones' scores before ranking the current ones.
// The scores of the smaller class (one malicious shard, as a rule) are handed
// round the canary's lanes by one shuffle each and compared with the others.
//
// Pooled Mann-Whitney: one workgroup per configuration sorts the keys of the
// smaller class with a bitonic network, and every score of the larger class
// finds its place among them by a binary search: the keys below it and, if
// the one at its place equals it, the keys that tie.  Each thread holds
// E = max(1, P2 / 1024) consecutive keys of the padded length P2 in
// registers: compare-exchange stages between keys of one thread run in
// registers, stages between threads of one wave through lane shuffles, and
// only the stages that span waves go through LDS, with one barrier each.
#include "cdt_device.hpp"
#include "cdt_launch.hpp"
#include "cdt_rank.hpp"

namespace cdt {
namespace {

constexpr int kCountThreads = 1024;
constexpr int kCountWaves = kCountThreads / kWave;
constexpr int kPoolThreads = 1024;
constexpr uint32_t kPoolMax = 16384;
constexpr uint32_t kPoolKeys = kPoolMax / 2;  // the smaller class's scores

__device__ __forceinline__ uint64_t shard_mask(uint32_t S) {
    return S >= 64 ? ~0ull : ((1ull << S) - 1ull);
}

// Lane r gets the position of the r-th bit (0-based, ascending) that is set in
// m (uniform).  Every lane of the wave must call it.  Once per wave, so that a
// canary's choice of a benign shard is one shuffle: found for each canary by a
// loop over the malicious shards, 256 canaries of 64 shards with their control
// took 114.7 us with 32 malicious, 37.8 with 8 and 17.7 with one (93.9, 33.0 and
// 17.6 us); a list in LDS needs a barrier (1000 configurations of 16 x 64 scores
// 21.8 against 20.9 us).
__device__ __forceinline__ uint32_t set_bits_by_lane(uint64_t m) {
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                     __builtin_amdgcn_mbcnt_lo(
                                                         static_cast<uint32_t>(m), 0u));
    const uint32_t to =  // the other lanes send past the last of them: a permutation
        (m >> lane) & 1u ? below : __builtin_popcountll(m) + lane - below;
    return __builtin_amdgcn_ds_permute(static_cast<int>(to << 2), static_cast<int>(lane));
}

// Random-baseline score of (canary t, shard s): 24 random bits scaled into
// [0, 1), exact in fp32.
__device__ __forceinline__ float random_score(Key key, uint32_t t, uint32_t s, uint32_t tag) {
    return static_cast<float>(draw(key, t, s, 0, tag).x >> 8) * 0x1p-24f;
}

// A configuration the kernels can score without reading outside the score
// array or the pooled sort's LDS.  The host validates every table before it
// reaches the device; this check keeps a table reused against a different
// score array from reading out of bounds.
__device__ __forceinline__ bool cfg_in_bounds(const AurocCfgDev& cfg, uint64_t n_scores) {
    const uint64_t len = static_cast<uint64_t>(cfg.S) * cfg.C;
    return cfg.S <= 64 && cfg.score_off <= n_scores && len <= n_scores - cfg.score_off;
}

constexpr unsigned long long kBadCfg = ~0ull;  // counts of a configuration out of bounds

// Where a workgroup finds its configuration: in a device table, or in the
// launch's own arguments.  cdt_auroc and cdt_auroc_canaries are given host
// tables, and a copy of a small one costs as much as the ranking itself (the
// host waits for a staged copy, the GPU for its turn in the stream): up to
// kArgCfgs configurations (1 KB of arguments) travel with the launch.  The
// pipeline of 4 x 8 x 16 x 256 takes 46.6 us a step (48.7 us with the copy), a
// Table 1 attack of 12 x 100 x 48 x 768 321 us (324 us).
struct CfgTable {
    const AurocCfgDev* cfgs;
    const uint64_t* offsets;  // per-canary counts: canaries of the configurations before
    __device__ __forceinline__ AurocCfgDev cfg(uint32_t g) const { return cfgs[g]; }
    __device__ __forceinline__ uint64_t offset(uint32_t g) const { return offsets[g]; }
    __device__ __forceinline__ void keep(uint32_t) const {}
};

constexpr uint32_t kArgCfgs = 32;
struct CfgArgs {
    AurocCfgDev cfgs[kArgCfgs];
    AurocCfgDev* table;  // also left here, as a copy would have
    __device__ __forceinline__ AurocCfgDev cfg(uint32_t g) const { return cfgs[g]; }
    __device__ __forceinline__ uint64_t offset(uint32_t g) const {
        uint64_t before = 0;
        for (uint32_t i = 0; i < g; ++i) before += cfgs[i].C;
        return before;
    }
    __device__ __forceinline__ void keep(uint32_t g) const {
        if (threadIdx.x == 0) table[g] = cfgs[g];
    }
};

// What one wave needs to rank a configuration's canaries, `per_wave` at a
// time: lane = (canary within the wave) * width + shard, width the power of
// two from S on.
struct RankCtx {
    uint64_t pos, neg;
    uint32_t n_benign, tag, tag_random, width, per_wave;
    uint32_t shard, sub;  // this lane's
    uint32_t benign;      // with control, the lane-th negative shard
    bool lane_in, lane_pos, control, include_true, random;
};

__device__ __forceinline__ RankCtx rank_ctx(const AurocCfgDev& cfg, uint32_t flags) {
    const uint32_t lane = threadIdx.x % kWave;
    const uint64_t all = shard_mask(cfg.S);
    RankCtx r;
    r.pos = cfg.pos_mask & all;
    r.neg = all & ~r.pos;
    r.width = 1;
    while (r.width < cfg.S) r.width <<= 1;
    r.per_wave = kWave / r.width;
    r.shard = lane & (r.width - 1);
    r.sub = lane / r.width;
    r.lane_in = r.shard < cfg.S;
    r.lane_pos = r.lane_in && ((r.pos >> r.shard) & 1u);
    r.control = flags & 1u;
    r.benign = r.control ? set_bits_by_lane(r.neg) : 0u;  // uniform
    r.include_true = flags & 4u;
    r.random = flags & 8u;
    r.n_benign = __builtin_popcountll(r.neg);
    r.tag = stream_tag(kStreamScramble, cfg.cfg_id);
    r.tag_random = stream_tag(kStreamRandom, cfg.cfg_id);
    return r;
}

// Wins and ties of the positive shards over the negative ones, as this
// lane's part of its canary's pairs: the smaller class's keys go round.
// counted: this lane holds a score (its shard exists and so does its canary).
__device__ __forceinline__ void pair_counts(const RankCtx& r, uint32_t k, bool counted,
                                            uint32_t& wins, uint32_t& ties) {
    const bool pos_round = __builtin_popcountll(r.pos) <= __builtin_popcountll(r.neg);
    const int base = static_cast<int>(r.sub * r.width);
    const bool mine = counted && (pos_round ? !r.lane_pos : r.lane_pos);
    for (uint64_t m = pos_round ? r.pos : r.neg; m; m &= m - 1) {
        const uint32_t kj = __shfl(k, base + __builtin_ctzll(m), kWave);
        wins += mine && (pos_round ? kj > k : k > kj);
        ties += mine && kj == k;
    }
}

// The Eq. 5 counts of this lane's canary t as the lane sees them: the
// detector's wins and ties (q = 0, 1), the scrambled-label control's chosen
// stage against this lane's (q = 2, 3) and the random baseline's (q = 4, 5);
// summed over the canary's lanes they are the canary's.  cur is this lane's
// score.  Every lane of the wave must call it; lanes past the last canary
// count nothing.
__device__ __forceinline__ void rank_canaries(const RankCtx& r, const AurocCfgDev& cfg, Key key,
                                              uint32_t t, float cur, uint32_t (&c)[6]) {
#pragma unroll
    for (int q = 0; q < 6; ++q) c[q] = 0;
    const bool counted = r.lane_in && t < cfg.C;
    const uint32_t k = order_key(cur);
    pair_counts(r, k, counted, c[0], c[1]);
    if (r.random) {
        const uint32_t kr =
            order_key(random_score(key, cfg.canary_base + t, r.shard, r.tag_random));
        pair_counts(r, kr, counted, c[4], c[5]);
    }
    if (r.control && r.n_benign > 0) {
        const uint32_t u = draw(key, cfg.canary_base + t, 0, 0, r.tag).x;
        const uint32_t js = __shfl(r.benign, static_cast<int>(u % r.n_benign), kWave);
        const uint32_t kjs = __shfl(k, static_cast<int>(r.sub * r.width + js), kWave);
        const bool against = counted && r.shard != js && (r.include_true || !r.lane_pos);
        c[2] = against && kjs > k;
        c[3] = against && kjs == k;
    }
}

// This lane's score of canary t, 0 where it has none.
__device__ __forceinline__ float lane_score(const RankCtx& r, const AurocCfgDev& cfg,
                                            const float* __restrict__ base, uint64_t t) {
    return r.lane_in && t < cfg.C ? base[t * cfg.S + r.shard] : 0.0f;
}

// Eqs. 5-6 counts of configuration cfg_index (every thread of the workgroup calls it).
__device__ __forceinline__ void counts_body(
    uint32_t cfg_index, const AurocCfgDev& cfg, const float* __restrict__ scores,
    uint64_t n_scores, Key key, uint32_t flags, unsigned long long* __restrict__ counts,
    unsigned long long* __restrict__ baseline) {
    if (!cfg_in_bounds(cfg, n_scores)) {  // uniform over the workgroup
        if (threadIdx.x == 0) {
            for (int q = 0; q < 6; ++q) counts[6ull * cfg_index + q] = kBadCfg;
            if (flags & 8u)
                for (int q = 0; q < 3; ++q) baseline[3ull * cfg_index + q] = kBadCfg;
        }
        return;
    }
    const uint32_t lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const RankCtx r = rank_ctx(cfg, flags);
    unsigned long long part[6] = {0, 0, 0, 0, 0, 0};
    const float* base = scores + cfg.score_off;
    const uint64_t step = kCountWaves * r.per_wave;
    float next = lane_score(r, cfg, base, wave * r.per_wave + r.sub);
    for (uint64_t t0 = wave * r.per_wave; t0 < cfg.C; t0 += step) {
        const float cur = next;
        next = lane_score(r, cfg, base, t0 + step + r.sub);
        uint32_t c[6];
        rank_canaries(r, cfg, key, static_cast<uint32_t>(t0 + r.sub), cur, c);
#pragma unroll
        for (int q = 0; q < 6; ++q) part[q] += c[q];
    }

    __shared__ unsigned long long lds[6][kCountWaves];
#pragma unroll
    for (int q = 0; q < 6; ++q) part[q] = wave_sum(part[q]);
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < 6; ++q) lds[q][wave] = part[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long tot[6] = {0, 0, 0, 0, 0, 0};
        for (int q = 0; q < 6; ++q)
            for (int w = 0; w < kCountWaves; ++w) tot[q] += lds[q][w];
        const unsigned long long n_pos = __builtin_popcountll(r.pos);
        unsigned long long* out = counts + 6ull * cfg_index;
        out[0] = tot[0];
        out[1] = tot[1];
        out[2] = static_cast<unsigned long long>(cfg.C) * n_pos * r.n_benign;
        unsigned long long n_ctrl = 0;
        if (r.control && r.n_benign > 0) n_ctrl = r.include_true ? cfg.S - 1 : r.n_benign - 1;
        out[3] = r.control ? tot[2] : 0;
        out[4] = r.control ? tot[3] : 0;
        out[5] = static_cast<unsigned long long>(cfg.C) * n_ctrl;
        if (r.random) {
            unsigned long long* rb = baseline + 3ull * cfg_index;
            rb[0] = tot[4];
            rb[1] = tot[5];
            rb[2] = out[2];
        }
    }
}

// Eq. 5 per canary: the same ranking as auroc_counts_kernel, each canary's
// six counts summed over its lanes and written by the first of them to
// out[(offset(g) + t) * 6 + q].  A configuration out of bounds gets
// 0xFFFFFFFF in its entries instead of being read.
template <typename Src>
__global__ __launch_bounds__(kCountThreads) void auroc_canaries_kernel(
    Src src, const float* __restrict__ scores, uint64_t n_scores, Key key, uint32_t flags,
    uint32_t* __restrict__ out) {
    const AurocCfgDev cfg = src.cfg(blockIdx.x);
    uint32_t* o = out + 6ull * src.offset(blockIdx.x);
    const uint32_t wave = threadIdx.x / kWave;
    if (!cfg_in_bounds(cfg, n_scores)) {  // uniform over the workgroup
        for (uint64_t i = threadIdx.x; i < 6ull * cfg.C; i += kCountThreads) o[i] = ~0u;
        return;
    }
    const RankCtx r = rank_ctx(cfg, flags);
    const float* base = scores + cfg.score_off;
    const uint64_t step = kCountWaves * r.per_wave;
    float next = lane_score(r, cfg, base, wave * r.per_wave + r.sub);
    for (uint64_t t0 = wave * r.per_wave; t0 < cfg.C; t0 += step) {
        const float cur = next;
        next = lane_score(r, cfg, base, t0 + step + r.sub);
        const uint64_t t = t0 + r.sub;
        uint32_t c[6];
        rank_canaries(r, cfg, key, static_cast<uint32_t>(t), cur, c);
        // a canary's counts stay below 64 * 64: two to a word
        uint32_t w[3] = {c[0] | c[1] << 16, c[2] | c[3] << 16, c[4] | c[5] << 16};
        for (uint32_t off = r.width >> 1; off > 0; off >>= 1) {
#pragma unroll
            for (int q = 0; q < 3; ++q) w[q] += __shfl_xor(w[q], static_cast<int>(off), kWave);
        }
        if (r.shard == 0 && t < cfg.C) {
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                o[6 * t + 2 * q] = w[q] & 0xFFFFu;
                o[6 * t + 2 * q + 1] = w[q] >> 16;
            }
        }
    }
}

// Ascending bitonic sort of P2 (a power of two, <= kE * kPoolThreads)
// elements, thread t holding elements t*kE .. t*kE + kE - 1 in x; v is LDS
// scratch of P2 elements.  Every thread of the workgroup must call it.
template <int kE>
__device__ __forceinline__ void bitonic_sort_regs(uint32_t (&x)[kE], uint32_t P2, uint32_t* v) {
    const uint32_t t = threadIdx.x, base = t * kE;
    for (uint32_t k = 2; k <= P2; k <<= 1) {
        uint32_t j = k >> 1;
        if (j >= kWave * kE) {  // partners in other waves: in place in LDS
#pragma unroll
            for (int r = 0; r < kE; ++r)
                if (base + r < P2) v[base + r] = x[r];
            __syncthreads();
            for (; j >= kWave * kE; j >>= 1) {
                for (uint32_t p = t; p < P2 / 2; p += kPoolThreads) {
                    const uint32_t i = 2 * p - (p & (j - 1));
                    const uint32_t l = i + j;
                    const uint32_t a = v[i], b = v[l];
                    if ((a > b) == ((i & k) == 0)) {
                        v[i] = b;
                        v[l] = a;
                    }
                }
                __syncthreads();
            }
#pragma unroll
            for (int r = 0; r < kE; ++r)
                if (base + r < P2) x[r] = v[base + r];
        }
        for (; j >= static_cast<uint32_t>(kE); j >>= 1) {  // partner lane t ^ (j / kE)
            const int m = static_cast<int>(j / kE);
            const bool keep_min = ((t & m) == 0) == ((base & k) == 0);
#pragma unroll
            for (int r = 0; r < kE; ++r) {
                const uint32_t y = __shfl_xor(x[r], m, kWave);
                x[r] = keep_min ? (x[r] < y ? x[r] : y) : (x[r] < y ? y : x[r]);
            }
        }
#pragma unroll
        for (int jj = kE / 2; jj >= 1; jj >>= 1) {  // partner in this thread
            if (static_cast<uint32_t>(jj) < k) {
#pragma unroll
                for (int r = 0; r < kE; ++r) {
                    const int rp = r ^ jj;
                    if (rp > r) {
                        const uint32_t a = x[r], b = x[rp];
                        if ((a > b) == (((base + r) & k) == 0)) {
                            x[r] = b;
                            x[rp] = a;
                        }
                    }
                }
            }
        }
    }
}

// The smaller class's n keys (its `m` shards, listed in `shards`, of every
// canary), padded to P2, sorted and left in v[0 .. P2).  The pads are the
// largest key, which a NaN score shares.
template <int kE>
__device__ void pooled_sort(const float* tab, uint32_t n, uint32_t P2, uint32_t S, uint32_t m,
                            const uint8_t* shards, uint32_t* v) {
    uint32_t x[kE];
    const uint32_t base = threadIdx.x * kE;
#pragma unroll
    for (int r = 0; r < kE; ++r) {
        const uint32_t i = base + r, t = i / m;
        x[r] = i < n ? order_key(tab[t * S + shards[i - t * m]]) : 0xFFFFFFFFu;
    }
    bitonic_sort_regs<kE>(x, P2, v);
#pragma unroll
    for (int r = 0; r < kE; ++r)
        if (base + r < P2) v[base + r] = x[r];
    __syncthreads();
}

// How many of the P2 sorted keys of v lie below each of kN keys (kOrEqual:
// or equal it), P2 a power of two.
template <int kN, bool kOrEqual>
__device__ __forceinline__ void place_keys(const uint32_t* v, uint32_t P2,
                                           const uint32_t (&key)[kN], uint32_t (&at)[kN]) {
#pragma unroll
    for (int q = 0; q < kN; ++q) at[q] = 0;
    for (uint32_t step = P2 >> 1; step > 0; step >>= 1) {
#pragma unroll
        for (int q = 0; q < kN; ++q) {
            const uint32_t x = v[at[q] + step - 1];
            at[q] += (kOrEqual ? x <= key[q] : x < key[q]) ? step : 0u;
        }
    }
#pragma unroll
    for (int q = 0; q < kN; ++q) {
        const uint32_t x = v[at[q]];
        at[q] += kOrEqual ? x <= key[q] : x < key[q];
    }
}

// Pooled Mann-Whitney counts of configuration cfg_index (every thread of the
// workgroup calls it).
__device__ __forceinline__ void pooled_body(
    uint32_t cfg_index, const AurocCfgDev& cfg, const float* __restrict__ scores,
    uint64_t n_scores, unsigned long long* __restrict__ pooled) {
    __shared__ uint32_t v[kPoolKeys];
    __shared__ uint8_t shards[kWave];
    __shared__ unsigned long long red[2][kPoolThreads / kWave];
    unsigned long long* out = pooled + 3ull * cfg_index;
    if (!cfg_in_bounds(cfg, n_scores) ||
        static_cast<uint64_t>(cfg.S) * cfg.C > kPoolMax) {  // uniform over the workgroup
        if (threadIdx.x == 0)
            for (int q = 0; q < 3; ++q) out[q] = kBadCfg;
        return;
    }
    const uint64_t pos = cfg.pos_mask & shard_mask(cfg.S);
    const uint64_t neg = shard_mask(cfg.S) & ~pos;
    const uint32_t n_pos = __builtin_popcountll(pos), n_neg = __builtin_popcountll(neg);
    const bool pos_sorted = n_pos <= n_neg;
    const uint64_t sorted = pos_sorted ? pos : neg;
    const uint32_t m = pos_sorted ? n_pos : n_neg;
    if (m == 0 || cfg.C == 0) {  // no pairs
        if (threadIdx.x < 3) out[threadIdx.x] = 0;
        return;
    }
    if (threadIdx.x < cfg.S && ((sorted >> threadIdx.x) & 1u))
        shards[__builtin_popcountll(sorted & ((1ull << threadIdx.x) - 1))] =
            static_cast<uint8_t>(threadIdx.x);
    __syncthreads();
    const float* tab = scores + cfg.score_off;
    const uint32_t n = m * cfg.C;
    uint32_t P2 = 1;
    while (P2 < n) P2 <<= 1;
    static_assert(kPoolKeys == 8 * kPoolThreads, "at most 8 keys per thread");
    switch (P2 <= kPoolThreads ? 1u : P2 / kPoolThreads) {  // uniform over the workgroup
        case 1: pooled_sort<1>(tab, n, P2, cfg.S, m, shards, v); break;
        case 2: pooled_sort<2>(tab, n, P2, cfg.S, m, shards, v); break;
        case 4: pooled_sort<4>(tab, n, P2, cfg.S, m, shards, v); break;
        default: pooled_sort<8>(tab, n, P2, cfg.S, m, shards, v); break;
    }

    // The larger class, kN scores per thread at a time so that their searches
    // overlap: keys below and keys equal.
    constexpr int kN = 4;
    const uint32_t all = cfg.S * cfg.C, stride = kPoolThreads % cfg.S;
    uint32_t s = threadIdx.x % cfg.S;
    unsigned long long below = 0, equal = 0;
    uint32_t searched = 0;
    for (uint32_t e0 = threadIdx.x; e0 < all; e0 += kN * kPoolThreads) {
        uint32_t key[kN], at[kN], upto[kN];
        bool in[kN], tie = false;
#pragma unroll
        for (int q = 0; q < kN; ++q) {
            const uint32_t e = e0 + q * kPoolThreads;
            in[q] = e < all && !((sorted >> s) & 1u);
            key[q] = in[q] ? order_key(tab[e]) : 0u;
            s += stride;
            s -= s >= cfg.S ? cfg.S : 0u;
        }
        place_keys<kN, false>(v, P2, key, at);
#pragma unroll
        for (int q = 0; q < kN; ++q) {
            upto[q] = at[q];
            tie = tie || (in[q] && at[q] < n && v[at[q]] == key[q]);
        }
        if (tie) place_keys<kN, true>(v, P2, key, upto);
#pragma unroll
        for (int q = 0; q < kN; ++q) {
            if (!in[q]) continue;
            below += at[q];
            equal += min(upto[q], n) - at[q];  // a NaN's place also counts the pads
            ++searched;
        }
    }
    // Sorted positives: a negative is beaten by the keys above it.
    unsigned long long wins =
        pos_sorted ? static_cast<unsigned long long>(searched) * n - below - equal : below;
    wins = wave_sum(wins);
    equal = wave_sum(equal);
    const uint32_t lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    if (lane == 0) {
        red[0][wave] = wins;
        red[1][wave] = equal;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long G = 0, E = 0;
        for (int w = 0; w < kPoolThreads / kWave; ++w) {
            G += red[0][w];
            E += red[1][w];
        }
        out[0] = G;
        out[1] = E;
        out[2] = static_cast<unsigned long long>(n_pos) * cfg.C * n_neg * cfg.C;
    }
}

template <typename Src>
__global__ __launch_bounds__(kCountThreads) void auroc_counts_kernel(
    Src src, const float* __restrict__ scores, uint64_t n_scores, Key key, uint32_t flags,
    unsigned long long* __restrict__ counts, unsigned long long* __restrict__ baseline) {
    src.keep(blockIdx.x);
    counts_body(blockIdx.x, src.cfg(blockIdx.x), scores, n_scores, key, flags, counts, baseline);
}

// The counts and the pooled ranking of a configuration, a workgroup each in
// one launch.  16 waves per workgroup: a 256-canary run of 16 shards takes
// four rounds of the counts and four scores per thread of the search.
// Kernel times with every count, against one workgroup per configuration that
// sorted all of its scores: 4 x 8 scores 5.5 us (11.3 us), 16 x 256 scores
// three times 8.7 us (67 us), 216 configurations of 8, 16 and 32 x 32 scores
// 12.1 us (34.5 us); 40 of 48 x 240 scores, with the per-canary counts and
// every launch, 59 us (498 us).
static_assert(kCountThreads == kPoolThreads, "one workgroup shape for both parts");
template <typename Src>
__global__ __launch_bounds__(kCountThreads) void auroc_counts_pooled_kernel(
    Src src, const float* __restrict__ scores, uint64_t n_scores, Key key, uint32_t flags,
    unsigned long long* __restrict__ counts, unsigned long long* __restrict__ baseline,
    unsigned long long* __restrict__ pooled) {
    const AurocCfgDev cfg = src.cfg(blockIdx.x);
    if (blockIdx.y) {
        pooled_body(blockIdx.x, cfg, scores, n_scores, pooled);
    } else {
        src.keep(blockIdx.x);
        counts_body(blockIdx.x, cfg, scores, n_scores, key, flags, counts, baseline);
    }
}

// Eq. 6 from integer counts: G / pairs (ties count 0, the equation as
// printed) and (G + E / 2) / pairs (ties count one half, the Mann-Whitney
// form), in fp64.  A triple with no pairs, or one holding the out-of-bounds
// marker, gives NaN.
__device__ __forceinline__ void ratios(const unsigned long long* c, double* out) {
    const unsigned long long G = c[0], E = c[1], N = c[2];
    if (N == 0 || G == kBadCfg || E == kBadCfg || N == kBadCfg) {
        out[0] = out[1] = __builtin_nan("");
        return;
    }
    const double n = static_cast<double>(N);
    out[0] = static_cast<double>(G) / n;
    out[1] = (static_cast<double>(G) + 0.5 * static_cast<double>(E)) / n;
}

__global__ void auroc_values_kernel(uint32_t n_cfg, const unsigned long long* __restrict__ counts,
                                    const unsigned long long* __restrict__ pooled,
                                    const unsigned long long* __restrict__ baseline,
                                    double* __restrict__ values) {
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n_cfg) return;
    double* v = values + 8ull * g;
    ratios(counts + 6ull * g, v);
    ratios(counts + 6ull * g + 3, v + 2);
    if (pooled) {
        ratios(pooled + 3ull * g, v + 4);
    } else {
        v[4] = v[5] = __builtin_nan("");
    }
    if (baseline) {
        ratios(baseline + 3ull * g, v + 6);
    } else {
        v[6] = v[7] = __builtin_nan("");
    }
}

}  // namespace

hipError_t launch_auroc_values(uint32_t n_cfg, const uint64_t* counts, const uint64_t* pooled,
                               const uint64_t* baseline, double* values, hipStream_t st) {
    if (n_cfg == 0) return hipSuccess;
    hipLaunchKernelGGL(auroc_values_kernel, dim3((n_cfg + 255) / 256), dim3(256), 0, st, n_cfg,
                       reinterpret_cast<const unsigned long long*>(counts),
                       reinterpret_cast<const unsigned long long*>(pooled),
                       reinterpret_cast<const unsigned long long*>(baseline), values);
    return hipGetLastError();
}

namespace {

CfgArgs cfg_args(uint32_t n_cfg, const AurocCfgDev* cfgs, AurocCfgDev* table) {
    CfgArgs a{};
    for (uint32_t g = 0; g < n_cfg; ++g) a.cfgs[g] = cfgs[g];
    a.table = table;
    return a;
}

template <typename Src>
hipError_t launch_canaries_t(const Src& src, uint32_t n_cfg, const float* scores,
                             uint64_t n_scores, uint64_t seed, uint32_t flags,
                             uint32_t* per_canary, hipStream_t st) {
    if (n_cfg == 0) return hipSuccess;
    const Key key{static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32)};
    hipLaunchKernelGGL(auroc_canaries_kernel<Src>, dim3(n_cfg), dim3(kCountThreads), 0, st, src,
                       scores, n_scores, key, flags, per_canary);
    return hipGetLastError();
}

template <typename Src>
hipError_t launch_auroc_t(const Src& src, uint32_t n_cfg, const float* scores, uint64_t n_scores,
                          uint64_t seed, uint32_t flags, uint64_t* counts, uint64_t* pooled,
                          uint64_t* baseline, hipStream_t st) {
    if (n_cfg == 0) return hipSuccess;
    const Key key{static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32)};
    if (flags & 2u) {
        hipLaunchKernelGGL(auroc_counts_pooled_kernel<Src>, dim3(n_cfg, 2), dim3(kCountThreads),
                           0, st, src, scores, n_scores, key, flags,
                           reinterpret_cast<unsigned long long*>(counts),
                           reinterpret_cast<unsigned long long*>(baseline),
                           reinterpret_cast<unsigned long long*>(pooled));
    } else {
        hipLaunchKernelGGL(auroc_counts_kernel<Src>, dim3(n_cfg), dim3(kCountThreads), 0, st, src,
                           scores, n_scores, key, flags,
                           reinterpret_cast<unsigned long long*>(counts),
                           reinterpret_cast<unsigned long long*>(baseline));
    }
    return hipGetLastError();
}

}  // namespace

bool auroc_in_args(uint32_t n_cfg) { return n_cfg <= kArgCfgs; }

hipError_t launch_auroc_canaries(uint32_t n_cfg, const AurocCfgDev* cfgs_dev,
                                 const uint64_t* offsets_dev, const float* scores,
                                 uint64_t n_scores, uint64_t seed, uint32_t flags,
                                 uint32_t* per_canary, hipStream_t st) {
    return launch_canaries_t(CfgTable{cfgs_dev, offsets_dev}, n_cfg, scores, n_scores, seed,
                             flags, per_canary, st);
}

hipError_t launch_auroc_canaries_args(uint32_t n_cfg, const AurocCfgDev* cfgs,
                                      const float* scores, uint64_t n_scores, uint64_t seed,
                                      uint32_t flags, uint32_t* per_canary, hipStream_t st) {
    return launch_canaries_t(cfg_args(n_cfg, cfgs, nullptr), n_cfg, scores, n_scores, seed, flags,
                             per_canary, st);
}

hipError_t launch_auroc(uint32_t n_cfg, const AurocCfgDev* cfgs_dev, const float* scores,
                        uint64_t n_scores, uint64_t seed, uint32_t flags, uint64_t* counts,
                        uint64_t* pooled, uint64_t* baseline, hipStream_t st) {
    return launch_auroc_t(CfgTable{cfgs_dev, nullptr}, n_cfg, scores, n_scores, seed, flags,
                          counts, pooled, baseline, st);
}

hipError_t launch_auroc_args(uint32_t n_cfg, const AurocCfgDev* cfgs, AurocCfgDev* table,
                             const float* scores, uint64_t n_scores, uint64_t seed,
                             uint32_t flags, uint64_t* counts, uint64_t* pooled,
                             uint64_t* baseline, hipStream_t st) {
    return launch_auroc_t(cfg_args(n_cfg, cfgs, table), n_cfg, scores, n_scores, seed, flags,
                          counts, pooled, baseline, st);
}

}  // namespace cdt
