// Device-side building blocks shared by the libcdt kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cdt {

constexpr int kWave = 64;

// MI355X has 8 accelerator complex dies (XCDs), each with its own L2;
// consecutive workgroup ids are dispatched round-robin over them.
constexpr uint32_t kXcds = 8;

// Remap a work index so that each XCD walks one contiguous range of
// [0, total): index `it` runs on XCD it % 8 (true when the grid stride is a
// multiple of 8 or the grid covers all of [0, total) once).  A bijection of
// [0, total) for every total.
__device__ __forceinline__ uint64_t xcd_contiguous(uint64_t it, uint64_t total) {
    const uint64_t x = it % kXcds, local = it / kXcds;
    const uint64_t base = total / kXcds, rem = total % kXcds;
    return x * base + (x < rem ? x : rem) + local;
}

// Iteration `it` of `total` chunks, `per_shard` of them to a shard -> its chunk:
// XCD it % 8 walks one contiguous eighth of each shard, shard by shard.  What an
// uneven eighth leaves of the shards comes last.
__host__ __device__ __forceinline__ uint64_t shard_eighths(uint64_t it, uint64_t total,
                                                           uint64_t per_shard) {
    const uint64_t eighth = per_shard / kXcds, rest = per_shard % kXcds;
    const uint64_t even = total / per_shard * (eighth * kXcds);
    if (it < even) {
        const uint64_t x = it % kXcds, l = it / kXcds, s = l / eighth;
        return s * per_shard + x * eighth + (l - s * eighth);
    }
    const uint64_t l = it - even, s = l / rest;
    return s * per_shard + eighth * kXcds + (l - s * rest);
}

// Native 16-byte vectors (usable with the nontemporal load/store builtins).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Pointers into device memory (the global address space).  Loads and stores
// through them compile to global_* instructions also where the pointer was
// read from memory (a batched launch's job table), where a generic pointer
// would give flat_* instructions, which also count against the LDS and
// scalar-load counter and so make every wait on either one wait for them.
template <typename T>
using gptr = __attribute__((address_space(1))) T*;

template <typename T>
__device__ __forceinline__ gptr<T> global_ptr(T* p) {
    return (gptr<T>)p;
}

// Random stream ids (fourth counter word = stream << 24 | id).
enum : uint32_t {
    kStreamRef = 0,
    kStreamBenign = 1,
    kStreamT12 = 2,
    kStreamT3 = 3,
    kStreamTamperAdd = 4,
    kStreamTamperFlip = 5,
    kStreamScramble = 6,
    kStreamRandom = 7,
    kStreamOutlier = 8,
    kStreamAlt = 9,
    kStreamAltT12 = 10,
    kStreamAltT3 = 11,
};

struct Words4 {
    uint32_t x, y, z, w;
};

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two
// 32x32->64 multiplies on counter words 0 and 2, XOR of the high halves into
// words 1 and 3 with the round key, and a word permutation; the key advances
// by the two Weyl increments between rounds.  Each round is two
// v_mad_u64_u32 and two 3-input XORs (v_bitop3_b32, truth table 0x96 =
// a ^ b ^ c); while a counter word is wave-uniform (the canary, shard and
// stream words are) the product stays on the scalar unit.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

__device__ __forceinline__ Words4 philox_round(Words4 c, uint32_t k0, uint32_t k1) {
    const uint64_t p0 = static_cast<uint64_t>(kPhiloxM0) * c.x;
    const uint64_t p1 = static_cast<uint64_t>(kPhiloxM1) * c.z;
    return Words4{xor3(static_cast<uint32_t>(p1 >> 32), c.y, k0), static_cast<uint32_t>(p1),
                  xor3(static_cast<uint32_t>(p0 >> 32), c.w, k1), static_cast<uint32_t>(p0)};
}

__device__ __forceinline__ Words4 philox10(Words4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (uint32_t r = 0; r < 10; ++r) c = philox_round(c, k0 + r * kPhiloxW0, k1 + r * kPhiloxW1);
    return c;
}

struct Key {
    uint32_t k0, k1;
};

__device__ __forceinline__ Key make_key(uint64_t seed) {
    return Key{static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32)};
}

__device__ __forceinline__ Words4 draw(Key k, uint32_t q, uint32_t c, uint32_t s, uint32_t tag) {
    return philox10(Words4{q, c, s, tag}, k.k0, k.k1);
}

__host__ __device__ constexpr uint32_t stream_tag(uint32_t stream, uint32_t id) {
    return (stream << 24) | (id & 0xFFFFFFu);
}

// A wave-uniform value held in a vector register.  A two-operand VALU
// instruction issues in 2 cycles when both operands are vector registers and
// in 4 with a scalar one (measured: v_xor_b32 2.6 against 4.4 cycles per
// wave64 instruction and SIMD, launch included), so the few constants that
// every Philox call XORs once are worth a register each.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t x) {
    asm("" : "+v"(x));
    return x;
}

// The draws of one (canary, shard) block.  The live passes spend most of
// their time in philox10's rounds, and the counters (q, c, s, tag) of a
// block's draws differ in few words, so the first three rounds are taken
// apart by what they depend on (round outputs x, y, z, w, round keys k0, k1):
//   round 0: x1, y1 from (c, s): uniform; z1 = hi(M0 q) ^ tag ^ k1, w1 = lo(M0 q);
//   round 1: x2 = hi(M1 z1) ^ y1 ^ k0, y2 = lo(M1 z1);
//            z2 = hi(M0 x1) ^ w1 ^ k1, which no tag enters, w2 = lo(M0 x1): uniform;
//   round 2: x3 = hi(M1 z2) ^ y2 ^ k0, y3 = lo(M1 z2) (no tag), z3 = hi(M0 x2) ^ w2 ^ k1,
//            w3 = lo(M0 x2).
// BlockDraw holds the uniform parts, DrawBase what depends on q alone (two of
// the 18 multiplies left per call, shared by every stream and run drawn at
// the same q), and finish_draw does the rest: 16 multiplies, 14 three-operand
// XORs and 4 two-operand ones (before: 18 and 19).  Same words as draw().
// Together with irwin_hall4's subtraction this took 1.9% off the step of three
// 16 x 128 x 256 x 8192 runs (18.96 to 18.6 ms; 16.0 ms with what came after),
// 2.8% off a Student-t run of 16 x 128 x 128 x 4096 with its Eq. 4 (4.31 to 4.19
// ms; now 4.0) and 2.3% off the fused pass of 32 x 32 x 64 x 8192 (646 to 631
// us; now 544).
struct BlockDraw {
    uint32_t k0, k1;          // the key
    uint32_t z2, x2, z3, x3;  // hi(M0 x1) ^ k1, y1 ^ k0, w2 ^ k1 and k0 of rounds 1, 1, 2, 2
};

struct DrawBase {
    uint32_t h0;  // hi(M0 q)
    uint32_t x3;  // hi(M1 z2) ^ k0 of round 2
    uint32_t y3;  // lo(M1 z2)
};

__device__ __forceinline__ BlockDraw block_draw(Key k, uint32_t c, uint32_t s) {
    const uint64_t p1 = static_cast<uint64_t>(kPhiloxM1) * s;
    const uint32_t x1 = static_cast<uint32_t>(p1 >> 32) ^ c ^ k.k0;
    const uint64_t p0 = static_cast<uint64_t>(kPhiloxM0) * x1;
    BlockDraw b;
    b.k0 = k.k0;
    b.k1 = k.k1;
    b.z2 = in_vgpr(static_cast<uint32_t>(p0 >> 32) ^ (k.k1 + kPhiloxW1));
    b.x2 = in_vgpr(static_cast<uint32_t>(p1) ^ (k.k0 + kPhiloxW0));
    b.z3 = in_vgpr(static_cast<uint32_t>(p0) ^ (k.k1 + 2 * kPhiloxW1));
    b.x3 = in_vgpr(k.k0 + 2 * kPhiloxW0);
    return b;
}

__device__ __forceinline__ DrawBase draw_base(const BlockDraw& b, uint32_t q) {
    const uint64_t p0 = static_cast<uint64_t>(kPhiloxM0) * q;
    const uint64_t p1 = static_cast<uint64_t>(kPhiloxM1) * (static_cast<uint32_t>(p0) ^ b.z2);
    return DrawBase{static_cast<uint32_t>(p0 >> 32), static_cast<uint32_t>(p1 >> 32) ^ b.x3,
                    static_cast<uint32_t>(p1)};
}

// tag_key: the stream's tag ^ the key's high word.
__device__ __forceinline__ Words4 finish_draw(const BlockDraw& b, const DrawBase& d,
                                              uint32_t tag_key) {
    const uint64_t p1 = static_cast<uint64_t>(kPhiloxM1) * (d.h0 ^ tag_key);
    const uint64_t p0 =
        static_cast<uint64_t>(kPhiloxM0) * (static_cast<uint32_t>(p1 >> 32) ^ b.x2);
    Words4 c{d.x3 ^ static_cast<uint32_t>(p1), d.y3, static_cast<uint32_t>(p0 >> 32) ^ b.z3,
             static_cast<uint32_t>(p0)};
#pragma unroll
    for (uint32_t r = 3; r < 10; ++r)
        c = philox_round(c, b.k0 + r * kPhiloxW0, b.k1 + r * kPhiloxW1);
    return c;
}

// Unit normal stand-in: the Irwin-Hall sum of the four 16-bit halves of two
// Philox words, centred (4 * 32767.5) and scaled by fp32(sqrt(3/(2^32-1))).
// v_sad_u16(w, 0, acc) adds both 16-bit halves of w to acc.  The accumulator
// starts at the bits of 1.5 * 2^23 less 131070, so it ends as the bits of the
// float 1.5 * 2^23 + n (|n| <= 131070, one bit step is 1), and subtracting
// 1.5 * 2^23 leaves n exactly: a 2-cycle subtraction for the 4-cycle int-to-
// float conversion.
__device__ __forceinline__ float irwin_hall4(uint32_t w0, uint32_t w1) {
    const uint32_t bits = __builtin_amdgcn_sad_u16(
        w0, 0u, __builtin_amdgcn_sad_u16(w1, 0u, 0x4B400000u - 131070u));
    return (__uint_as_float(bits) - 0x1.8p23f) * 0x1.bb67aep-16f;
}

// fp32 -> fp16 bits, IEEE round to nearest even (v_cvt_f16_f32 under the
// default round-to-nearest mode; fp16 subnormals are kept).
__device__ __forceinline__ uint16_t to_half_bits(float v) {
    const _Float16 h = static_cast<_Float16>(v);
    return __builtin_bit_cast(uint16_t, h);
}

// Two fp32 values -> packed fp16 bits (lo in bits 0-15), the same IEEE
// round to nearest even as to_half_bits; gfx950 converts the pair with one
// v_cvt_pk_f16_f32.
__device__ __forceinline__ uint32_t to_half2_bits(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, f16x2));
}

__device__ __forceinline__ float half_bits_to_float(uint32_t bits16) {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(bits16)));
}

// Order-preserving key of a score: numeric order with -0 == +0, and NaN
// above every number (+inf included): a block whose mismatch is not a number
// ranks as the most suspicious stage (Eq. 5 ranks larger mismatches higher).
// Every number maps below 0xFFFFFFFF (+inf maps to 0xFF800000).
__device__ __forceinline__ uint32_t order_key(float x) {
    if (x != x) return 0xFFFFFFFFu;
    uint32_t u = __float_as_uint(x);
    if (x == 0.0f) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Wave-wide sums (wave64, butterfly through ds_swizzle/DPP lowering).
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Reading the fp32 reference of one wave's 64 groups of 8 elements (512
// elements, 2 KB).  One 16-byte load per group and thread (lane L: quads
// 2L and 2L + 1 of the wave's 128 four-element quads) makes each load
// instruction touch every other 16 bytes of the 2 KB span, and such a
// stream runs a few percent below contiguous runs.  So lane L loads quads
// L and 64 + L instead (two contiguous 1 KB runs), and quads_to_groups
// moves them to their owners in two steps:
//   1. neighbours 2m and 2m + 1 swap one quad (DPP quad_perm [1, 0, 3, 2]):
//      lane 2m then holds quads 2m, 2m + 1 and lane 2m + 1 holds 64 + 2m,
//      65 + 2m;
//   2. lane L pulls both quads from lane 2L (L < 32) or 2L - 63 (L >= 32)
//      (ds_bpermute).
// The values each thread ends with are exactly those of the direct loads.
// Every lane of the wave must execute it: callers branch on a
// workgroup-uniform condition.
__device__ __forceinline__ float swap_adjacent_lanes(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));
}

__device__ __forceinline__ float pull_from_lane(int src_lane, float x) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(src_lane * 4, __float_as_int(x)));
}

// r0, r1: quads L and 64 + L (as loaded); lo, hi: quads 2L and 2L + 1.
__device__ __forceinline__ void quads_to_groups(const f32x4& r0, const f32x4& r1, f32x4& lo,
                                                f32x4& hi) {
    const int lane = static_cast<int>(threadIdx.x % kWave);
    const bool even = (lane & 1) == 0;
    const int src = ((lane << 1) & (kWave - 1)) | (lane >> 5);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float got = swap_adjacent_lanes(even ? r1[k] : r0[k]);
        lo[k] = pull_from_lane(src, even ? r0[k] : got);
        hi[k] = pull_from_lane(src, even ? got : r1[k]);
    }
}

}  // namespace cdt
