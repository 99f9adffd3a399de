// Shared device helpers of libcard (gfx950 / CDNA4, 64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "card_layout.h"

namespace card {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(4))) unsigned int uint4v;

// ---- weights in three planes (CodedDesc) --------------------------------------------------------------
// Eight weights of a lane as they are stored: low bytes, high nibbles, rest nibbles.  Bits 8-14 of a weight are (base + c) ^ (rest << 3),
// where base + c <= 127: any value has one c and one rest.  The nibbles of weights 0-3 lie in byte i as the byte that they
// become needs them (sign in bit 7, c in bits 0-2; rest in bits 3-6), those of weights 4-7 likewise, but four bits further left.
__device__ __forceinline__ uint32_t rotate_right4(uint32_t v) { return __builtin_amdgcn_alignbit(v, v, 4); }
__device__ __forceinline__ uint32_t high_bytes(uint32_t high, uint32_t rest, uint32_t base4) {
    return ((high & 0x87878787u) + base4) ^ (rest & 0x78787878u);  // (no carry: base + c < 128)
}
// low bytes and high bytes of eight weights -> the weights
__device__ __forceinline__ uint4v join_weights(uint4v v) {
    return uint4v{__builtin_amdgcn_perm(v[2], v[0], 0x05010400u), __builtin_amdgcn_perm(v[2], v[0], 0x07030602u),
                                             __builtin_amdgcn_perm(v[3], v[1], 0x05010400u), __builtin_amdgcn_perm(v[3], v[1], 0x07030602u)};
}
// {low, low, high, rest} as loaded -> the weights
__device__ __forceinline__ uint4v decode_weights(uint4v v, uint32_t base4) {
    return join_weights(uint4v{v[0], v[1], high_bytes(v[2], v[3], base4), high_bytes(rotate_right4(v[2]), rotate_right4(v[3]), base4)});
}
// and back
__device__ __forceinline__ uint4v encode_weights(bf16x8 w, uint32_t base) {
    const uint4v d = __builtin_bit_cast(uint4v, w);
    uint4v out = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t x = (d[e >> 1] >> ((e & 1) * 16)) & 0xffffu, h = (x >> 8) & 127u;
        const uint32_t c = (h - base) & 7u, rest = ((base + c) ^ h) >> 3;
        const uint32_t hb = ((x >> 15) << 7 | c) << ((e & 3) * 8), rb = rest << ((e & 3) * 8 + 3);
        out[e >> 2] |= (x & 255u) << ((e & 3) * 8);
        out[2] |= e < 4 ? hb : (hb << 4 | hb >> 28);
        out[3] |= e < 4 ? rb : (rb << 4 | rb >> 28);
    }
    return out;
}

// Data handed from one workgroup to another inside a kernel goes through device-scope accesses:
// the store writes through the compute die's own L2, the load bypasses it.  (A full device fence
// would write back and invalidate the whole L2 on every call - tens of microseconds.)
__device__ __forceinline__ void st_agent(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// order-preserving map float -> uint32 (larger float, larger key)
__device__ __forceinline__ uint32_t float_key(float v) {
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
// fp32 -> bf16 high part + bf16 remainder: two matrix instructions then see ~16 mantissa bits
__device__ __forceinline__ void split_bf16(float v, __bf16& hi, __bf16& lo) {
    hi = static_cast<__bf16>(v);
    lo = static_cast<__bf16>(v - static_cast<float>(hi));
}
// Rotary embedding of a pair: which product is rounded before the sum is fixed here, so that the verify kernels and the wide levels (which
// promise each other's bits) write the same K.  (The prompt pass sums its products in another order anyway.)
__device__ __forceinline__ float rotate_first(float z0, float z1, float cs, float sn) { return fmaf(z0, cs, -(z1 * sn)); }
__device__ __forceinline__ float rotate_second(float z0, float z1, float cs, float sn) { return fmaf(z1, cs, z0 * sn); }
// Reductions over the four rows of sixteen lanes of a wavefront (lanes l, l ^ 16, l ^ 32, l ^ 48), the same in all of them: register
// swaps.  A shuffle goes through LDS, 100 clocks and more each beside the weight stream: four of them stood in every round of an
// attention task, three in front of an RMSNorm scale, one in a residual epilogue (verify step, same states, us with shuffles / without:
// 1B decode 902 / 899, 8B r = 8 3246 / 3241, 7B r = 32 4370 / 4337, r = 13 3310 / 3297, 32 tree rows of the 1B shape 1279 / 1271).
template <typename F>
__device__ __forceinline__ float across_rows(float v, F&& op) {
    typedef __attribute__((ext_vector_type(2))) unsigned int pair;
    const uint32_t u = __float_as_uint(v);
    const pair p = __builtin_bit_cast(pair, __builtin_amdgcn_permlane16_swap(u, u, false, false));  // rows (0, 0, 2, 2) and (1, 1, 3, 3)
    v = op(__uint_as_float(p[0]), __uint_as_float(p[1]));
    const uint32_t w = __float_as_uint(v);
    const pair q = __builtin_bit_cast(pair, __builtin_amdgcn_permlane32_swap(w, w, false, false));  // the halves
    return op(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float max_across_rows(float v) {
    return across_rows(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float sum_across_rows(float v) {
    return across_rows(v, [](float a, float b) { return a + b; });
}
// Sum over a group of LPR neighbouring lanes (2, 4 or 8, all of them active), the same in all of them; register moves again.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    const int i = int(__float_as_uint(v));
    return v + __uint_as_float(uint32_t(__builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false)));
}
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {
    static_assert(LPR == 2 || LPR == 4 || LPR == 8, "part of a row of lanes");
    v = dpp_add<0xB1>(v);                            // lane ^ 1
    if constexpr (LPR > 2) v = dpp_add<0x4E>(v);     // lane ^ 2
    if constexpr (LPR > 4) v = dpp_add<0x141>(v);    // mirrored in eight: the other four
    return v;
}
// Largest of a group of LPR neighbouring lanes' values (8 or 16, all of them active): register moves
// inside a row of sixteen lanes, no trip through LDS.
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_max_step(unsigned long long v) {
    const int lo = int(uint32_t(v)), hi = int(uint32_t(v >> 32));
    const unsigned long long o = uint64_t(uint32_t(__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false))) |
                                 (uint64_t(uint32_t(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false))) << 32);
    return o > v ? o : v;
}
template <int LPR>
__device__ __forceinline__ unsigned long long group_max(unsigned long long v) {
    static_assert(LPR == 8 || LPR == 16, "part of a row of lanes");
    v = dpp_max_step<0xB1>(v);   // lane ^ 1
    v = dpp_max_step<0x4E>(v);   // lane ^ 2
    v = dpp_max_step<0x141>(v);  // mirrored in eight: the other four
    if constexpr (LPR == 16) v = dpp_max_step<0x140>(v);  // mirrored in sixteen: the other eight
    return v;
}
// element (head element j, token t) inside the V block of one page and head: pairs of 16-row
// tiles are interleaved so that one 16-byte load per lane feeds two P*V matrix instructions
__device__ __forceinline__ int v_page_index(int j, int t) {
    return ((((j >> 5) * 64) + (t >> 2) * 16 + (j & 15)) << 3) + ((j >> 4) & 1) * 4 + (t & 3);
}

}  // namespace card
