// philox.hpp -- device Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
//
// Counter-based: the output is a pure function of (counter, key), so every
// 64-site word draws its own random words from (g, t, 2j + parity, 0) with no
// per-thread generator state to load or store (the paper keeps a TinyMT
// state per thread, Sec. II-B).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sca {

struct u32x4 {
    uint32_t v0, v1, v2, v3;
};

constexpr uint32_t kMulA = 0xD2511F53u;
constexpr uint32_t kMulB = 0xCD9E8D57u;
constexpr uint32_t kWeylA = 0x9E3779B9u;
constexpr uint32_t kWeylB = 0xBB67AE85u;

// Rounds FIRST..9 of the ten, with the keys of round FIRST.
template <int FIRST = 0>
__device__ __forceinline__ u32x4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = FIRST; r < 10; ++r) {
        // One 32x32->64 product gives both halves (v_mad_u64_u32, full rate on
        // gfx950, where separate mul_hi and mul_lo take two instructions), and
        // each three-way xor is one v_bitop3_b32 (truth table 0x96).
        const uint64_t pA = (uint64_t)kMulA * c0;
        const uint64_t pB = (uint64_t)kMulB * c2;
        const uint32_t hiA = (uint32_t)(pA >> 32), loA = (uint32_t)pA;
        const uint32_t hiB = (uint32_t)(pB >> 32), loB = (uint32_t)pB;
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hiB, c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hiA, c3, k1, 0x96);
        c0 = n0;
        c1 = loB;
        c2 = n2;
        c3 = loA;
        k0 += kWeylA;
        k1 += kWeylB;
    }
    return {c0, c1, c2, c3};
}

// The block of counter (g, t, c2, 0) for a word index g that varies from lane
// to lane and t, c2, k0, k1 that are the same for the whole wave, as in every
// sweep.  The first two rounds are then mostly scalar: round 1 multiplies c2
// and round 2 the word that round 1 makes of c2, t and the key.  They are
// written with plain operators on the uniform values so that they run on the
// scalar unit; handed to the bitop3 builtin the uniform xor and the product of
// its result went to the vector unit (v_bitop3, v_mul_lo, v_mul_hi: three of 37
// vector instructions per block; 34 are left).  The p = 15/16 sweep of 2^16 x
// 2^16 is bound by these: 21 MCS in 5.02 ms instead of 5.24 ms.
__device__ __forceinline__ u32x4 philox_word(uint32_t g, uint32_t t, uint32_t c2, uint32_t k0, uint32_t k1)
{
    const uint64_t pB1 = (uint64_t)kMulB * c2;                               // scalar
    const uint32_t u0 = (uint32_t)(pB1 >> 32) ^ t ^ k0, u1 = (uint32_t)pB1;  // scalar
    const uint64_t pA1 = (uint64_t)kMulA * g;
    const uint32_t v2 = (uint32_t)(pA1 >> 32) ^ k1, v3 = (uint32_t)pA1;      // c3 = 0
    const uint64_t pA2 = (uint64_t)kMulA * u0;                               // scalar
    const uint64_t pB2 = (uint64_t)kMulB * v2;
    const uint32_t x0 = u1 ^ (k0 + kWeylA);                                  // scalar
    const uint32_t x2 = (uint32_t)(pA2 >> 32) ^ (k1 + kWeylB);               // scalar
    return philox4x32_10<2>((uint32_t)(pB2 >> 32) ^ x0, (uint32_t)pB2, v3 ^ x2, (uint32_t)pA2, k0 + 2 * kWeylA,
                            k1 + 2 * kWeylB);
}

}  // namespace sca
