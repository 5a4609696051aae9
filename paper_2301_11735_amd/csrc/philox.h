// Philox4x32-10 counter-based generator (Salmon, Moraes, Dror, Shaw,
// "Parallel random numbers: as easy as 1, 2, 3", SC'11), usable on the host
// and in gfx950 kernels.  Ten rounds; each round multiplies counter words 0
// and 2 by the round multipliers, the high halves are xored with the other
// two words and the round key, and the key advances by the Weyl constants.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lat {

struct u32x4 {
    uint32_t x, y, z, w;
};

constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u;
constexpr uint32_t kPhiloxW1 = 0xBB67AE85u;

// Counter word 1 selects the stream: the phase (0..3) for pair updates, or
// one of these domains.
constexpr uint32_t kDomSchedule = 0x100u;
constexpr uint32_t kDomInit = 0x200u;

// A call on its way: counter words and round key.  philox_rounds lets a kernel
// put other work between a call's rounds.
struct PhiloxRun {
    uint32_t c0, c1, c2, c3, k0, k1;
};
template <int Rounds>
__host__ __device__ __forceinline__ void philox_rounds(PhiloxRun &r)
{
#pragma unroll
    for (int i = 0; i < Rounds; ++i) {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * r.c0;
        const uint64_t p1 = (uint64_t)kPhiloxM1 * r.c2;
#if defined(__HIP_DEVICE_COMPILE__)
        // gfx950 three-input boolean op; truth table 0x96 is a ^ b ^ c
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), r.c1, r.k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), r.c3, r.k1, 0x96);
#else
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ r.c1 ^ r.k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ r.c3 ^ r.k1;
#endif
        r.c1 = (uint32_t)p1;
        r.c3 = (uint32_t)p0;
        r.c0 = n0;
        r.c2 = n2;
        r.k0 += kPhiloxW0;
        r.k1 += kPhiloxW1;
    }
}

__host__ __device__ __forceinline__ u32x4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                                        uint32_t c3, uint32_t k0, uint32_t k1)
{
    PhiloxRun r{c0, c1, c2, c3, k0, k1};
    philox_rounds<10>(r);
    return {r.c0, r.c1, r.c2, r.c3};
}

__host__ __device__ __forceinline__ uint32_t mulhi_u32(uint32_t a, uint32_t b)
{
    return (uint32_t)(((uint64_t)a * b) >> 32);
}

}  // namespace lat
