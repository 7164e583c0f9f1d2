// Philox4x32-10 for kernels in which a lane draws one block for many rails of
// one step: the counter is (c0, rail, n, c3), of which c0 and c3 are fixed per
// lane and n per step, so the parts of the first rounds that depend on those
// alone are computed once (34 instead of 40 VALU instructions per block).  The
// words equal philox4x32_10(c0, rail, n, c3, k0, k1).
#pragma once
#include "kmc_device.h"

namespace kmc {

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u, kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

struct PhiloxLane {  // of one lane
    uint32_t lo1_k;  // round 1: lo(M1 x2) ^ (k0 + 2 W0)
    uint32_t hi1_k;  // hi(M1 x2) ^ (k0 + W0)
    uint32_t y3_k;   // round 0: lo(M0 c0) ^ (k1 + W1)
};
struct PhiloxStep {  // of one step
    uint32_t y0;     // round 0: hi(M1 n) ^ k0
    uint32_t lo2, hi2_k;  // round 2: M0 x0, its upper half ^ (k1 + 2 W1)
};

__device__ __forceinline__ PhiloxLane philox_lane(uint32_t c0, uint32_t c3, uint32_t k0, uint32_t k1) {
    const uint64_t m0 = (uint64_t)kPhiloxM0 * c0;
    const uint64_t m1 = (uint64_t)kPhiloxM1 * ((uint32_t)(m0 >> 32) ^ c3 ^ k1);
    return {(uint32_t)m1 ^ (k0 + 2u * kPhiloxW0), (uint32_t)(m1 >> 32) ^ (k0 + kPhiloxW0),
            (uint32_t)m0 ^ (k1 + kPhiloxW1)};
}

__device__ __forceinline__ PhiloxStep philox_step(const PhiloxLane &c, uint32_t n, uint32_t k0, uint32_t k1) {
    const uint64_t m1 = (uint64_t)kPhiloxM1 * n;
    const uint64_t a2 = (uint64_t)kPhiloxM0 * (c.hi1_k ^ (uint32_t)m1);
    return {(uint32_t)(m1 >> 32) ^ k0, (uint32_t)a2, (uint32_t)(a2 >> 32) ^ (k1 + 2u * kPhiloxW1)};
}

__device__ __forceinline__ uint4 philox_words(const PhiloxLane &c, const PhiloxStep &s, uint32_t rail, uint32_t k0,
                                              uint32_t k1) {
    const uint64_t a1 = (uint64_t)kPhiloxM0 * (s.y0 ^ rail);
    const uint64_t b2 = (uint64_t)kPhiloxM1 * ((uint32_t)(a1 >> 32) ^ c.y3_k);
    uint32_t x0 = (uint32_t)(b2 >> 32) ^ c.lo1_k, x1 = (uint32_t)b2;
    uint32_t x2 = s.hi2_k ^ (uint32_t)a1, x3 = s.lo2;
    uint32_t kr0 = k0 + 2u * kPhiloxW0, kr1 = k1 + 2u * kPhiloxW1;
#pragma unroll
    for (int round = 3; round < 10; ++round) {
        kr0 += kPhiloxW0;
        kr1 += kPhiloxW1;
        const uint64_t m0 = (uint64_t)kPhiloxM0 * x0;
        const uint64_t m1 = (uint64_t)kPhiloxM1 * x2;
        const uint32_t y0 = xor3((uint32_t)(m1 >> 32), x1, kr0);
        const uint32_t y2 = xor3((uint32_t)(m0 >> 32), x3, kr1);
        x1 = (uint32_t)m1;
        x3 = (uint32_t)m0;
        x0 = y0;
        x2 = y2;
    }
    return make_uint4(x0, x1, x2, x3);
}

}  // namespace kmc
