// Philox4x64-10 counter-based generator (Salmon, Moraes, Dror, Shaw, SC'11), host and device.
// Ten rounds of (hi0,lo0) = M0*x0, (hi1,lo1) = M1*x2, x <- (hi1^x1^k0, lo1, hi0^x3^k1, lo0), with
// the key advanced by the Weyl constants between rounds.
#pragma once

#include <math.h>
#include <stdint.h>

#include "fh_fft.h"  // FH_HD

namespace fh {

constexpr uint64_t kPhiloxM0 = 0xD2E7470EE14C6C93ull;
constexpr uint64_t kPhiloxM1 = 0xCA5A826395121157ull;
constexpr uint64_t kPhiloxW0 = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kPhiloxW1 = 0xBB67AE8584CAA73Bull;

constexpr uint64_t kTagPath = 0;
constexpr uint64_t kTagGibbs = 1;
constexpr uint64_t kTagLocal = 2;  // local link updates; pass k uses kTagLocal + 256 k
constexpr uint64_t kTagMala = 3;        // MALA proposal noise per (site, slice)
constexpr uint64_t kTagMalaAccept = 4;  // MALA acceptance uniform per chain
constexpr uint64_t kTagPerm = 5;        // reconnection swaps; pass k uses kTagPerm + 256 k

// Both halves of a 64 x 64 product from four 32 x 32 + 64 multiply-adds: a round needs both, and
// the high half's multiply-adds already hold the low one (the two taken apart cost two more
// quarter-rate multiplications per product; the field draw of 16 chains of 160 x 32 x 32 sites
// 42 -> 37 us, with the cosine below).
FH_HD inline void mul128(uint64_t a, uint64_t b, uint64_t* hi, uint64_t* lo) {
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
    const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
    const uint64_t p = (uint64_t)a0 * b0;
    const uint64_t t = (uint64_t)a1 * b0 + (p >> 32);
    const uint64_t u = (uint64_t)a0 * b1 + (uint32_t)t;
    *hi = (uint64_t)a1 * b1 + (t >> 32) + (u >> 32);
    *lo = (u << 32) | (uint32_t)p;
}

struct u64x4 {
    uint64_t x0, x1, x2, x3;
};

// R rounds of the generator on counter x with keys k0, k1 (both advanced).
template <int R>
FH_HD inline void philox_rounds(u64x4& x, uint64_t& k0, uint64_t& k1) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint64_t hi0, lo0, hi1, lo1;
        mul128(kPhiloxM0, x.x0, &hi0, &lo0);
        mul128(kPhiloxM1, x.x2, &hi1, &lo1);
        x = {hi1 ^ x.x1 ^ k0, lo1, hi0 ^ x.x3 ^ k1, lo0};
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
    }
}

FH_HD inline u64x4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0,
                                  uint64_t k1) {
    u64x4 x = {c0, c1, c2, c3};
    philox_rounds<10>(x, k0, k1);
    return x;
}

// 53-bit uniform in [0, 1).
FH_HD inline double u01_from(uint64_t x) { return (double)(x >> 11) * 0x1.0p-53; }

// Box-Muller standard normal: u1 in (0, 1], u2 in [0, 1).
FH_HD inline double normal_from(uint64_t x0, uint64_t x1) {
    const double u1 = (double)((x0 >> 11) + 1) * 0x1.0p-53;
    const double u2 = (double)(x1 >> 11) * 0x1.0p-53;
#if defined(__HIP_DEVICE_COMPILE__)
    return sqrt(-2.0 * log(u1)) * cospi(2.0 * u2);  // 2 u2 is exact: no argument reduction
#else
    return sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
#endif
}

}  // namespace fh
