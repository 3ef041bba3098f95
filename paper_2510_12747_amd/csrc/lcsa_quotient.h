// Division of non-negative 32-bit numbers by one that the host knows: three instructions, where a division takes some thirty, each
// waiting for the one before (a kernel's first addresses are behind four or five of them: 0.1 us each).
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define LCSA_ANYWHERE __host__ __device__
#else
#define LCSA_ANYWHERE
#endif

namespace lcsa {

// n / d = floor(n m / 2^(31 + l)), 2^(l - 1) < d <= 2^l, m = ceil(2^(31 + l) / d) < 2^32: m d exceeds 2^(31 + l) by less than d <= 2^l, and so
// n m / 2^(31 + l) exceeds n / d by less than n / (2^31 d), which is less than 1 / d.
struct Quotient {
    uint32_t m, l;
    LCSA_ANYWHERE int operator()(int n) const { return (int)((uint32_t)(((uint64_t)(2u * (uint32_t)n) * m) >> 32) >> l); }
};

inline Quotient quotient_by(int d) {
    uint32_t l = 0;
    while ((1ull << l) < (uint64_t)d) ++l;
    return {(uint32_t)(((1ull << (31 + l)) + (uint64_t)d - 1) / (uint64_t)d), l};
}

} // namespace lcsa
