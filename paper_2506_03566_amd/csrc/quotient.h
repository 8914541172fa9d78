// Many quotients by one divisor, plain C++ (the same on the host, where it is compared with the division).
#pragma once
#include <math.h>
#include <string.h>
#ifdef __HIPCC__
#define POSS_HD __host__ __device__ __forceinline__
#else
#define POSS_HD static inline
#endif

namespace poss {

// x / z with y = 1 / z (rounded to nearest), rounded to nearest as the division is: one correction makes the quotient faithful,
// the second, its remainder exact, rounds it (Markstein).  Five operations where the compiler's division takes about ten.  Holds
// where the remainders and the quotient stay above the subnormals and 1 / z is finite: quotient_divisor(z), and x zero or at
// least 2^-100 (an exact remainder of x reaches 47 bits below it); elsewhere it can be another number than x / z, or none.
POSS_HD float quotient(float x, float z, float y) {
    float q = x * y;
    q = fmaf(fmaf(-q, z, x), y, q);
    return fmaf(fmaf(-q, z, x), y, q);
}

POSS_HD bool quotient_divisor(float z) { return z >= 0x1p-100f && z <= 0x1p24f; }

// x >= 0 is too small for quotient() iff quotient_key(x) < QUOTIENT_LEAST (zero is not): the least key of several stands for all.
POSS_HD unsigned quotient_key(float x) {
    unsigned b;
    memcpy(&b, &x, sizeof b);
    return b - 1u;
}
constexpr unsigned QUOTIENT_LEAST = ((127u - 100u) << 23) - 1u;     // 2^-100

}  // namespace poss
