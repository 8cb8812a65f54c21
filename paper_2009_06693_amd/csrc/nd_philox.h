// Device-side random numbers and integer helpers.
//
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy
// as 1, 2, 3", SC'11): a counter-based generator, so a draw is a pure function
// of (seed, sample, slot, step, attempt) and the grouping of samples by transit
// (Section 5.2 of the NextDoor paper) cannot change what is drawn.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nd_common.h"

namespace nd {

struct Rand4 {
    uint32_t r0, r1, r2, r3;
};

// a ^ b ^ c in one instruction, which the compiler (ROCm 7.2) does not choose by itself.  A generator call is ten
// rounds of two multiplications and two of these, each waiting for the one before: 296 cycles alone on a SIMD with two
// exclusive ors in their place, 202 like this; 199 and 162 cycles of issue where eight wavefronts share the SIMD.
// JOINED false: two instructions after all, for a kernel that was measured to be the faster for it.
template <bool JOINED>
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return JOINED ? (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96) : a ^ b ^ c;
}

template <bool JOINED = true>
__device__ __forceinline__ Rand4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3<JOINED>((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3<JOINED>((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return Rand4{c0, c1, c2, c3};
}

// Counter layout of every draw: (sample id, slot within the sample, step, attempt).
template <bool JOINED = true>
__device__ __forceinline__ Rand4 draw4(uint64_t seed, uint32_t sample_id, uint32_t slot,
                                       uint32_t step, uint32_t attempt) {
    return philox4x32_10<JOINED>(sample_id, slot, step, attempt, (uint32_t)seed, (uint32_t)(seed >> 32));
}

__device__ __forceinline__ uint32_t mulhi32(uint32_t a, uint32_t b) { return __umulhi(a, b); }
__device__ __forceinline__ uint64_t mulhi64(uint64_t a, uint64_t b) { return __umul64hi(a, b); }
__device__ __forceinline__ uint64_t cat64(uint32_t hi, uint32_t lo) { return ((uint64_t)hi << 32) | lo; }

// n / T and the remainder for n < 2^24 T, n < 2^63, T < 2^39, inv = 1 / T rounded: the product is within
// 2^-27 of the quotient, so its whole part is off by at most one.
__device__ __forceinline__ uint32_t divide_step(uint64_t n, uint64_t T, double inv, uint64_t* rest) {
    uint32_t q = (uint32_t)((double)n * inv);
    int64_t r = (int64_t)(n - (uint64_t)q * T);
    if (r < 0) {
        --q;
        r += (int64_t)T;
    } else if (r >= (int64_t)T) {
        ++q;
        r -= (int64_t)T;
    }
    *rest = (uint64_t)r;
    return q;
}
// ceil(c * 2^64 / T) for 0 <= c < T < 2^39: long division, 24 + 24 + 16 bits at a time.
__device__ __forceinline__ uint64_t scaled_threshold(uint64_t c, uint64_t T) {
    const double inv = 1.0 / (double)T;
    uint64_t r;
    const uint64_t q1 = divide_step(c << 24, T, inv, &r);
    const uint64_t q2 = divide_step(r << 24, T, inv, &r);
    const uint64_t q3 = divide_step(r << 16, T, inv, &r);
    return (q1 << 40) + (q2 << 16) + q3 + (r != 0 ? 1u : 0u);  // below 2^64: c < T
}

__device__ __forceinline__ uint32_t fastdiv(uint32_t n, const FastDiv& f) {
    return f.d == 1 ? n : (__umulhi(n, f.magic) >> f.shift);
}

}  // namespace nd
