// The lazy Shoup product of the 64-bit integer butterflies.  No dependency but <stdint.h>: a CPU test compares it with 128-bit integers.
//
// a * w mod q for any 64-bit a, w < q, w_sh = floor(w * 2^64 / q), nq = 2^64 - q: the quotient's high word is taken from three of its four
// partial products, each cut to its high half, so it is at most three below the exact floor(a * w / q): two for what is cut, one for w_sh's
// own rounding.  The result, computed modulo 2^64, is in [0, 4q).  q < 2^58.
// The exact product takes four partial products with a zero-extension in front of each addition and both low products apart: 31 instructions
// of a butterfly, 26 now, and fewer of them off the full rate (v_mad_u64_u32 has it, v_mul_lo_u32 does not).  56-bit primes, forward and
// inverse: 65 limb-polys at N = 2^14 45.0 -> 43.4 us, 490 at 2^16 495 -> 464, 40 at 2^12 18.1 -> 16.8.  (The two partial products of which only
// the high half counts stay with the compiler's v_mul_hi_u32: forced to v_mad_u64_u32 44.4 and 479.)
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define SHOUP_FN __host__ __device__ __forceinline__
#else
#define SHOUP_FN static inline
#endif

SHOUP_FN uint64_t mul_shoup_lazy4(uint64_t a, uint64_t w, uint64_t w_sh, uint64_t nq) {
    const uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32), sl = (uint32_t)w_sh, sh = (uint32_t)(w_sh >> 32);
    const uint64_t m1 = (uint64_t)ah * sl, m2 = (uint64_t)al * sh;
    const uint64_t t = (uint64_t)ah * sh + ((m1 >> 32) + (m2 >> 32));
    const uint32_t tl = (uint32_t)t, th = (uint32_t)(t >> 32);
    // a * w - t * q = a * w + t * nq modulo 2^64: the low words, then the cross products, of which the low halves count
    const uint64_t low = (uint64_t)al * (uint32_t)w + (uint64_t)tl * (uint32_t)nq;
    uint64_t c = (uint64_t)al * (uint32_t)(w >> 32);
#if defined(__HIP_DEVICE_COMPILE__)
#define SHOUP_WIDE asm("" : "+v"(c));  // all 64 bits: the compiler would make it a slower 32-bit multiplication and an addition
#else
#define SHOUP_WIDE
#endif
    SHOUP_WIDE
    c += (uint64_t)ah * (uint32_t)w;
    SHOUP_WIDE
    c += (uint64_t)tl * (uint32_t)(nq >> 32);
    SHOUP_WIDE
    c += (uint64_t)th * (uint32_t)nq;
    SHOUP_WIDE
#undef SHOUP_WIDE
    return low + (c << 32);
}
