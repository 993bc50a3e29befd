// Device-side 32-bit modular arithmetic for RNS primes q < 2^31 on the
// integer VALU of gfx950 (v_mul_lo_u32 / v_mul_hi_u32 / v_mad_i64_i32).
//
// Reductions (Sec. 4.1, Alg. 2 and Table 3):
//  * mont(a, b)        a*b*2^-32 mod q for data x data products (Montgomery;
//                      the 2^-32 factors are folded into precomputed
//                      constants downstream, Sec. 5.1 Seq.2).
//  * mulc(x, W, Wt)    x*w mod q for a known constant w, stored "twisted":
//                      W = w*2^32 mod q and Wt = W*q^-1 mod 2^32, so the
//                      Montgomery quotient needs no product of x with a
//                      data-dependent value: 3 multiplies, 3 adds, output
//                      canonical in [0, q) for any 32-bit x.
//  * mulr(x, w, nq)    x*w mod q for a known constant and any signed 32-bit x,
//                      in (-3q/4, 3q/4): 3 multiply-adds (the NTT butterflies).
//  * smr64(x, t, tinv) signed Montgomery reduction (Seiler's signed variant
//                      of Montgomery's method) of a 64-bit signed sum: the
//                      reduction Sec. 4.1 picks for base conversion.
//  All outputs are canonical [0, q) unless stated.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ckks {

// r in (-q, q) held as a wrapped uint32 -> [0, q)
__device__ __forceinline__ uint32_t fix_signed(uint32_t r, uint32_t q) { return min(r, r + q); }

__device__ __forceinline__ uint32_t add_mod(uint32_t a, uint32_t b, uint32_t q)
{
    uint32_t r = a + b;  // < 2q < 2^32
    return min(r, r - q);
}

__device__ __forceinline__ uint32_t sub_mod(uint32_t a, uint32_t b, uint32_t q) { return fix_signed(a - b, q); }

// x * w mod q, (W, Wt) = (w*2^32 mod q, W*q^-1 mod 2^32); any x < 2^32.
__device__ __forceinline__ uint32_t mulc(uint32_t x, uint32_t W, uint32_t Wt, uint32_t q)
{
    uint32_t hi = __umulhi(x, W);
    uint32_t t = __umulhi(x * Wt, q);
    return fix_signed(hi - t, q);
}

__device__ __forceinline__ uint32_t mulc(uint32_t x, uint2 w, uint32_t q) { return mulc(x, w.x, w.y, q); }

// a*b*2^-32 mod q for a*b < q*2^32 (e.g. both canonical): the 64-bit product
// plus m q, m = -lo q^-1, is divisible by 2^32 with a quotient in [0, 2q)
// (a product and two multiply-adds, one correction).
__device__ __forceinline__ uint32_t mont(uint32_t a, uint32_t b, uint32_t q, uint32_t qinv)
{
    const uint64_t p = (uint64_t)a * b;
    const uint32_t m = (uint32_t)p * (0u - qinv);
    const uint32_t r = (uint32_t)((p + (uint64_t)m * q) >> 32);
    return min(r, r - q);
}

// A prime as the kernels use it: q, q^-1 mod 2^32, -q mod 2^32, round(2^32 / q).
struct PrimeC {
    uint32_t q, qinv, nq;
    int32_t rc;
};

// Product by a constant w, centred: the constant is the pair (w, ws) with w
// the centred representative (|w| < q/2) and ws = round(w 2^32 / q).  With
// e = round(x ws / 2^32) the result x w - e q has
//   |x w - e q| <= q/2 + |x| q / 2^33  (rounding of e, and of ws times x),
// so below 3q/4 for every 32-bit signed x: no correction, and the sign bit
// is kept for the sums that follow.  Three multiply-add instructions:
// v_mad_i64_i32 with 2^31 added in (its high word is e), v_mul_lo, and
// v_mad_u64_u32 with -q for the low word.
__device__ __forceinline__ int32_t round_quot(int32_t x, int32_t ws)
{
    return (int32_t)(((int64_t)x * ws + 0x80000000ll) >> 32);
}
__device__ __forceinline__ int32_t mulr(int32_t x, int2 w, uint32_t nq)
{
    return (int32_t)((uint32_t)round_quot(x, w.y) * nq + (uint32_t)x * (uint32_t)w.x);
}
// the same plus c (the multiply-add of x w takes it: no instruction more)
__device__ __forceinline__ uint32_t mulr_add(int32_t x, int2 w, uint32_t nq, uint32_t c)
{
    return (uint32_t)round_quot(x, w.y) * nq + ((uint32_t)x * (uint32_t)w.x + c);
}
// mulr by 1: any 32-bit signed x to its residue in (-3q/4, 3q/4)
__device__ __forceinline__ int32_t centre(int32_t x, const PrimeC& p)
{
    return (int32_t)((uint32_t)round_quot(x, p.rc) * p.nq + (uint32_t)x);
}
// The pair of a constant kept as ws alone: ws q = w 2^32 + d q with
// |d| <= 1/2, so w = round(ws q / 2^32) (one v_mad_i64_i32; q < 2^31).
__device__ __forceinline__ int2 const_from_quot(int32_t ws, uint32_t q)
{
    return make_int2(round_quot(ws, (int32_t)q), ws);
}

// [0, 2m) -> [0, m)
__device__ __forceinline__ uint32_t red2(uint32_t x, uint32_t m) { return min(x, x - m); }

// Signed Montgomery reduction: r = x 2^-32 (mod t) with |r| <= |x| / 2^32 +
// t / 2, below t for |x| <= t 2^31; odd t < 2^31, tinv = t^-1 mod 2^32.
// Why it works: m = x t^-1 mod 2^32, read as a signed 32-bit value, makes
// x - m t divisible by 2^32 and |m t| <= t 2^31.  One product and one 64-bit
// multiply-add, whose high word is the quotient. (Two instructions; the high words
// subtracted took eight, the compiler's 64-bit high product of a signed m.)
__device__ __forceinline__ int32_t smr64(int64_t x, uint32_t t, uint32_t tinv)
{
    const int32_t m = (int32_t)((uint32_t)x * tinv);
    return (int32_t)((x + (int64_t)m * (int64_t)(0 - (int32_t)t)) >> 32);
}

// (-t, t) -> [0, t)
__device__ __forceinline__ uint32_t canon_signed(int32_t y, uint32_t t) { return (uint32_t)(y < 0 ? y + (int32_t)t : y); }

// centred representative of v in [0, q): v if 2v < q else v - q
__device__ __forceinline__ int32_t lift(uint32_t v, uint32_t q) { return (int32_t)(v > (q >> 1) ? v - q : v); }

}  // namespace ckks
