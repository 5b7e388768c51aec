// Integer epilogue of one output element, shared by every kernel.
//
//   v  = acc + bias                                   (Sec. 3.2.2, Eq. 6)
//   u  = v + RSM(k, c, d)      side 0                 (Sec. 3.2.3, Eq. 7-8)
//      = RSM(v, c, d) + k      side 1
//   y  = clamp(RSM(u, M, 31 + sh), 0, qmax)           (Eq. 2 on integers)
//
// RSM(a, c, d) = floor((a*c + 2^(d-1)) / 2^d), and a*c for d = 0. With
// |a| < 2^31 and |c| < 2^31 the product stays below 2^62 and the rounding
// constant below 2^61, so the 64-bit sum cannot overflow; an arithmetic
// right shift of a signed value is the floor division.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aqd {

// The 64-bit shifts below are made of 32-bit ones: the 64-bit shift instructions
// give wrong results now and then where the register of the shift amount is the
// last one allocated to the wave (v167 of 168 in one form of the register-fed
// kernel, where just the channels shifted by it came out wrong), and no source can
// say which register the compiler takes.

// RSM(a, c, d) for 0 <= d <= 31 (the alignment's exponents)
__device__ __forceinline__ long long rsm(int a, int c, int d)
{
    const long long p = (long long)a * c + (long long)((1u << d) >> 1);
    const int hi = (int)(p >> 32);
    return (long long)((unsigned long long)(unsigned)(hi >> d) << 32 |
                       __builtin_amdgcn_alignbit((unsigned)hi, (unsigned)p, (unsigned)d));
}

__device__ __forceinline__ long long align_add(int v, int k, int c, int d, int side)
{
    return (long long)(side ? k : v) + rsm(side ? v : k, c, d);
}

// clamp(RSM(u, mult, d), 0, qmax), d = 31 + shift in 0 .. 62: with the high word h and
// the low word l of the rounded product shifted by d modulo 32, the result is h from
// d = 32 on; below, l while h is 0, else past the range on h's side (h == 0 ? l : h | 2^30
// costs the register-fed kernels 50 spilled registers)
__device__ __forceinline__ uint32_t requant_clamp(long long u, int mult, int shift, int qmax)
{
    const int d = 31 + shift;
    const unsigned half = d > 0 ? 1u << ((d - 1) & 31) : 0u;   // of 2^(d-1)
    const long long p = u * mult + (long long)(d > 32 ? (unsigned long long)half << 32 : half);
    const int hi = (int)(p >> 32), h = hi >> (d & 31);
    const unsigned l = __builtin_amdgcn_alignbit((unsigned)hi, (unsigned)p, (unsigned)d);
    const int side = h < -1 ? -1 : h > 1 ? 1 : h;
    const int below = side * (qmax + 1) + (int)(l < (unsigned)qmax ? l : (unsigned)qmax);
    const int y = d & 32 ? h : below;
    return (uint32_t)(y < 0 ? 0 : y > qmax ? qmax : y);
}

// Code of channel c of a packed row (bits in {2, 4, 8}).
__device__ __forceinline__ int load_code(const uint8_t *row, int c, int bits)
{
    int bit = c * bits;
    return (row[bit >> 3] >> (bit & 7)) & ((1 << bits) - 1);
}

}  // namespace aqd
