// fp32 numbers as three bf16 terms each, x = h + m + l, every term the rounded rest of the ones before it: all 24 bits of
// the mantissa (each rest is exact).  Internal.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ag {

// (A byte permutation: the compiler sees through a shift, and converts the number a second time instead, two instructions of
// thirteen a pair of weights.)
__device__ __forceinline__ float widen_lo(uint32_t pair) { return __builtin_bit_cast(float, __builtin_amdgcn_perm(pair, pair, 0x01000C0Cu)); }
__device__ __forceinline__ float widen_hi(uint32_t pair) { return __builtin_bit_cast(float, pair & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack(float a, float b)
{
    typedef __bf16 pair __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, pair{(__bf16)a, (__bf16)b});
}

// The leading terms of two numbers, packed; a and b become their rests.
__device__ __forceinline__ uint32_t take_term(float& a, float& b)
{
    const uint32_t t = pack(a, b);
    a -= widen_lo(t);
    b -= widen_hi(t);
    return t;
}

// Two numbers as packed terms.  Both halves of a packed term are widened by one instruction each (left to itself the
// compiler converts every number a second time).  An infinity (or what rounds to one) leaves NaN as its rest.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = take_term(a, b);
    m = take_term(a, b);
    l = pack(a, b);
}

// Eight numbers as packed terms: operands of a 16-bit product, smallest terms first when they are summed.
struct Terms {
    typedef uint32_t words __attribute__((ext_vector_type(4)));
    words h, m, l;
    __device__ __forceinline__ void set_pair(int i, float a, float b)          // numbers 2 i and 2 i + 1
    {
        uint32_t hh, mm, ll;
        split_pair(a, b, hh, mm, ll);
        h[i] = hh;
        m[i] = mm;
        l[i] = ll;
    }
};

// ---- fp32 products as six products of terms (attn_prefill_f32.hip, attn_prefill_split.hip) ----
constexpr float kLargeQuery = 0x1p90f;  // scale * |q| up to which what small keys lose (2^-126, times 128 channels) is nothing

// The smallest size among numbers, zero left out because it is exact: of 2 |bits| - 1, where zero comes out largest.
struct Least {
    uint32_t u = ~0u;
    __device__ __forceinline__ void take(float x) { u = min(u, (__builtin_bit_cast(uint32_t, x) << 1) - 1); }
    __device__ __forceinline__ bool small(float unit = 1.f) const        // (no number but zeros: NaN)
    {
        return __builtin_bit_cast(float, u >> 1) * unit < 0x1p-100f;
    }
};

constexpr float kWeightUnit = 0x1p48f;  // what a weight of 1 is multiplied as; their sum is in the same unit

typedef float Four __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Terms split8(const Four& a, const Four& b)
{
    Terms t;
#pragma unroll
    for (int i = 0; i < 4; ++i) t.set_pair(i, i < 2 ? a[2 * i] : b[2 * i - 4], i < 2 ? a[2 * i + 1] : b[2 * i - 3]);
    return t;
}

}  // namespace ag
