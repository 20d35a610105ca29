// A pair of fp32 weights as two bf16 terms each, hi + lo: 16 bits of mantissa where one term has 8.  Internal.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ag {

typedef __bf16 bf16_pair __attribute__((ext_vector_type(2)));

// What lo leaves of p: p - hi in bf16.  Both halves of the packed hi are widened by one instruction each (left to itself
// the compiler converts every weight a second time, 64 conversions a tile of 32 weights instead of 32).
__device__ __forceinline__ bf16_pair low_terms(float p0, float p1, bf16_pair hi)
{
    const uint32_t bits = __builtin_bit_cast(uint32_t, hi);
    return bf16_pair{(__bf16)(p0 - __builtin_bit_cast(float, bits << 16)), (__bf16)(p1 - __builtin_bit_cast(float, bits & 0xFFFF0000u))};
}

}  // namespace ag
