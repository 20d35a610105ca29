// One (row, query head) of paged attention by one wave, in fp32 arithmetic: the general kernel's work, and what kernels for
// the same shapes fall back on where their result is not finite.  Internal.
#pragma once

#include "ag_internal.h"

namespace ag {
namespace general {

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(__bf16 x) { return (float)x; }
__device__ __forceinline__ void store_out(float* p, float x) { *p = x; }
__device__ __forceinline__ void store_out(__bf16* p, float x) { *p = (__bf16)x; }   // round to nearest even

__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}
__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// Row t (session s, position pos), query head h; s_q: 256 floats of LDS private to this wave.
template <typename T>
__device__ __forceinline__ void attend_row(const AttnArgs& a, int64_t t, int h, int s, int pos, float* s_q)
{
    const int lane = threadIdx.x & 63;
    const int D = a.c.d, ps = a.c.ps, hkv = a.c.hkv;
    const int g = h / (a.hq / hkv);
    T* out = (T*)a.out + (t * a.hq + h) * D;
    if (pos < 0) {                        // empty context: defined as a row of zeros
        for (int d = lane; d < D; d += 64) store_out(out + d, 0.0f);
        return;
    }

    const T* q = (const T*)a.q + (t * a.hq + h) * D;
    for (int d = lane; d < D; d += 64) s_q[d] = to_f32(q[d]);
    __builtin_amdgcn_wave_barrier();      // s_q is private to this wave

    const T* kp = (const T*)a.c.k;
    const T* vp = (const T*)a.c.v;
    const int32_t* bt = a.bt + (int64_t)s * a.max_pages;

    float m = -INFINITY, l = 0.0f;
    float o[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // channels lane, lane+64, lane+128, lane+192

    for (int base = 0; base <= pos; base += 64) {
        const int j = base + lane;
        const bool valid = j <= pos;
        int64_t page = 0;
        int slot = 0;
        float x = -INFINITY;
        if (valid) {
            page = bt[j >> a.c.ps_shift];
            slot = j & (ps - 1);
            const T* kr = kp + (page * hkv + g) * (int64_t)D * ps + slot * 8;   // chunk c of this slot: + c * ps * 8
            float dot = 0.0f;
            for (int d = 0; d < D; ++d) dot = fmaf(s_q[d], to_f32(kr[(int64_t)(d >> 3) * ps * 8 + (d & 7)]), dot);
            x = a.scale * dot;
        }
        const float m_new = fmaxf(m, wave_max(x));      // finite: lane 0 of every block is valid
        const float alpha = expf(m - m_new);            // exp(-inf) = 0 on the first block
        const float p = valid ? expf(x - m_new) : 0.0f;
        l = l * alpha + wave_sum(p);
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] *= alpha;
        const int cnt = min(64, pos - base + 1);
        for (int jj = 0; jj < cnt; ++jj) {
            const float pj = __shfl(p, jj);
            const int64_t pg = __shfl((int)page, jj);
            const int sl = __shfl(slot, jj);
            const T* vr = vp + (pg * hkv + g) * (int64_t)D * ps;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int d = lane + 64 * c;
                if (d < D) o[c] = fmaf(pj, to_f32(vr[v_offset(sl, d, ps, D)]), o[c]);
            }
        }
        m = m_new;
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int d = lane + 64 * c;
        if (d < D) store_out(out + d, o[c] * inv);
    }
}

// For kernels that multiply whole tiles: an infinity or NaN among the values of a tile turns the columns that may not see it
// into NaN too (0 x inf), and terms of split numbers can turn an infinite result into NaN.  Columns whose result is not
// finite are therefore taken again, one at a time, in plain arithmetic, and give what they would have given.
// Bit c of `again` (uniform over the wave): row `rows` of lane c, a row of Q as t * hq + head, of session s, whose first
// row of Q is row0 at position P.
template <typename T>
__device__ __forceinline__ void attend_rows_again(const AttnArgs& a, uint64_t again, int64_t rows, int s, int row0, int P, float* s_q)
{
    while (again) {
        const int c = __builtin_ctzll(again);
        again &= again - 1;
        const int64_t row = ((int64_t)__builtin_amdgcn_readlane((int)(rows >> 32), c) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)rows, c);
        const int64_t t = row / a.hq;
        attend_row<T>(a, t, (int)(row - t * a.hq), s, P + (int)(t - row0), s_q);
    }
}

// NaN unless x is finite; sums of it stay NaN.
__device__ __forceinline__ float trouble_of(float x, float sum = 0.f) { return fmaf(x, 0.f, sum); }

}  // namespace general
}  // namespace ag
