// One (row, query head) of paged attention by one wave, in fp32 arithmetic: the general kernel's work; and the same for
// several rows at once, which kernels for the same shapes fall back on where their result is not finite.  Internal.
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
// finite are therefore taken again, in plain arithmetic, and give what they would have given: attend_row()'s numbers bit
// for bit, for caches with pages of 16 tokens or more and 16-byte aligned pools (whose layout allows 16-byte loads).
// R rows of one session and KV head share a pass over its keys and values, because whoever sees one value that is not
// finite is seldom alone: every later row of the session does.
// s_q: R * D floats of LDS private to this wave; C: 64-channel blocks of head_dim.
template <typename T, int R, int C>
__device__ __forceinline__ void attend_rows(const AttnArgs& a, const int64_t (&rows)[R], const int (&pos)[R], int s, int g, float* s_q)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int kVecs = (int)sizeof(T) / 2;             // 16-byte loads of 8 numbers
    union Eight { u32x4 u[kVecs]; T e[8]; };
    const int lane = threadIdx.x & 63;
    const int D = a.c.d, ps = a.c.ps, hkv = a.c.hkv;
    const int64_t block = (int64_t)D * ps;
    const T* kp = (const T*)a.c.k;
    const T* vp = (const T*)a.c.v;
    const int32_t* bt = a.bt + (int64_t)s * a.max_pages;
    auto load8 = [](Eight& x, const T* p) {
#pragma unroll
        for (int i = 0; i < kVecs; ++i) x.u[i] = reinterpret_cast<const u32x4*>(p)[i];
    };
    int last = pos[0];
#pragma unroll
    for (int r = 1; r < R; ++r) last = max(last, pos[r]);
    float m[R], l[R], o[R][C];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        for (int d = lane; d < D; d += 64) s_q[r * D + d] = to_f32(((const T*)a.q)[rows[r] * D + d]);
        m[r] = -INFINITY;
        l[r] = 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c) o[r][c] = 0.f;
    }
    __builtin_amdgcn_wave_barrier();                      // s_q is private to this wave

#pragma unroll 1
    for (int base = 0; base <= last; base += 64) {
        const int j = base + lane, at = min(j, last);     // lane = key
        const int page = bt[at >> a.c.ps_shift];
        const T* kr = kp + ((int64_t)page * hkv + g) * block + (at & (ps - 1)) * 8;
        float dot[R];
#pragma unroll
        for (int r = 0; r < R; ++r) dot[r] = 0.f;
#pragma unroll 4
        for (int c = 0; c < D / 8; ++c) {
            Eight k;
            load8(k, kr + (int64_t)c * ps * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int r = 0; r < R; ++r) dot[r] = fmaf(s_q[r * D + c * 8 + e], to_f32(k.e[e]), dot[r]);
        }
        float p[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            p[r] = 0.f;
            if (base > pos[r]) continue;                  // uniform: the row has ended
            const float x = j <= pos[r] ? a.scale * dot[r] : -INFINITY;
            const float m_new = fmaxf(m[r], wave_max(x));
            const float alpha = expf(m[r] - m_new);
            p[r] = j <= pos[r] ? expf(x - m_new) : 0.f;
            l[r] = l[r] * alpha + wave_sum(p[r]);
#pragma unroll
            for (int c = 0; c < C; ++c) o[r][c] *= alpha;
            m[r] = m_new;
        }
#pragma unroll 1
        for (int first = base; first < base + 64 && first <= last; first += 16) {       // lane = channel, a 16-token group at a time
            const int64_t pg = __builtin_amdgcn_readlane(page, first - base);
            const T* vr = vp + (pg * hkv + g) * block + (int64_t)((first & (ps - 1)) >> 4) * 16 * D;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (64 * c >= D) break;                   // uniform
                Eight v[2];                               // keys 0..3 and 8..11 of the group, keys 4..7 and 12..15 (v_offset)
#pragma unroll
                for (int h = 0; h < 2; ++h) load8(v[h], vr + (h * D + min(lane + 64 * c, D - 1)) * 8);
#pragma unroll
                for (int i = 0; i < 16; ++i)
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        if (first + i > pos[r]) continue; // uniform
                        const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, p[r]), first - base + i));
                        o[r][c] = fmaf(w, to_f32(v[(i >> 2) & 1].e[(i & 3) + (i >> 3) * 4]), o[r][c]);
                    }
                __builtin_amdgcn_sched_barrier(0);        // one block of channels at a time: registers, of which the callers have few
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float inv = 1.0f / l[r];
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (lane + 64 * c < D) store_out((T*)a.out + rows[r] * D + lane + 64 * c, o[r][c] * inv);
    }
}

// Bit c of `again` (uniform over the wave): row `row` of lane c, a row of Q as t * hq + head, of session s and KV head g, at
// position `pos` of lane c.
template <typename T, int R, int C>
__device__ __forceinline__ void attend_rows_again(const AttnArgs& a, uint64_t again, int64_t row, int pos, int s, int g, float* s_q)
{
    while (again) {
        int64_t rows[R];
        int at[R], c = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {                     // (fewer than R are left: the last one once more)
            if (again) c = __builtin_ctzll(again);
            again &= again - 1;
            rows[r] = ((int64_t)__builtin_amdgcn_readlane((int)(row >> 32), c) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)row, c);
            at[r] = __builtin_amdgcn_readlane(pos, c);
        }
        attend_rows<T, R, C>(a, rows, at, s, g, s_q);
    }
}

// NaN unless x is finite; sums of it stay NaN.
__device__ __forceinline__ float trouble_of(float x, float sum = 0.f) { return fmaf(x, 0.f, sum); }

}  // namespace general
}  // namespace ag
