// Which session of a batch an item number belongs to.  Internal.
#pragma once

#include "ag_internal.h"

namespace ag {

struct Session { int s, new_len, prefix, row0, first; };         // first: its first item

// Sessions are given item numbers that follow from their place and row offset alone, first_of(s, cu_new[s]), nondecreasing in
// s with first_of(0, 0) = 0, each session at least as many as it has items: so that no lengths have to be added up, and a wave
// finds the last session that starts at or before the item with 64 lanes a step, one memory round trip for up to 64 sessions
// and two for up to 4096.  Uniform over the wave.  (A scan of the lengths is a round trip and six cross-lane steps for every 64
// sessions: an append of four tokens by groups to each of 2048 sessions, 8 KV heads x 128, 237 -> 42 us.)
template <class FirstOf>
__device__ __forceinline__ Session find_session(const int32_t* __restrict__ new_lens, const int32_t* __restrict__ prefix_lens,
                                                const int32_t* __restrict__ cu_new, int batch, int item, FirstOf first_of)
{
    const int lane = threadIdx.x & 63;
    int lo = 0, len = batch;                    // the session lies in [lo, lo + len)
    while (len > 64) {
        const int stride = (len + 63) >> 6;
        const int at = lane * stride, s = lo + at;
        const bool starts = at < len && first_of(s, at < len ? cu_new[s] : 0) <= item;
        const int n = max(__builtin_popcountll(__builtin_amdgcn_ballot_w64(starts)) - 1, 0);
        lo += n * stride;
        len = min(stride, len - n * stride);
    }
    const int s = lo + lane;
    const bool in = lane < len;
    const int cu = in ? cu_new[s] : 0, n = in ? new_lens[s] : 0, p = in && prefix_lens ? prefix_lens[s] : 0;
    const int first = first_of(s, cu);
    const int l = max(__builtin_popcountll(__builtin_amdgcn_ballot_w64(in && first <= item)) - 1, 0);
    return Session{lo + l, __builtin_amdgcn_readlane(n, l), __builtin_amdgcn_readlane(p, l), __builtin_amdgcn_readlane(cu, l),
                   __builtin_amdgcn_readlane(first, l)};
}

}  // namespace ag
