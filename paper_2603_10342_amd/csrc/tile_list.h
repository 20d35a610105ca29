// The compact tile list of the prefill kernels: which (session, query tile) tile number j of a KV head is.  Internal.
#pragma once

#include "ag_internal.h"

namespace ag {

// Every wave scans the batch's lengths for itself (lane l of a pass holds session 64 * pass + l); tiles_of(len) is the
// number of tiles a chunk of len rows is cut into.  s stays -1 when j lies beyond the batch's tiles; otherwise s, its
// tile qt (the session's tiles count down: longest context first), its lengths N and P and its first row row0.
template <class TilesOf>
__device__ __forceinline__ void find_tile(const AttnArgs& a, int j, TilesOf tiles_of, int& s, int& qt, int& N, int& P, int& row0)
{
    const int ln = threadIdx.x & 63;
    int before = 0;                             // tiles of the sessions of earlier passes
    for (int s0 = 0; s0 < a.batch && s < 0; s0 += 256) {
        // four passes' lengths are fetched together, and with them the prefix length and the row offset of
        // every session: whichever session the tile turns out to belong to, no second round trip follows
        int lens[4], pre[4], cu[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int ss = s0 + 64 * k + ln;
            const bool in = ss < a.batch;
            lens[k] = in ? a.new_lens[ss] : 0;
            pre[k] = in && a.prefix_lens ? a.prefix_lens[ss] : 0;
            cu[k] = in ? a.cu_new[ss] : 0;
        }
        // A batch that fits one pass is walked longest context first: workgroups start in list order, and a
        // launch ends sooner when the tiles left for its end are the short ones (each has P + position keys
        // to go through).  Every wave ranks the sessions itself; equal contexts keep the given order.
        int sess = ln;                          // the session this lane's entry describes
        if (a.batch <= 64) {
            const int key = ln < a.batch ? pre[0] + lens[0] : -1;
            const int key0 = __builtin_amdgcn_readlane(key, 0);
            if (__builtin_amdgcn_ballot_w64(ln < a.batch && key != key0) != 0) {       // uniform
                int rank = 0;                   // sessions ahead of this one: longer, or as long and earlier
                for (int o = 0; o < a.batch; ++o) {
                    const int ko = __builtin_amdgcn_readlane(key, o);
                    rank += (ko > key || (ko == key && o < ln)) ? 1 : 0;
                }
                if (ln >= a.batch) rank = ln;   // entries without a session stay where they are
                sess = __builtin_amdgcn_ds_permute(rank << 2, sess);
                lens[0] = __builtin_amdgcn_ds_permute(rank << 2, lens[0]);
                pre[0] = __builtin_amdgcn_ds_permute(rank << 2, pre[0]);
                cu[0] = __builtin_amdgcn_ds_permute(rank << 2, cu[0]);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (s >= 0) break;                  // uniform
            const int len = lens[k];
            const int cnt = tiles_of(len);
            int incl = cnt;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int t = __shfl_up(incl, d);
                if (ln >= d) incl += t;
            }
            const int pass_total = __builtin_amdgcn_readlane(incl, 63);
            if (j < before + pass_total) {      // uniform
                const unsigned long long hit = __builtin_amdgcn_ballot_w64(j < before + incl);
                const int l = __builtin_ctzll(hit);              // first session whose tiles reach past j
                s = s0 + 64 * k + (k == 0 ? __builtin_amdgcn_readlane(sess, l) : l);
                N = __builtin_amdgcn_readlane(len, l);
                P = __builtin_amdgcn_readlane(pre[k], l);
                row0 = __builtin_amdgcn_readlane(cu[k], l);
                qt = before + __builtin_amdgcn_readlane(incl, l) - 1 - j;   // the session's tiles, longest first
            }
            before += pass_total;
        }
    }
}

// Columns of a (session, KV head): number token * G + head.  A workgroup's columns start at col0 (total_rows * G fits an
// int); token and head of a column are found from those of col0 with one multiplication - a 64-bit division for each of the
// handful a workgroup needs took 1 % of a long prefill.
struct Columns {
    int t0, r0, G;          // token of col0, its head
    float inv;
    __device__ __forceinline__ Columns(int col0, int G_) : t0((unsigned)col0 / (unsigned)G_), r0(col0 - t0 * G_), G(G_), inv(1.0f / (float)G_) {}
    // exact: r0 + col < G + 256, and half a column is far more than the product's rounding
    __device__ __forceinline__ int token(int col) const { return t0 + (int)(((float)(r0 + col) + 0.5f) * inv); }
    __device__ __forceinline__ int head(int col, int token) const { return r0 + col - (token - t0) * G; }
};

}  // namespace ag
