// The compact tile list of the prefill kernels: which (KV head, tile number) a workgroup takes, and which (session, query tile)
// tile number j of a KV head is.  Internal.
#pragma once

#include <algorithm>

#include "ag_internal.h"
#include "find_session.h"

namespace ag {

// Workgroups land on XCD blockIdx.x % 8.  KV heads are dealt to the XCDs, so that a head's keys and values stay in the L2s of
// few: 8 / gcd(heads, 8) XCDs share a set of heads and its list of tiles, longest context first (find_tile()).  While an XCD's part
// of the list fits it at once, each takes one run of it, whose keys are the fewest sessions'.  A longer list is dealt in turn, in
// runs of up to four tiles of a session (eight runs an XCD at least): in one run each, the XCD with the longest contexts, or with the ends
// of the prompts, ends long after the others - but for prompts of one length that come out even, where a run is whole prompts and
// begins with their longest tiles.  Graph replay, append included, one run -> dealt, us: 16 / 1 heads x 128, 26 chunks of 4..732
// rows on 133..6759 tokens 381 -> 228, three prompts of 99..3867 138 -> 81; 8 / 2 six of 39..3985 160 -> 109; 16 / 2, 31 of about 200 on
// 1418..5227 262 -> 187, 23 of 7..31 on 1190..1378 28.8 -> 19.5 (single tiles 25.2), fp32 x 64 eleven of 209..472 on 461..2721 331 -> 222;
// 6 / 2 x 256 13 of 150..850 83 -> 61; but 16 / 2 four prompts of 1151..1419 46.6 -> 50.7.  Where it fits, dealt: 6 / 2, 23 of 26..57 on 892..6241
// 39.9 -> 55.4, 16 / 1, 15 of 9..54 on 365..817 14.1 -> 16.1, but 16 / 2 pages of 32, 12 of 12..385 on 306..2893 138 -> 111.  Over 130 and over 110
// drawn batches of heads that eight does not divide 1.073 and 1.069 on average (runs of eight 1.066, of a sixteenth of the list 1.068, single tiles always 1.060).
struct Deal {
    int tiles_max;          // tiles of a KV head, a bound
    int items;              // tiles of a set of heads
    int share;              // log2 of the XCDs that share a set
    int run;                // consecutive tiles that go to one XCD
};

// at_once: workgroups of an XCD that are resident together
inline Deal deal_of(const AttnArgs& a, int64_t tiles_max, int at_once)
{
    int share = 3;
    while (share > 0 && a.c.hkv % (16 >> share) == 0) --share;
    const int64_t heads = a.c.hkv >> (3 - share), items = heads * tiles_max, part = (items + (1 << share) - 1) >> share;
    const int64_t prompts = heads * a.batch, each = (prompts + (1 << share) - 1) >> share;
    const bool even = a.max_ctx == a.max_new && 5 * (int64_t)a.total_rows >= 4 * (int64_t)a.batch * a.max_new && 7 * prompts >= 6 * (each << share);
    const int64_t session = (tiles_max + a.batch - 1) / a.batch;
    const int64_t run = share == 0 || part <= at_once || even ? part : std::max<int64_t>(1, std::min({session, part / 8, (int64_t)4}));
    return Deal{(int)tiles_max, (int)items, share, (int)run};
}
// At most kDealtPast more than there are tiles: a last round of runs of four on eight XCDs, or of one on each.
constexpr int kDealtPast = 32;
inline int64_t workgroups_of(const Deal& d)
{
    const int64_t round = (int64_t)d.run << d.share;
    return 8 * ((d.items + round - 1) / round) * d.run;
}

__device__ __forceinline__ bool place_of(const Deal& d, int hkv, int& g, int& j)
{
    const unsigned xcd = blockIdx.x & 7, ord = blockIdx.x >> 3, run = (unsigned)d.run;
    unsigned before = 0, head = 0;              // runs this XCD has taken; divisions only where they are needed
    if (ord >= run) before = ord / run;
    const unsigned k = ((before << d.share) + (xcd & ((1u << d.share) - 1)) - before) * run + ord;
    if (k >= (unsigned)d.items) return false;
    if (k >= (unsigned)d.tiles_max) head = k / (unsigned)d.tiles_max;
    g = (int)(xcd >> d.share) * (hkv >> (3 - d.share)) + (int)head;
    j = (int)(k - head * (unsigned)d.tiles_max);
    return true;
}

// Tiles of C columns, G columns a row.  s stays -1 when tile j is nobody's; otherwise s, its tile qt (the session's tiles
// count down: longest context first), its lengths N and P and its first row row0.
// Up to 64 sessions: every wave scans the lengths for itself, and the tiles are numbered without gaps.  More: find_session().
template <int C>
__device__ __forceinline__ void find_tile(const AttnArgs& a, int j, int G, int& s, int& qt, int& N, int& P, int& row0)
{
    auto tiles_of = [G](int len) { return (int)(((int64_t)len * G + C - 1) / C); };
    if (a.batch > 64) {
        // the host's two bounds on the tiles of a batch (tiles_bound() in the kernels' files), for the sessions before s
        const int most = tiles_of(a.max_new);
        const Session f = find_session(a.new_lens, a.prefix_lens, a.cu_new, a.batch, j, [G, most](int ss, int cu) {
            return (int)min((int64_t)cu * G / C + ss, (int64_t)ss * most);
        });
        const int tiles = tiles_of(f.new_len), k = j - f.first;
        if (k >= tiles) return;                 // uniform
        // Put into scalar registers by hand: the compiler does not see that the search is uniform, and what it then keeps per
        // lane spilled 4 VGPRs in the widened 8-wave kernel of 128 channels (8 chunks of 2048, pages of 32: 524 -> 565 us).
        s = __builtin_amdgcn_readfirstlane(f.s);
        N = __builtin_amdgcn_readfirstlane(f.new_len);
        P = __builtin_amdgcn_readfirstlane(f.prefix);
        row0 = __builtin_amdgcn_readfirstlane(f.row0);
        qt = __builtin_amdgcn_readfirstlane(tiles - 1 - k);
        return;
    }
    // the lengths are fetched together with the prefix length and the row offset of every session: whichever session the
    // tile turns out to belong to, no second round trip follows
    const int ln = threadIdx.x & 63;
    const bool in = ln < a.batch;
    int len = in ? a.new_lens[ln] : 0, pre = in && a.prefix_lens ? a.prefix_lens[ln] : 0, cu = in ? a.cu_new[ln] : 0;
    // The batch is walked longest context first: workgroups start in list order, and a launch ends sooner when the tiles
    // left for its end are the short ones (each has P + position keys to go through).  Every wave ranks the sessions
    // itself; equal contexts keep the given order.
    int sess = ln;                              // the session this lane's entry describes
    const int key = in ? pre + len : -1;
    const int key0 = __builtin_amdgcn_readlane(key, 0);
    if (__builtin_amdgcn_ballot_w64(in && key != key0) != 0) {       // uniform
        int rank = 0;                           // sessions ahead of this one: longer, or as long and earlier
        for (int o = 0; o < a.batch; ++o) {
            const int ko = __builtin_amdgcn_readlane(key, o);
            rank += (ko > key || (ko == key && o < ln)) ? 1 : 0;
        }
        if (!in) rank = ln;                     // entries without a session stay where they are
        sess = __builtin_amdgcn_ds_permute(rank << 2, sess);
        len = __builtin_amdgcn_ds_permute(rank << 2, len);
        pre = __builtin_amdgcn_ds_permute(rank << 2, pre);
        cu = __builtin_amdgcn_ds_permute(rank << 2, cu);
    }
    int incl = tiles_of(len);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(incl, d);
        if (ln >= d) incl += t;
    }
    if (j < __builtin_amdgcn_readlane(incl, 63)) {                   // uniform
        const int l = __builtin_ctzll(__builtin_amdgcn_ballot_w64(j < incl));    // first session whose tiles reach past j
        s = __builtin_amdgcn_readlane(sess, l);
        N = __builtin_amdgcn_readlane(len, l);
        P = __builtin_amdgcn_readlane(pre, l);
        row0 = __builtin_amdgcn_readlane(cu, l);
        qt = __builtin_amdgcn_readlane(incl, l) - 1 - j;             // the session's tiles, longest first
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
