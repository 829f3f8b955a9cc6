// How the products of the language-model head are divided: rows into chunks, a product into tiles, parts and
// work items.  Plain integer arithmetic on sizes, the same on the host and on the device (lmhead.hpp uses it
// in its kernels; a host compiler takes it alone).
#pragma once

#include <climits>

#ifndef __HIP__
#define __host__
#define __device__
#endif

namespace {

constexpr int LM_BM = 256, LM_BN = 256, LM_BK = 64;  // tile of C, K step
constexpr int LM_GROUP_M = 8;                        // tile rows that share a sweep along N
constexpr int LM_SPLIT_MAX = 64;                     // parts the contraction of one tile of dL/dH may be cut into

// Which of n_live rows chunk number `chunk` covers when no chunk may hold more than cap rows
// (cap a multiple of 256): the fewest chunks that can hold them, each of the same size rounded
// up to whole 256-row tiles.  Chunks beyond those are empty (count 0).
__host__ __device__ inline void lm_chunk_range(int n_live, int cap, int chunk, int &base, int &count)
{
    const int needed = (n_live + cap - 1) / cap;
    if (chunk >= needed) {
        base = n_live;
        count = 0;
        return;
    }
    const int per = ((n_live + needed - 1) / needed + 255) / 256 * 256;  // <= cap
    base = chunk * per;  // < n_live: (needed - 1) cap < n_live and per <= cap
    count = n_live - base < per ? n_live - base : per;
}

// Workgroup -> tile.  The hardware deals consecutive workgroups to the 8 XCDs in turn;
// each XCD has its own L2.  Workgroups of one XCD are given a contiguous run of the
// tile order below, and that order walks LM_GROUP_M tile rows down before it moves one
// tile column on, so the tiles in flight on an XCD at any moment share a few A and B
// panels and most operand traffic is served by that XCD's L2.  The number of tile rows
// comes from the device-side row count, so that the live tiles are spread over all XCDs
// whatever part of the launched grid they are.
__host__ __device__ inline void lm_tile_of(int L, int tiles_m, int tiles_n, int &tm, int &tn)
{
    const int group_tiles = LM_GROUP_M * tiles_n;
    const int grp = L / group_tiles;
    const int in_grp = L - grp * group_tiles;
    const int left = tiles_m - grp * LM_GROUP_M, rows_here = left < LM_GROUP_M ? left : LM_GROUP_M;
    tm = grp * LM_GROUP_M + in_grp % rows_here;
    tn = in_grp / rows_here;
}

// The work of one product.  A tile row of C whose live rows do not reach past its first 128 (the last one, as often
// as not) is "thin": the lower four wavefronts, which share their SIMDs with the upper four, skip its products, and it
// takes about 0.55 of a whole tile's time.  Whole tiles come first, in the order of lm_tile_of, thin ones behind
// them, so that the workgroups that got one whole tile less than the others take the first of them - two each,
// as far as there are more than these workgroups (640 rows of a vocabulary of 50304: 394 whole tiles and 197 thin ones, at
// most 2 and none or 1 and 2 for a workgroup, not 2 and 1: a call with 768 values a row 312 and 302 us).
//
// Whole tiles that do not fill a round of the CUs (780 tiles on 256 CUs: three rounds and twelve tiles) would run that
// round on a few CUs, each for a whole tile's time.  Two ways out, for the `rest` tiles behind the last whole round:
//  - where the contraction may be split (dL/dH), each is cut into s2 parts along it, so that the last round is s2 times
//    shorter and spread over all CUs, and thin tiles into t2 = half as many, so that all parts take the same time.
//    The number of parts minimises lm_split_cost.  Every workgroup of the product, and lm_split_reduce, which reads the
//    blocks that the parts have written, computes the plan anew from the same numbers: in whole numbers, so that all of
//    them, and the host, come to the same one whatever a compiler makes of each place.
//  - else each is cut into its upper and lower 128 rows, two thin tiles, if all thin tiles then fit one round.
struct LmPlan {
    int rows_w, has_thin;  // whole tile rows; 1 if a thin one follows
    int full;              // whole tiles computed as they are
    int rest, s2;          // whole tiles cut into s2 parts each along the contraction
    int halves;            // whole tiles cut into two thin ones
    int thin, t2;          // tiles of the thin tile row, and the parts each is cut into
    int pairs;             // of each XCD's list of thin tiles: how many places at its beginning hold two
};
// What `over` whole and `thin` thin tiles of k_tiles K steps cost with S parts to a whole one and T to a thin one (1 and 1: not
// cut): nanoseconds to rank the parts of one product by, not its time.  A K step is 1200 in a whole tile, 700 in a thin
// one; a part 6000 more; its 256 KB of fp32 results (128 KB of a thin tile), written and read again, 40 each 128 KB.  That is
// a K step with operands in the caches at a clock that short products hold; the whole chip at it for milliseconds lowers
// its clock to 1610 (1949 rows of 152064 x 5120: 2385 us and 72 for the sum, 1914 by this; 612 of 50304 x 768: 60 and 12,
// and 52).  Which number of parts wins is a matter of rounds, which all take the same clock: 128 rows of 152064 x 1024,
// 510 us a call with an earlier rule, take 341.
__host__ __device__ inline long long lm_split_cost(int S, int T, int over, int thin, int k_tiles, int max_items, int n_cu)
{
    const int items = over * S + thin * T;
    if (S > 1 && items > max_items) return LLONG_MAX;
    const int per_xcd = n_cu >= 8 ? n_cu / 8 : 1, longest = (over * S + 7) / 8 + (thin * T + 7) / 8;  // see lm_map_item
    // (k_tiles <= 2^17: see lm_bwd_vocab_ok)
    const unsigned one = over > 0 ? 1200u * (unsigned)k_tiles / (unsigned)S : 700u * (unsigned)k_tiles / (unsigned)T;
    return (long long)((longest + per_xcd - 1) / per_xcd) * (one + 6000u) + (S > 1 ? 40ll * (2 * over * S + thin * T) : 0);
}
// The candidates are S = 1 .. LM_SPLIT_MAX parts of 8 K steps or more to a whole tile and half as many to a thin one, which then
// take the same time; where there are only thin tiles, S is theirs.
__host__ __device__ inline int lm_split_thin_parts(int S, int over) { return over > 0 ? (S + 1) / 2 : S; }
__host__ __device__ inline long long lm_split_candidate(int S, int over, int thin, int k_tiles, int max_items, int n_cu)
{
    if (S > 1 && S > k_tiles / 8) return LLONG_MAX;
    return lm_split_cost(S, lm_split_thin_parts(S, over), over, thin, k_tiles, max_items, n_cu);
}
__host__ __device__ inline bool lm_split_better(long long cost, int S, long long than_cost, int than_S)
{
    return cost < than_cost || (cost == than_cost && S < than_S);
}
__host__ __device__ inline LmPlan lm_plan(int M, int tiles_n, int k_tiles, bool split, int max_items, int n_cu)
{
    LmPlan pl;
    const int tail = M % LM_BM;
    pl.has_thin = tail > 0 && tail <= LM_BM / 2 ? 1 : 0;
    pl.rows_w = M / LM_BM + (tail > LM_BM / 2 ? 1 : 0);
    pl.thin = pl.has_thin * tiles_n;
    pl.full = pl.rows_w * tiles_n;
    pl.rest = pl.halves = 0;
    pl.s2 = pl.t2 = 1;
    pl.pairs = 0;
    const int over = pl.full % n_cu;
    if (!split) {
        if (over > 0 && 2 * over + pl.thin <= n_cu) {
            pl.halves = over;
            pl.full -= over;
        } else if (n_cu >= 8) {
            const int per_xcd = n_cu / 8, left = ((pl.full + 7) / 8) % per_xcd, free = left > 0 ? per_xcd - left : 0;
            const int more = (pl.thin + 7) / 8 - free;
            pl.pairs = more <= 0 ? 0 : more < free ? more : free;
        }
        return pl;
    }
    if (over + pl.thin == 0) return pl;
    int s_best = 1;
#ifdef __HIP_DEVICE_COMPILE__
    // a lane to a candidate (64 of them one after the other are 5 us)
    static_assert(LM_SPLIT_MAX == 64, "one candidate for each lane");
    s_best = (int)(threadIdx.x & 63) + 1;
    long long c = lm_split_candidate(s_best, over, pl.thin, k_tiles, max_items, n_cu);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long c2 = __shfl_xor(c, o, 64);
        const int s2 = __shfl_xor(s_best, o, 64);
        if (lm_split_better(c2, s2, c, s_best)) c = c2, s_best = s2;
    }
    s_best = __builtin_amdgcn_readfirstlane(s_best);
#else
    long long best = lm_split_candidate(1, over, pl.thin, k_tiles, max_items, n_cu);
    for (int S = 2; S <= LM_SPLIT_MAX; ++S) {
        const long long c = lm_split_candidate(S, over, pl.thin, k_tiles, max_items, n_cu);
        if (lm_split_better(c, S, best, s_best)) best = c, s_best = S;
    }
#endif
    if (s_best == 1) return pl;
    pl.rest = over;
    pl.full -= over;
    pl.s2 = s_best;
    pl.t2 = lm_split_thin_parts(s_best, over);
    return pl;
}

// Work item -> tile, part and height.  Each XCD takes a contiguous run of each list - whole tiles, parts or halves
// of the rest, thin tiles - so that all kinds of work are spread evenly over the XCDs; parts are ordered part by
// part (the same K range of neighbouring tiles shares operand panels).
// idx: position in the XCD's lists, below lm_items_per_xcd; false: no work at that position.
struct LmItem {
    int row0, tn;     // first row, tile column
    int height;       // 256, or 128 for a thin item
    int part, parts;  // which part of the contraction
    int block;        // parts > 1: index of its fp32 block
    int pair;         // 1: the same place holds the thin tile of the next column too
};
__host__ __device__ inline int lm_items_per_xcd(const LmPlan &pl)
{
    return (pl.full + 7) / 8 + (pl.rest * pl.s2 + 2 * pl.halves + 7) / 8 + (pl.thin * pl.t2 + 7) / 8 - pl.pairs;
}
__host__ __device__ inline bool lm_map_item(int xcd, int idx, int tiles_n, const LmPlan &pl, LmItem &it)
{
    const int n1 = (pl.full + 7) / 8, mid = pl.rest * pl.s2 + 2 * pl.halves, n2 = (mid + 7) / 8;
    it.part = 0;
    it.parts = 1;
    it.block = -1;
    it.pair = 0;
    it.height = LM_BM;
    int L, half = 0;
    if (idx < n1) {
        L = xcd * n1 + idx;
        if (L >= pl.full) return false;
    } else if (idx < n1 + n2) {
        const int j = xcd * n2 + (idx - n1);
        if (j >= mid) return false;
        if (pl.halves > 0) {  // the two halves of a tile side by side: they share the B panel
            L = pl.full + (j >> 1);
            half = j & 1;
            it.height = LM_BM / 2;
        } else {
            it.part = j / pl.rest;
            it.parts = pl.s2;
            L = pl.full + (j - it.part * pl.rest);
            it.block = (j - it.part * pl.rest) * pl.s2 + it.part;
        }
    } else {
        const int items = pl.thin * pl.t2, n3 = (items + 7) / 8;
        const int place = idx - n1 - n2, in_run = place + (place < pl.pairs ? place : pl.pairs), j = xcd * n3 + in_run;
        if (in_run >= n3 || j >= items) return false;
        it.pair = place < pl.pairs && in_run + 1 < n3 && j + 1 < items ? 1 : 0;
        it.part = j / pl.thin;
        it.parts = pl.t2;
        it.tn = j - it.part * pl.thin;
        it.row0 = pl.rows_w * LM_BM;
        it.height = LM_BM / 2;
        it.block = pl.rest * pl.s2 + it.tn * pl.t2 + it.part;
        return true;
    }
    int tm;
    lm_tile_of(L, pl.rows_w, tiles_n, tm, it.tn);
    it.row0 = tm * LM_BM + half * (LM_BM / 2);
    return true;
}

// Workgroups launched for each XCD: one for each of its CUs, or as many as its lists can have places if those are
// fewer (others would return at once).  M: the most rows there can be.  A tile is at most two items, and two of an
// XCD's three lists may be rounded up: bounded by the number of items alone, one workgroup had to take two places
// one after the other while others had none (log-probs of 511 rows x 511 x 1024: 44 us, 33 with a place each).
inline int lm_workgroups_per_xcd(int M, int tiles_n, bool split, int n_cu)
{
    const int cus = n_cu >= 8 ? n_cu / 8 : 1;
    const long long places = (2 * (long long)((M + (long long)LM_BM - 1) / LM_BM) * tiles_n + 14) / 8;
    return split || places > cus ? cus : places > 1 ? (int)places : 1;
}

}  // namespace
