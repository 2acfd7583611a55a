// The launch shapes of the attention kernels: how many workgroups, and which head and which query
// rows each of them takes.  Plain integer code shared by the host (which fills the shape in), the
// kernels (which decode their workgroup number with it) and the CPU tests (which check, through the
// library's diagnostic calls, that the decoded items tile every head's rows exactly once).
//
// Workgroups are dealt round-robin to the 8 XCDs (workgroup w runs on XCD w % 8), each with an L2
// of its own.  A head's K/V stream is shared by all its workgroups, so a head is given to as few
// XCDs as possible: every XCD takes all workgroups of `whole_heads` heads of its own, then its
// share of the heads % 8 heads that are left: each of those split over `share` XCDs, `left_chunk`
// workgroups apiece (when heads % 8 divides 8), or (share == 0) their workgroups dealt out
// contiguously, `left_chunk` per XCD.
//
// A head's ceil(n / 32) wavefronts' worth of query rows go to its q_tiles = ceil(n / 256)
// workgroups as evenly as whole wavefronts allow: the first `q_more` of them take q_waves + 1
// wavefronts' rows, the others q_waves (<= 8 either way).  With full workgroups and one short one,
// the short one runs ahead of the others through the head's keys, out of reach of the L2 they
// share, and the head is fetched from memory twice.
#pragma once
#include <hip/hip_runtime.h>

namespace ifx {

struct attn_shape {
    int q_tiles;   // workgroups per head
    int q_waves, q_more;
    int whole_heads, left_heads, share, left_chunk;
    unsigned grid;  // workgroups of the launch (a few of them may find nothing to do and exit)
};

// What one workgroup does: `waves` wavefronts of 32 query rows from row0 on (the last row of the
// last one may lie past n - 1), or nothing (waves == 0).
struct attn_item {
    int head, q_tile, row0, waves;
};

// row_waves: the most wavefronts' worth of rows a workgroup takes (8, or 4 with two key groups)
inline attn_shape attn_shape_for(int n, int heads, int row_waves = 8)
{
    attn_shape s;
    const int q_wavefronts = (n + 31) / 32;
    s.q_tiles = (q_wavefronts + row_waves - 1) / row_waves;  // so 1 <= q_waves <= row_waves
    s.q_waves = q_wavefronts / s.q_tiles;
    s.q_more = q_wavefronts % s.q_tiles;
    s.whole_heads = heads / 8;
    s.left_heads = heads % 8;
    s.share = s.left_heads > 0 && 8 % s.left_heads == 0 ? 8 / s.left_heads : 0;
    s.left_chunk = s.left_heads == 0 ? 0
                   : s.share > 0     ? (s.q_tiles + s.share - 1) / s.share
                                     : (s.left_heads * s.q_tiles + 7) / 8;
    s.grid = 8u * (unsigned)(s.whole_heads * s.q_tiles + s.left_chunk);
    return s;
}

// Into how many groups of wavefronts a call's keys are dealt.  One (a wavefront takes every key) is
// the least copying per flop and the choice wherever 256-row workgroups fill the chip, and where a
// head's rows are so few that its keys are read once either way: up to 5 wavefronts of rows per head
// two groups have (almost) the same workgroups, twice the start and end, and nothing to gain at the
// memory's rate (128 rows x 300 heads x 896 keys: 41 us, 46 with two; 32 x 257 x 256: 16.2, 17.6;
// 136 x 100 x 136: 9.6, 9.7; 168 x 100 x 168: 10.8, 9.8).
// Two (128 rows per workgroup, half the keys per wavefront: half the serial chain at 1.15 times the
// work) is taken by its rounds of workgroups on 256 CUs:
//  - one round: 1.04 .. 1.8 times as fast (1560 rows x 12 heads x 10920 keys 176 -> 106 us; 4680 x 6 x
//    14040 228 -> 168); one more workgroup is a second round (4680 x 7: 231 -> 316);
//  - two, where 256-row workgroups need a short second one, which costs as long as a full one: 1.1 ..
//    1.5 (264 x 135 x 1056 50 -> 39 us; 10800 x 6 x 32400 1259 -> 820);
//  - three short ones instead of two long ones: three of a two-group workgroup take 0.9 of two of the
//    others, so it pays only where a workgroup's start and end are lost in its keys, from about 1150
//    rows on (1160 x 52: 1.02 .. 1.1 times as fast, 4680 x 18 1.06 .. 1.1; 1032 x 57 .. 76 0.98 .. 1.09, 392 x 135
//    0.87 .. 1.02), and only up to about 680 workgroups (level at 690 .. 760).
// Measured on both caches, with and without a block table, under and past the norm bound: the lines lie
// in the same places (an fp8 cache gains a little less throughout).
// Eight (ifx_attn_few.hpp: 32 rows per workgroup) when even that is one round: 2 .. 3 times as fast
// as one group, 1.5 as two (1560 x 5 x 10920: 176, 102, 63 us; 264 x 2 x 792: 21.2, 16.5, 10.1); level
// with one for a handful of keys (64 rows and less, no cached keys); at two rounds (1560 x 6) it falls
// behind two groups.
// The rule looks at the rows only, never at the keys: a block's calls all take the same path.
inline int attn_groups_for(int n, int heads)
{
    const int row_wavefronts = (n + 31) / 32;
    if ((int64_t)row_wavefronts * heads <= 256) return 8;
    if (row_wavefronts <= 5) return 1;
    const unsigned whole = attn_shape_for(n, heads).grid, halved = attn_shape_for(n, heads, 4).grid;
    if (halved <= 256) return 2;
    return whole > 256 && halved <= (row_wavefronts > 36 ? 680 : 512) ? 2 : 1;
}

// Workgroups that share a 32-row tile of a call of eight key groups without parts: each takes all of the tile's scores and its
// own of the 4 slabs of 32 output dimensions, and reads 256 of a key's 512 bytes for the scores and 64 or 128 for the values.
// What a step takes there is what one CU's L1 passes on, so on CUs that would be idle the tile ends sooner, and the wavefronts'
// shares are put together a slab or two at a time; nothing is exchanged between the workgroups.  As many as
// leave all of them one round on 256 CUs.  us, by one workgroup and shared, bf16 cache: 264 rows x 2 heads, 792 keys 9.6 ->
// 7.7; 1584 keys 12.7 -> 9.9; 88 x 4, 352 7.5 -> 6.4; two to a tile: 136 x 20, 680 9.6 -> 8.4; 760 x 3, 1520 12.9 -> 11.2; 1000
// x 4, 2000 15.1 -> 14.2; fp8: 208 x 11, 1664 13.6 -> 12.0; 264 x 2, 792 9.3 -> 7.7.
inline int few_slab_groups(int n, int heads)
{
    const int64_t workgroups = (int64_t)((n + 31) / 32) * heads;
    return workgroups <= 64 ? 4 : workgroups <= 128 ? 2 : 1;
}

// How a bf16 call's keys are dealt: `groups` inside a workgroup (attn_groups_for), and those of heads
// [whole_heads, heads) to `parts` workgroups per row tile (of 256 rows, one group, or of 32, eight); parts == 1: no head's.
struct attn_plan {
    int groups, whole_heads, parts;
};

// Units of 32 rows that a call's partial results may take (16.25 KiB each).
constexpr int64_t SPLIT_MOST_UNITS = 2048;

// The parts that a split of a call's keys would have, whatever their number.
inline attn_plan attn_split_candidate(int n, int heads)
{
    const int64_t row_waves = (n + 31) / 32, per_head = (row_waves + 7) / 8, workgroups = per_head * heads;
    attn_plan p = {1, 0, 1};
    if (workgroups <= 128) {
        p.parts = (int)(256 / workgroups);
    } else if (workgroups > 256 && workgroups % 256 <= 80 && workgroups % 256 != 0) {
        p.whole_heads = (int)(workgroups / 256 * 256 / per_head);
        const int parts = (int)(192 / (workgroups % 256));
        p.parts = parts < 2 ? 2 : parts > 8 ? 8 : parts;
    }
    const int64_t most = SPLIT_MOST_UNITS / (row_waves * (heads - p.whole_heads));
    if (p.parts > most) p.parts = (int)most;
    return p;
}

// Parts are worth a second launch and the way of their results through memory (fp32, 16 KiB per 32 rows and part:
// they meet in the memory-side cache, 0.5 us a MB there and back) where
//  - one round of 256-row workgroups leaves most CUs idle: the keys of every head to 256 / workgroups of them.
//    Against the best unsplit kernel (us, bf16 cache, two layers in turn): 1560 rows x 3 heads x 10920 keys 56 -> 42,
//    x 5 62 -> 55, x 8 98 -> 74, x 12 109 -> 101 (fp8 127 -> 100); 4680 x 1 x 32760 143 -> 90, x 2 277 -> 147, x 4
//    302 -> 266; 800 x 12 x 6400 62 -> 43; 10800 x 1 x 54000 453 -> 266.  Level, or behind, on short key runs: 600 x
//    16 x 2400 30 -> 28, 800 x 10 x 6400 39 -> 38, 400 x 5 x 2000 15 -> 20.
//  - 32-row workgroups are at most half a round: the same with those, whose partial results are fewer.  What a step of
//    such a workgroup takes is the 128 KiB of keys that its CU's L1 can pass on (45 of 64 bytes per cycle), so only more
//    CUs shorten it.  Against tiles shared by slabs (few_slab_groups), whole -> parts: 1560 x 1 x 3120 14.9 -> 14.1, x 10920 41 ->
//    22; 1000 x 2 x 3000 15.9 -> 14.9, x 4000 19.0 -> 15.9; 264 x 2 x 3168 14.3 -> 12.7; two to a tile: 760 x 3 x 3800 18.0 -> 16.5,
//    1424 x 2 x 4272 20.8 -> 19.5, 464 x 6 x 4640 21.7 -> 20.5; level from 9 to 11 steps (two to a tile 12 to 17): 264 x 2 x 2112
//    11.2 -> 11.8, 552 x 3 x 2760 14.1 -> 14.3, 400 x 5 x 2800 14.7 -> 15.2, 760 x 3 x 3040 15.6 -> 15.5, 1000 x 3 x 4000 19.3 -> 19.3; and
//    behind below: 1000 x 1 x 2000 11.5 -> 12.8, 400 x 2 x 2000 11.2 -> 12.2, 680 x 1 x 2040 11.3 -> 12.0, 440 x 3 x 2200 12.1 -> 12.9.
//    A step over codes takes workgroups that share a tile longer (each widens them), so an fp8 cache's keys come in parts a step
//    or two earlier: 264 x 2 x 2112 12.1 -> 11.4, 216 x 1 x 1944 11.6 -> 11.0, 760 x 3 x 3040 16.7 -> 15.1, 752 x 4 x 3760 19.4 -> 18.7,
//    360 x 8 x 4320 21.6 -> 20.0; behind: 144 x 1 x 1728 10.8 -> 10.9, 160 x 12 x 1920 11.5 -> 13.7.  Of some 480 calls about the lines
//    the side taken is the faster one or at most 4 % behind it in all but ten (5 to 7: 264 x 2 x 2112, 136 x 8 x 2584).
//  - a last round would be nearly empty: whole heads fill the rounds, the keys of the rest go to as many
//    workgroups as its CUs.  4680 x 14 x 18720 648 -> 496, x 15 653 -> 526, x 16 654 -> 560, x 17 658 -> 595, x 18
//    675 -> 642; x 28 x 14040 899 -> 753; 10800 x 7 x 32400 1120 -> 981; 1560 x 40 x 10920 379 -> 295; but 1560 x 37
//    281 -> 275 and 10800 x 6 840 -> 840, where two groups take two rounds.
// Below: the sides' times (us) as fitted to such measurements.  The tiles are the call's 64-key tiles.
inline attn_plan attn_plan_for(int n, int heads, int tiles, bool fp8)
{
    const attn_plan whole = {attn_groups_for(n, heads), heads, 1};
    const int row_waves = (n + 31) / 32;
    const float rows = (float)row_waves * (float)heads;
    attn_plan p = attn_split_candidate(n, heads);
    if (p.parts > tiles / 4) p.parts = tiles / 4;
    if (p.parts > 1 && p.whole_heads > 0) {
        const unsigned halved = attn_shape_for(n, heads, 4).grid;
        return tiles >= 100 && halved > 512 ? p : whole;
    }
    const float few_steps = (float)((tiles + 3) / 4);  // of a wavefront, 32 keys each
    float us = 8.f + tiles * 1.0f;                     // one group
    if (whole.groups == 8) {
        const int sharing = few_slab_groups(n, heads);
        const float busy = rows * (float)sharing / 256.f;
        us = sharing == 4   ? 5.1f + few_steps * (fp8 ? 0.81f + 0.09f * busy : 0.73f + 0.12f * busy)
             : sharing == 2 ? 5.1f + few_steps * (fp8 ? 0.85f + 0.16f * busy : 0.68f + 0.31f * busy)
                            : 5.3f + few_steps * 1.13f * (1.f + 0.2f * busy * busy);
    } else if (whole.groups == 2) {
        const float busy = (float)((row_waves + 3) / 4 * heads) / 256.f;
        us = 8.f + tiles * (busy <= 0.4f ? 0.52f : 0.52f + 0.4f * (busy - 0.4f));
    }
    const float us_whole = us;
    us *= 0.95f;
    attn_plan best = whole;
    if (p.parts > 1) {
        const float part = (float)tiles / (float)p.parts, per_tile = 0.85f + 0.0065f * part;
        const float us_split = 15.f + rows * p.parts * 0.0083f + part * (per_tile < 1.38f ? per_tile : 1.38f);
        if (us_split < us) {
            us = us_split;
            best = p;
        }
    }
    if (whole.groups == 8) {
        const int workgroups = row_waves * heads, most = tiles / 4, enough = 256 / workgroups, parts = enough < most ? enough : most;
        if (parts > 1) {
            // (against whole calls: fitted where the two are level; against 256-row parts: to the longer runs where those are)
            const bool few = best.parts > 1 ? 11.f + 1.15f * (float)((tiles + 4 * parts - 1) / (4 * parts)) < us
                                            : 9.7f + 1.07f * (float)tiles / (float)(4 * parts) + 2.f * rows * (float)parts / 256.f < us_whole;
            if (few) best = {8, 0, parts};
        }
    }
    return best;
}

// Keys of a head dealt to several workgroups per row tile.  With 32-row tiles: row_tiles_for(n, heads * parts, 32), whose
// `head` counts (head, part) pairs.  With 256-row ones the launch is the workgroups of the whole heads
// (shape of whole_heads heads), then those of the split ones: the shape of parts * (heads - whole_heads)
// heads, whose `head` counts (head, part) pairs, so that the workgroups that read one part of one head's keys sit
// on one XCD, or few.
struct attn_split {
    attn_shape shape;     // of the split heads' workgroups
    unsigned whole_grid;  // workgroups before those
    int whole_heads, parts;
    int row_tiles;        // of 32 rows, per head
    bool exact_sums;      // every row's sum from the weights as rounded to bf16: what calls of eight groups take
};

inline attn_split attn_split_for(int n, int heads, const attn_plan &p)
{
    attn_split s = {};
    if (p.parts == 1) return s;
    if (p.groups == 1) s.shape = attn_shape_for(n, (heads - p.whole_heads) * p.parts);
    s.whole_grid = p.whole_heads > 0 ? attn_shape_for(n, p.whole_heads).grid : 0;
    s.whole_heads = p.whole_heads;
    s.parts = p.parts;
    s.row_tiles = (n + 31) / 32;
    s.exact_sums = attn_groups_for(n, heads) == 8;  // (the split takes no row's precision)
    return s;
}

// Units of partial results that calls over up to `tiles` tiles of keys need, of either cache.
inline int64_t attn_split_units(int n, int heads, int64_t tiles)
{
    const int64_t rows = (n + 31) / 32;
    int64_t most = 0;
    for (int64_t t = 8; t <= tiles; ++t) {
        for (const bool fp8 : {false, true}) {
            const attn_plan p = attn_plan_for(n, heads, (int)t, fp8);
            const int64_t units = p.parts > 1 ? rows * (heads - p.whole_heads) * p.parts : 0;
            if (units > most) most = units;
        }
    }
    return most;
}

// First of the tiles that part `part` of `parts` takes: `tiles` dealt as evenly as whole tiles allow.
__host__ __device__ inline int part_begin(int tiles, int parts, int part) { return (int)((int64_t)tiles * part / parts); }

// Where the partial result of 32 rows of a split head's part lies.
__host__ __device__ inline int64_t split_unit_of(const attn_split &s, int split_head, int part, int row_tile)
{
    return ((int64_t)split_head * s.parts + part) * s.row_tiles + row_tile;
}

__host__ __device__ inline attn_item attn_item_of(const attn_shape &s, unsigned workgroup)
{
    const int xcd = (int)(workgroup & 7u);
    const int idx = (int)(workgroup >> 3);
    attn_item it = {0, 0, 0, 0};
    if (idx < s.whole_heads * s.q_tiles) {
        it.head = xcd * s.whole_heads + idx / s.q_tiles;
        it.q_tile = idx % s.q_tiles;
    } else {
        const int rest = idx - s.whole_heads * s.q_tiles;
        if (s.share > 0) {
            it.head = 8 * s.whole_heads + xcd / s.share;
            it.q_tile = (xcd % s.share) * s.left_chunk + rest;
            if (it.q_tile >= s.q_tiles) return it;
        } else {
            const int item = xcd * s.left_chunk + rest;
            if (item >= s.left_heads * s.q_tiles) return it;
            it.head = 8 * s.whole_heads + item / s.q_tiles;
            it.q_tile = item % s.q_tiles;
        }
    }
    it.row0 = 32 * (it.q_tile * s.q_waves + (it.q_tile < s.q_more ? it.q_tile : s.q_more));
    it.waves = s.q_waves + (it.q_tile < s.q_more ? 1 : 0);
    return it;
}

// The kernels whose workgroups take one tile of rows each (bf16 with the keys dealt to eight groups, 32
// rows; fp32, 16 rows): the (head, tile) items in order, every XCD a contiguous run of them, so that
// a head's keys are read into as few L2s as possible.
struct row_tiles {
    int tiles;    // per head
    int per_xcd;  // workgroups per XCD: 8 times as many are launched, the last few may exit at once
};

struct row_tile {
    int head, tile;  // head < 0: nothing to do
};

// sharing: workgroups per tile of rows
inline row_tiles row_tiles_for(int n, int heads, int rows, int sharing = 1)
{
    row_tiles t;
    t.tiles = (n + rows - 1) / rows * sharing;
    t.per_xcd = (int)(((int64_t)t.tiles * heads + 7) / 8);
    return t;
}

__host__ __device__ inline row_tile row_tile_of(const row_tiles &t, int heads, unsigned workgroup)
{
    const int item = (int)(workgroup & 7u) * t.per_xcd + (int)(workgroup >> 3);
    if (item >= heads * t.tiles) return {-1, 0};
    const int head = item / t.tiles;
    return {head, item - head * t.tiles};
}

}  // namespace ifx
