// fp32 block attention for gfx950: fp32 matrix instructions, accurate expf, online softmax.
//
// Operation (paper, Introduction, framework paragraph + abstract): every query
// of the block attends to all resident cached tokens and all tokens of its own
// block; softmax over that whole key set; no other mask.
//
// Shape of the computation
//   Bound by the fp32 matrix rate (64 flop per cycle and SIMD; the pipes are 64 % busy on a large call),
//   and by the chain inside a wavefront where rows are few.  A workgroup owns 16 query rows of a
//   head; its 4 or 8 wavefronts deal the keys among themselves in subtiles of 16 (wavefront w takes
//   subtiles w, w + S, ...) and their partial results are combined through LDS at the end.  So even
//   the 512 rows of a 256-token block with 2 heads are 32 workgroups of 8 busy wavefronts.  Both
//   contractions run on v_mfma_f32_16x16x4_f32 (fp32 products and sums, nothing is rounded on the
//   way), transposed so that a lane's scores all belong to one query:
//     S^T (keys x queries) = K * Q^T          O^T (d x queries) += V^T * P^T
//   Lane (i = lane % 16, g = lane / 16).  A and B hold row / column i at contraction index g, the
//   accumulator holds column i, rows 4 g + r.  So register r of S^T is the score of query i against
//   key 4 g + r, and the exponentials are, as they stand, the B operands of four PV steps in which
//   lane group g contributes key 4 g + r.  The contraction over d is taken in the order
//   d = 16 j + 4 g + t, which makes a lane's K operands of four steps 16 contiguous bytes; output
//   dimension 64 s + 4 row + slab is row `row` of accumulator slab 4 s + slab, which makes its V
//   operands of four slabs 16 contiguous bytes too (two slabs where only 32 dimensions are left).
//   Nothing but the end is shared between wavefronts: no barrier in the loop.  V goes from memory
//   straight into registers (16 lanes read 256 contiguous bytes of a row) and is on its way under the
//   score MFMAs.  K cannot: 64 lanes would read 16 bytes of a line each, 64 address cycles per
//   load instead of 16, more than the matrix instructions they feed.  It is copied row by row into a
//   piece of LDS of the wavefront's own (direct global->LDS loads, the next subtile's in flight
//   from the moment this one's operands have been read) and read from there, swizzled at 16-byte
//   granularity so that the 16 rows of a read lie in 16 different bank groups.
// (Calls with rows enough go to attn_f32l_kernel, ifx_attn_f32_large.hpp, unless their keys are a selection: attn_f32_plan.)
// Measured (1560 rows, 12 heads x 128, 3120 keys): 291 us = 103 TFLOP/s, where the library's plain
// fp32 matrix product reaches 154 on the same card; 1840 us with fp32 FMA from LDS tiles.  With K
// straight from memory 393 us; with 32 rows per wavefront (half the bytes per flop, but fewer and
// larger workgroups) 390 us.  256 rows, 2 heads x 64, 1024 keys: 16.1 us whole (118 with 32-row workgroups
// that do not deal the keys out); in eight parts 9.6 to 10.3, 14.5 with the block's commit.  Traced, 7.4 of the
// attention, 3.2 of putting the parts together and 2.6 of the commit: 256 CUs whose wavefronts take one subtile
// each, half their cycles at wait counts (a subtile's K, then its V), the matrix pipes 6 % busy.
#pragma once
#include <cfloat>

#include "ifx_launch.hpp"
#include "ifx_types.hpp"

namespace ifx {

constexpr int F32_MAXD = 128;
constexpr int F32_ROWS = 16;  // query rows per workgroup
constexpr int F32_KEYS = 16;  // keys of a subtile

struct attn_f32_args {
    const float *q, *kc, *vc, *kb, *vb;  // [n, H, D]; layer regions [H][cache_tokens][D]; the block's K, V [n, H, D]
    float *out, *lse;                    // [n, H, D]; [n, H] or nullptr
    int n, C, n_blk, H, D;               // cached keys (the caller's selection, whole blocks of n tokens), then the block's: n or 0
    int64_t cache_tokens;
    float scale;
    row_tiles tiles;                     // workgroup -> (head, row tile), see ifx_launch.hpp; SPLIT: of heads * parts heads
    ifx_key_blocks blocks;
    int parts;                           // SPLIT instantiation only: workgroups per row tile,
    float *partial;                      // their unnormalised outputs [H][parts][tiles][16][DP] ...
    f32x2 *stats;                        // ... and maxima and sums [H][parts][tiles][16]
};

// Wavefronts per workgroup.  Up to one workgroup per CU: 8, two per SIMD.  Beyond that 4: three
// workgroups then share a CU, and one's start and end lie under the others' loops.  Measured with 4
// and 8 (us), head_dim 128: 264 workgroups 47.0, 50.6; 520: 121, 132; 756: 119, 132; 900: 186, 202; 1176:
// 290, 317; 1600: 407, 451.  head_dim 64: 264 workgroups 51.7, 48.9; 1008: 128.9, 128.2; head_dim 40: 300
// workgroups 31.8, 30.4; 1600: 226, 229 (shorter rows leave more to hide; up to 6 % lost there just past 256).
inline int attn_f32_waves(int64_t workgroups) { return workgroups <= 256 ? 8 : 4; }

// Workgroups per row tile that a call's `subs` subtiles of keys are dealt to; a second launch puts their results together
// (combine_f32_kernel; 3 us, and more as the parts' results grow).  Worth it where row tiles leave CUs, or a CU's
// slots, empty over a long key run: up to 128 row tiles one workgroup of 8 wavefronts per CU; up to 480 five parts, whose
// workgroups of 4 fill three slots a CU; up to 700, where some CUs have two workgroups and some three, three parts.
// Measured, whole and in parts (us, with a second launch that took 5): 256 rows x 2 heads x 64, 1024 keys 16.5, 11.8 (now 9.6); 2048 keys 27.7, 13.6; 400 x 4 x
// 128, 2000 keys 46.2, 29.8; 1560 x 1 x 128, 7800 keys 153, 75; 1560 x 2 x 128, 7800 156, 134; 1040 x 4 x 128, 5200 204,
// 132; 1560 x 4 x 128, 4680 186, 160; 1560 x 6 x 128, 4680 262, 221; but 1560 x 5 188, 197 and 1560 x 7 263, 274; 64 x 1 x
// 128, 320 keys 11.7, 12.1; 200 x 30 x 128, 1000 keys 48, 51.  With the second launch at 3 us, three parts and more: 104 x 2 x 128, 416 keys
// 14.6, 12.8; 136 x 8 x 72, 544 keys 14.2, 11.7; 256 x 2 x 96, 512 keys 13.3, 10.7; 344 x 1 x 64, 688 keys 12.3, 9.7.  Below: both sides' times (us) as fitted to these.
inline int attn_f32_parts(int64_t workgroups, int padded_d, int64_t subs)
{
    if (workgroups > 700) return 1;
    const float step = 0.0195f * padded_d, all = (float)workgroups * (float)subs * 1.06e-5f * padded_d;
    const int waves = workgroups <= 256 ? 8 : 4;
    float us = 0.94f * (6.f + (workgroups <= 512 ? step : 1.41f * step) * (float)((subs + waves - 1) / waves));
    int parts = 1;
    if (workgroups <= 128) {
        int64_t p = 256 / workgroups;
        if (p > subs / 8) p = subs / 8;
        // (three parts and more: 9.3, the second launch reading all parts at once; two of 108 tiles were 5 % behind there)
        const float split = p > 1 ? (p > 2 ? 9.3f : 11.f) + step * (float)((subs + 8 * p - 1) / (8 * p)) : us;
        if (split < us) {
            us = split;
            parts = (int)p;
        }
    }
    if (workgroups > 85 && subs >= 40 && 12.f + all < us) parts = workgroups <= 480 ? 5 : 3;
    return parts;
}
// Which kernel takes a call, and to how many workgroups per row tile its keys are dealt.  attn_f32l_kernel (256-row
// workgroups, ifx_attn_f32_large.hpp) where its workgroups, in parts, fill the chip for long enough.  Both sides measured (us, this
// kernel in its parts and that one): 1560 rows x 12 heads x 128, 3120 keys 294, 160; x 16, 4680 keys 591, 309; x 2, 7800 keys
// 133, 81; x 3, 3120 keys 89, 58; 1560 x 9 x 64, 4680 keys 197, 118; and on the other side 400 x 10 x 128, 1200 keys 30, 39; 800 x 3
// x 128, 1600 keys 33, 38; 1240 x 1 x 64, 6200 keys 32, 42.  The costs below were fitted when that kernel's tile took 4.6 and 3.0 us (now 4.2
// and 2.7) and a second launch 4 to 5 (now 3): the line lies on the 16-row kernel's side, where calls near it would gain 10 to 30 %
// (1368 x 3 x 72, 2736 keys 64, 45; 696 x 6 x 128, 1392 keys 52, 38; 808 x 6 x 40, 2424 keys 43, 38; level at 1568 x 1 x
// 96, 6272 keys 51, 52 and 600 x 4 x 72, 2400 keys 35, 37).  It takes no selection of blocks.
struct f32_plan {
    bool large;
    int parts;
};
inline f32_plan attn_f32_plan(int n, int heads, int head_dim, int64_t subs, bool listed)
{
    const int padded_d = (head_dim + 31) / 32 * 32;
    const int64_t row_tiles = (int64_t)((n + 15) / 16) * heads;
    const f32_plan small = {false, attn_f32_parts(row_tiles, padded_d, subs)};
    if (listed) return small;
    const float all = (float)row_tiles * (float)subs * 1.06e-5f * padded_d;
    float us;
    if (small.parts > 1) {
        const float step = 0.0195f * padded_d;
        us = row_tiles * small.parts <= 256 ? 11.f + step * (float)((subs + 8 * small.parts - 1) / (8 * small.parts)) : 12.f + all;
    } else {
        const int waves = row_tiles <= 256 ? 8 : 4;
        const float chain = 6.f + 0.0195f * padded_d * (row_tiles <= 512 ? 1.f : 1.41f) * (float)((subs + waves - 1) / waves);
        us = row_tiles > 768 && all > chain ? all : chain;
    }
    const int64_t workgroups = (int64_t)((n + 255) / 256) * heads, tiles = (subs + 1) / 2;
    int64_t parts = workgroups <= 128 ? 256 / workgroups : 1;
    if (parts > tiles / 4) parts = tiles / 4 > 1 ? tiles / 4 : 1;
    const float filled = (float)((n + 31) / 32) / (float)(8 * ((n + 255) / 256));  // of a workgroup's wavefronts
    const float tile = (head_dim <= 64 ? 3.0f : 4.6f) * (0.5f + 0.5f * filled), rounds = (float)((workgroups * parts + 255) / 256);
    float large = 8.f + rounds * tile * (float)((tiles + parts - 1) / parts);
    if (parts > 1) large += 4.f + 0.5e-6f * (float)(row_tiles * 16 * parts) * (4.f * padded_d + 8.f);
    return large < 0.92f * us ? f32_plan{true, (int)parts} : small;
}
// The most parts that attn_f32_plan deals keys of any number to.
inline int attn_f32_most_parts(int n, int heads)
{
    const int64_t row_tiles = (int64_t)((n + 15) / 16) * heads, workgroups = (int64_t)((n + 255) / 256) * heads;
    int most = workgroups <= 128 ? (int)(256 / workgroups) : 1;
    if (row_tiles <= 128 && 256 / row_tiles > most) most = (int)(256 / row_tiles);
    const int dealt = row_tiles <= 480 ? 5 : row_tiles <= 700 ? 3 : 1;
    return dealt > most ? dealt : most;
}
// Rows of partial results that calls over up to `blocks` cached blocks may leave: of every number of them, with the current
// block and without (a plan's parts rise and fall with the keys); beyond the first thousands the most there can be.
inline int64_t attn_f32_split_rows(int n, int heads, int head_dim, int64_t blocks)
{
    const int limit = attn_f32_most_parts(n, heads);
    const int64_t tiles = (n + 15) / 16;
    constexpr int64_t EACH = 4096;
    int most = blocks > EACH ? limit : 1;
    for (int64_t i = 0; i <= blocks && most < limit; ++i)
        for (const int64_t block : {(int64_t)0, tiles}) {
            // every block in slot order, or listed: those of 16 tokens and more in subtiles of their own, shorter ones either way
            const int64_t dense = (i * n + 15) / 16 + block, own = i * tiles + block;
            const int parts[3] = {attn_f32_plan(n, heads, head_dim, dense, false).parts, attn_f32_plan(n, heads, head_dim, own, true).parts,
                                  n < 16 ? attn_f32_plan(n, heads, head_dim, dense, true).parts : 1};
            for (const int p : parts)
                if (p > most) most = p;
        }
    return most > 1 ? tiles * heads * most * F32_ROWS : 0;
}
inline size_t attn_f32_split_row_bytes(int padded_d) { return (size_t)padded_d * 4 + 8; }

// LDS: each wavefront's K subtile during the loop; the partial results take its place afterwards.
inline size_t attn_f32_lds_bytes(int padded_d, int waves)
{
    return (size_t)waves * F32_ROWS * ((size_t)(padded_d + 4) + 2) * sizeof(float);
}

// GATHER: for listed blocks shorter than a subtile.  A subtile is then 16 consecutive keys of the listed
// ones, from several blocks, where otherwise it lies in one and holds as few keys as the block (200
// listed blocks of one token, 4 heads x 64: 45.6 us, now 17).  Each lane works out where one of the rows lies
// and the copies and loads fetch that from it (a lane exchange per instruction, so not the form for
// blocks that fill subtiles); the offsets are 32 bits, so a head's region must lie below GATHER_MOST.
constexpr int64_t GATHER_MOST = 0x7f000000;
// SPLIT: a row tile's subtiles are dealt to a.parts workgroups in runs, whose results combine_f32_kernel puts together.
template <int DP, bool GATHER = false, bool SPLIT = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(GATHER ? 2 : 3))) void attn_f32_kernel(const attn_f32_args a)
{
    static_assert(DP % 32 == 0 && DP <= F32_MAXD, "");
    constexpr int KJ = DP / 16;          // 16-byte K chunks of a lane per subtile
    constexpr int CH = DP / 4;           // 16-byte chunks of a row
    constexpr int QUADS = DP / 64;       // groups of four accumulator slabs
    constexpr bool PAIR = DP % 64 != 0;  // and one group of two
    constexpr int SLABS = DP / 16;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    typedef __attribute__((address_space(3))) void *lds_ptr;

    const int n = a.n, H = a.H, D = a.D, C = a.C;
    const row_tile item = row_tile_of(a.tiles, SPLIT ? H * a.parts : H, blockIdx.x);
    if (item.head < 0) return;
    const int h = SPLIT ? item.head / a.parts : item.head, row0 = item.tile * F32_ROWS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = (int)blockDim.x >> 6;
    const int i16 = lane & 15, g = lane >> 4;

    // A subtile is up to 16 keys that lie in one run of rows: of the cached tokens [0, C), of one block
    // of a selection, or of the current block.  It is read through a buffer descriptor that starts at
    // its first row and ends with its last one (rows behind that read as zero and are masked).
    const bool listed = a.blocks.magic != 0;
    const int seg_keys = GATHER ? a.blocks.count * n : listed ? n : C;  // keys of a cached segment
    const int seg_subs = (seg_keys + 15) >> 4;                          // its subtiles
    const int cached_subs = !GATHER && listed ? a.blocks.count * seg_subs : seg_subs;
    const int all_subs = cached_subs + ((a.n_blk + 15) >> 4), part = SPLIT ? item.head - h * a.parts : 0;
    const int subs = SPLIT ? part_begin(all_subs, a.parts, part + 1) : all_subs;
    const int own_sub = wave + (SPLIT ? part_begin(all_subs, a.parts, part) : 0);
    // 64 entries of a selection from tab_first on, one per lane: a lookup is a lane read.  A wavefront
    // walks its subtiles in order, so the 64 move along a longer list.
    int tab = 0, tab_first = 0;
    auto load_entries = [&](int e) __attribute__((always_inline)) {
        tab_first = e;
        if (e + lane < a.blocks.count) {  // (two plain indexed reads, see ifx_attn_bf16.hpp)
            if (a.blocks.list != nullptr)
                tab = a.blocks.list[e + lane];
            else
                tab = a.blocks.first[e + lane];
        }
    };
    if (listed) load_entries(0);
    struct run {
        int64_t at;            // element offset of the first row, in the cache region or in the block's tensor
        int stride, keys;      // elements between rows; rows
        bool cached;
    };
    auto run_of = [&](int sub) __attribute__((always_inline)) -> run {
        if (sub < cached_subs) {
            if constexpr (GATHER) return {(int64_t)h * a.cache_tokens * D, D, seg_keys - 16 * sub, true};  // (the region's start)
            int e = 0, first = 0;
            if (listed) {
                e = sub / seg_subs;
                if (e >= tab_first + 64) load_entries(e);
                first = __builtin_amdgcn_readlane(tab, e - tab_first);
            }
            const int j = 16 * (sub - e * seg_subs);
            return {((int64_t)h * a.cache_tokens + first + j) * D, D, seg_keys - j, true};
        }
        const int j = 16 * (sub - cached_subs);
        return {((int64_t)j * H + h) * D, H * D, a.n_blk - j, false};
    };
    // (the two candidate pointers as numbers: selecting between the pointers themselves makes the
    // compiler fetch the chosen one from the kernel arguments again)
    const uintptr_t kc = (uintptr_t)a.kc, kb = (uintptr_t)a.kb, vc = (uintptr_t)a.vc, vb = (uintptr_t)a.vb;
    auto rsrc_of = [&](const run &r, uintptr_t cache, uintptr_t block) __attribute__((always_inline)) -> __amdgpu_buffer_rsrc_t {
        const uintptr_t u = (r.cached ? cache : block) + 4 * (uintptr_t)r.at;
        const uintptr_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
        const int rows = r.keys < 16 ? r.keys : 16;
        const int bytes = GATHER && r.cached ? (int)(4 * a.cache_tokens * D) : 4 * ((rows - 1) * r.stride + D);
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
    };
    // K copies: LDS slot e = 64 x + lane (x = 0 .. KJ - 1; row e / CH, place e % CH) receives the row's
    // chunk place ^ z(row).  Dimensions past D are asked for behind the run's end and read as zero, like Q's
    // there (at a dimension of the row an infinite element would meet Q's zero and make the score NaN).
    constexpr int ROWS_X = 64 % CH == 0 ? 64 / CH : 0;  // whole rows per copy instruction
    // an offset behind any run or region: a run is at most 16 rows of 65535 heads of 128 floats, 2^29 bytes, and
    // this and a row's offset added stay below 2^32
    constexpr int PAST_RUN = (int)GATHER_MOST;
    // GATHER: the byte offset in the region of key i16 of subtile `sub` (other forms: unused)
    const int per_n = GATHER ? 65536 / n + 1 : 0;  // x * per_n >> 16 is x / n for the x < 32 and n < 16 below
    auto row_offset = [&](int sub) __attribute__((always_inline)) -> int {
        if (!GATHER || sub >= cached_subs) return 0;
        const int e0 = 16 * sub / n;
        if (e0 + 15 >= tab_first + 64) load_entries(e0);
        const int x = 16 * sub - e0 * n + i16, q = (x * per_n) >> 16, e = e0 + q;
        const int first = __shfl(tab, e - tab_first);
        return e < a.blocks.count ? 4 * D * (first + x - q * n) : PAST_RUN;
    };
    auto z = [](int r) { return CH % 16 == 0 ? r : r >> 1; };
    float *const ktile = smem + wave * (F32_ROWS * DP);
    auto copy_k = [&](int sub, int row_off) __attribute__((always_inline)) {
        const run r = run_of(sub);
        const __amdgpu_buffer_rsrc_t rs = rsrc_of(r, kc, kb);
#pragma unroll
        for (int x = 0; x < KJ; ++x) {
            const int e = 64 * x + lane, row = e / CH, d = 4 * ((e % CH) ^ z(row));
            // (not const: with arguments that depend on DP the host pass rejects the builtin's size, silently)
            int off_v = d < D ? 4 * ((ROWS_X ? lane / CH : row) * r.stride + d) : PAST_RUN, off_s = 4 * (ROWS_X * x) * r.stride;
            if (GATHER && r.cached) {
                const int off = __shfl(row_off, row);
                off_v = d < D ? off + 4 * d : PAST_RUN;
                off_s = 0;
            }
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(ktile + 256 * x), 16, off_v, off_s, 0, 0);
        }
    };
    // K operand j of a lane: row i16, d = 16 j + 4 g .. + 3, i.e. chunk 4 j + g; z reaches the low 3 or
    // 4 bits of a chunk number, so the places of j and j + Z_J are a constant apart
    constexpr int Z_J = CH % 16 == 0 ? 4 : 2;
    const float *kread[Z_J];
#pragma unroll
    for (int j = 0; j < Z_J; ++j) kread[j] = ktile + i16 * DP + 4 * ((4 * j + g) ^ z(i16));
    f32x4 V[4][QUADS > 0 ? QUADS : 1];
    f32x2 V2[4];
    int dv[QUADS > 0 ? QUADS : 1];
#pragma unroll
    for (int s = 0; s < QUADS; ++s) dv[s] = 64 * s + 4 * i16 < D ? 64 * s + 4 * i16 : 0;
    const int dv2 = 64 * QUADS + 2 * i16 < D ? 64 * QUADS + 2 * i16 : 0;
    auto load_v = [&](int sub, int row_off) __attribute__((always_inline)) -> int {  // returns the subtile's keys
        typedef uint32_t raw_u32x4 __attribute__((__vector_size__(16)));
        typedef uint32_t raw_u32x2 __attribute__((__vector_size__(8)));
        const run u = run_of(sub);
        const __amdgpu_buffer_rsrc_t rs = rsrc_of(u, vc, vb);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int off = 4 * (4 * g * u.stride), off_s = 4 * r * u.stride;
            if (GATHER && u.cached) {
                off = __shfl(row_off, 4 * g + r);
                off_s = 0;
            }
#pragma unroll
            for (int s = 0; s < QUADS; ++s)
                V[r][s] = __builtin_bit_cast(f32x4, (raw_u32x4)__builtin_amdgcn_raw_buffer_load_b128(rs, off + 4 * dv[s], off_s, 0));
            if constexpr (PAIR)
                V2[r] = __builtin_bit_cast(f32x2, (raw_u32x2)__builtin_amdgcn_raw_buffer_load_b64(rs, off + 4 * dv2, off_s, 0));
        }
        return u.keys;
    };

    int row_off = row_offset(own_sub);
    if (own_sub < subs) copy_k(own_sub, row_off);
    f32x4 Q[KJ];
    {
        const int i = row0 + i16;
        const float *qp = a.q + ((int64_t)(i < n ? i : n - 1) * H + h) * D;
#pragma unroll
        for (int j = 0; j < KJ; ++j) {
            const int d = 16 * j + 4 * g;
            Q[j] = *reinterpret_cast<const f32x4 *>(qp + (d < D ? d : 0));
            if (d >= D) Q[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    f32x4 O[SLABS];
#pragma unroll
    for (int s = 0; s < SLABS; ++s) O[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    // running maximum of the scaled scores (per query), this lane's share of the row sum.  The maximum starts
    // at the lowest finite value, not at -inf: a subtile whose scores are all -inf then has weight 0 (-inf
    // less -inf is NaN), and so has a wavefront without keys
    float m = -FLT_MAX, l = 0.f;

    for (int sub = own_sub; sub < subs; sub += S) {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the K copies (V has been consumed) are in LDS
        f32x4 K[KJ];
#pragma unroll
        for (int j = 0; j < KJ; ++j) K[j] = *reinterpret_cast<const f32x4 *>(kread[j % Z_J] + 16 * (j - j % Z_J));
        const int keys = load_v(sub, row_off);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this subtile's operands are in registers, the tile is free
        __builtin_amdgcn_sched_barrier(0);
        const int next = sub + S < subs ? sub + S : sub;  // (always copied: the wait counts then know what is in flight)
        row_off = row_offset(next);
        copy_k(next, row_off);
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < KJ; ++c)
#pragma unroll
            for (int t = 0; t < 4; ++t) s = __builtin_amdgcn_mfma_f32_16x16x4f32(K[c][t], Q[c][t], s, 0, 0, 0);
        s *= a.scale;
        if (keys < 16) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * g + r >= keys) s[r] = -INFINITY;
        }
        float t = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
        t = fmaxf(t, __shfl_xor(t, 16));
        t = fmaxf(t, __shfl_xor(t, 32));
        if (__any(t > m)) {
            const float m_new = fmaxf(m, t);
            const float alpha = expf(m - m_new);  // 0 on the first one
            l *= alpha;
#pragma unroll
            for (int e = 0; e < SLABS; ++e) O[e] *= alpha;
            m = m_new;
        }
        f32x4 p;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = expf(s[r] - m);
            l += p[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < SLABS; ++e)
                O[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(e < 4 * QUADS ? V[r][e >> 2][e & 3] : V2[r][e & 1], p[r], O[e], 0, 0, 0);
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);

    // ---- combine the wavefronts' shares of every row: partial O, maximum and sum through LDS
    __builtin_amdgcn_s_waitcnt(0x0F70);  // (the copy behind the last subtile has landed)
    __syncthreads();
    constexpr int LD = DP + 4;  // rows 4 floats apart from a multiple of the banks
    float *ml = smem + S * F32_ROWS * LD;
    {
        const int w = wave * F32_ROWS + i16;
        float *dst = smem + w * LD;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int s = 0; s < QUADS; ++s)
                *reinterpret_cast<f32x4 *>(dst + 64 * s + 16 * g + 4 * r) = f32x4{O[4 * s][r], O[4 * s + 1][r], O[4 * s + 2][r], O[4 * s + 3][r]};
            if constexpr (PAIR) *reinterpret_cast<f32x2 *>(dst + 64 * QUADS + 8 * g + 2 * r) = f32x2{O[SLABS - 2][r], O[SLABS - 1][r]};
        }
        if (g == 0) {
            ml[2 * w] = m;
            ml[2 * w + 1] = l;
        }
    }
    __syncthreads();
    for (int e = tid; e < F32_ROWS * CH; e += (int)blockDim.x) {
        const int rr = e / CH, c = e % CH;
        const int i = row0 + rr;
        if ((!SPLIT && i >= n) || 4 * c >= D) continue;
        float M = -FLT_MAX;
        for (int s = 0; s < S; ++s) M = fmaxf(M, ml[2 * (s * F32_ROWS + rr)]);
        float sum = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < S; ++s) {
            const int w = s * F32_ROWS + rr;
            const float f = expf(ml[2 * w] - M);  // 0 for a wavefront without keys
            sum += f * ml[2 * w + 1];
            o += f * *reinterpret_cast<const f32x4 *>(smem + w * LD + 4 * c);
        }
        if constexpr (SPLIT) {
            const int64_t row = ((int64_t)item.head * a.tiles.tiles + item.tile) * F32_ROWS + rr;
            *reinterpret_cast<f32x4 *>(a.partial + row * DP + 4 * c) = o;
            if (c == 0) a.stats[row] = f32x2{M, sum};
            continue;
        }
        if (a.lse != nullptr && c == 0) a.lse[(int64_t)i * H + h] = M + logf(sum);
        const float inv = 1.0f / sum;
        *reinterpret_cast<f32x4 *>(a.out + ((int64_t)i * H + h) * D + 4 * c) = o * inv;
    }
}

// out = sum_p f_p O_p / sum_p f_p l_p, f_p = exp(m_p - max m), parts in their order.  A thread: 4 dimensions of a row.
// Bound by latency: references, sums and results of BATCH parts are on their way at once (the references were read
// one after another before the first result was asked for; those beyond the first BATCH parts still are, and read again with
// their results), and workgroups are single wavefronts, which reach more CUs where rows are few.  Whole calls (us): 256 rows x 2 heads x 64, 1024 keys 11.5 -> 9.6, 200 x 1 x 96, 1000 keys 14.0 -> 11.7, 256 x
// 8 x 72, 1024 keys 17.9 -> 17.0, 1560 x 12 x 128, 3120 keys 157.7 -> 156.0.  BATCH: 4 for up to four parts (with 8: 17.2 and 25.6
// instead of 17.0 and 25.4 on 256 x 8 x 72 and 512 x 4 x 128), 8 beyond (with 4: 10.6 and 12.4 on the first two).
constexpr int COMBINE_F32_THREADS = 64;
template <int DP, int BATCH>
__global__ __launch_bounds__(COMBINE_F32_THREADS) void combine_f32_kernel(const attn_f32_args a)
{
    // (parts have rows for the area of one stream to hold: far below 2^32 threads)
    const unsigned chunks = (unsigned)a.D / 4u, tile_rows = (unsigned)(a.tiles.tiles * F32_ROWS);
    const unsigned g = blockIdx.x * COMBINE_F32_THREADS + threadIdx.x;
    const unsigned row = g / chunks;  // head-major
    const unsigned c = g - row * chunks, h = row / (unsigned)a.n, i = row - h * (unsigned)a.n;
    if (h >= (unsigned)a.H) return;
    const int64_t first = (int64_t)h * a.parts * tile_rows + i;
    f32x2 ml[BATCH];
    f32x4 v[BATCH];
    auto load = [&](int p0) {  // (past the last part: that one again, not used)
        auto at = [&](int b) -> int64_t { return first + (int64_t)(p0 + b < a.parts ? p0 + b : a.parts - 1) * tile_rows; };
#pragma unroll
        for (int b = 0; b < BATCH; ++b) ml[b] = a.stats[at(b)];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) v[b] = *reinterpret_cast<const f32x4 *>(a.partial + at(b) * DP + 4 * c);
    };
    load(0);
    float M = -FLT_MAX, sum = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < BATCH; ++b) M = fmaxf(M, ml[b][0]);
    for (int p = BATCH; p < a.parts; ++p) M = fmaxf(M, a.stats[first + (int64_t)p * tile_rows][0]);
    for (int p0 = 0;;) {
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
            if (p0 + b < a.parts) {
                const float f = expf(ml[b][0] - M);  // 0 for a part without a key that counts
                sum += f * ml[b][1];
                o += f * v[b];
            }
        p0 += BATCH;
        if (p0 >= a.parts) break;
        load(p0);
    }
    if (a.lse != nullptr && c == 0) a.lse[(int64_t)i * a.H + h] = (float)((double)M + log((double)sum));
    const float inv = 1.0f / sum;
    *reinterpret_cast<f32x4 *>(a.out + ((int64_t)i * a.H + h) * a.D + 4 * c) = o * inv;
}

}  // namespace ifx
