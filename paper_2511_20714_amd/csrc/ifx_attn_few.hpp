// bf16 block attention for gfx950 where the query rows are too few to occupy the chip: 32 rows per
// workgroup, the keys dealt to its 8 wavefronts.
//
// The same operation and arithmetic as the unbounded path of ifx_attn_bf16.hpp (running reference,
// output divided by the sum of the weights as rounded to bf16; the log-sum-exp from a second sum, of
// the fp32 exponentials); operand layouts as described there.
//
// Shape of the computation
//   A call of H heads x ceil(n / 32) row tiles that do not fill 256 CUs with 256-row workgroups is
//   bound by the serial chain over its keys.  Here every row tile is a workgroup of its own and
//   wavefront w takes the 32-key subtiles w, w + 8, ... of the key set (cached keys, then the current
//   block): the chain is an eighth as long.  The partial results (output, reference, sum) are put
//   together through LDS at the end, in a fixed order.  The price is that a subtile's keys are
//   read once per 32 rows instead of once per 256, 128 KiB per step of the 8 wavefronts, so larger
//   calls keep the other kernel (attn_groups_for).
//   Nothing but the end is shared between wavefronts, so the loop has no barrier.  K goes through 8 KiB
//   of LDS of the wavefront's own: a subtile is copied in by direct global->LDS loads, its operands
//   are read into registers, and the copy of the wavefront's next subtile starts at once into the same
//   place, under the whole of the current step.  Cached V lies as the PV product needs it and goes
//   straight into registers, asked for as soon as the registers' last product has been issued (through
//   LDS like K: 2 % slower, 18 % with an fp8 cache); only the current block's V needs LDS, for the
//   transposing reads.  fp8 codes are widened (exactly) as they are read.
//   Measured (5 heads x 1560 rows, 10920 keys): 64 us = 1.5 us per step of a wavefront's 43, against 176
//   with one key group; fp8 cache 60 us.  Counters: matrix pipes 30 % busy, VALU 34 %, LDS 10 %, no bank
//   conflicts, 1.40 GB read from the L2s (22 TB/s); wavefronts spend 24 % of their cycles at wait counts,
//   32 % waiting to issue.  No unit is full: a wavefront has one subtile's loads in flight and
//   its softmax between two products, and two wavefronts per SIMD do not cover that.
//   A CU's L1 passes on those 128 KiB a step at 45 and more of its 64 bytes per cycle.  Where CUs would be idle, 2 or 4 workgroups
//   share a row tile, each with all its scores and 2 slabs or 1 of 32 output dimensions (SLABS, few_slab_groups): 96 or 80 KiB
//   a step, 0.87 and 0.70 us where one workgroup takes 1.13, the same bytes per cycle; over codes 0.95 and 0.85, each workgroup
//   widening them.  264 rows, 2 heads, 792 keys 9.6 -> 7.7 us (21 with one group), four steps and the launch: matrix pipes 2 % busy,
//   wavefronts 47 % of their cycles at wait counts.  (Descriptors made once, not for every copy, and copies behind the last
//   subtile that touch no memory are worth 3 % over codes, and with one workgroup to a bf16 tile nothing.)  Where tiles are at most half a round and the keys many, those come in parts (SPLIT,
//   attn_plan_for): 1 head x 1560 rows, 10920 keys 54 -> 21.6 us.
#pragma once
#include "ifx_attn_bf16.hpp"

namespace ifx {

constexpr int FEW_WAVES = 8;
constexpr int FEW_ROWS = 32;
constexpr int FEW_WAVE_LDS = 16384;       // K subtile, V subtile of the current block
constexpr int few_ld(int slabs) { return 32 * slabs + 4; }  // floats between the rows of a partial result: 16-byte accesses of 16 rows hit 16 bank groups
constexpr int FEW_PARTIAL_LDS = FEW_WAVES * FEW_ROWS * few_ld(4) * 4;
constexpr int FEW_LDS_BYTES = FEW_PARTIAL_LDS + FEW_WAVES * FEW_ROWS * 16;  // partial results take the tiles' place, then references and sums
static_assert(FEW_LDS_BYTES >= FEW_WAVES * FEW_WAVE_LDS && FEW_LDS_BYTES <= 160 * 1024, "");

struct attn_few_args {
    const __bf16 *q;                  // [n, H, 128]
    const unsigned char *kc, *vt;     // the layer's K region and V region (see attn_bf16_args)
    const __bf16 *kb, *vb;            // the current block [n, H, 128], or nullptr when nb == 0
    __bf16 *out;                      // [n, H, 128]
    float *lse;                       // [n, H] or nullptr
    int n, H;
    int C, nb;                        // cached keys (whole blocks of n), keys of the current block (n or 0); C + nb > 0
    int64_t k_tokens, v_tokens;
    float scale_log2;
    row_tiles tiles;                  // workgroup -> (head, row tile), see ifx_launch.hpp
    ifx_key_blocks blocks;
    attn_split split;                 // SPLIT instantiation only, see ifx_launch.hpp: tiles is then of heads * parts heads
    f32x4 *partial, *stats;           // its partial results, as ifx_split.hpp lays them out
};

// TABLE: the cached keys are the blocks of a selection in a caller-given order.
// SPLIT: a row tile's keys are dealt to split.parts workgroups, each a run of subtiles; `head` of the launch
// counts (head, part) pairs.  Their results are left for combine_kernel (ifx_split.hpp).
// SLABS: the slabs of 32 output dimensions that a workgroup takes; 4 / SLABS workgroups share a row tile
// (`tile` of the launch counts them), each with all scores and its own slabs' values: few_slabs.
template <bool FP8, bool TABLE, bool SPLIT = false, int SLABS = 4>
__global__ __launch_bounds__(64 * FEW_WAVES, 1) void attn_few_kernel(const attn_few_args a)
{
    static_assert(!SPLIT || SLABS == 4, "");
    constexpr int KEYB = FP8 ? BF_D : BF_D * 2;  // bytes of a cached key row, and of a key's share of its V granule
    constexpr int COPIES = FP8 ? 4 : 8;          // copy instructions of a cached K subtile (of the block: always 8)
    constexpr int V_LOADS = 2 * SLABS;           // load or copy instructions of a V subtile
    constexpr int V_ROW = 64 * SLABS, V_CHUNKS = 4 * SLABS;  // bytes, and 16-byte chunks, of a V row's slabs
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    const int n = a.n, H = a.H;
    const row_tile item = row_tile_of(a.tiles, SPLIT ? H * a.split.parts : H, blockIdx.x);
    if (item.head < 0) return;
    const int head = SPLIT ? item.head / a.split.parts : item.head, part = SPLIT ? item.head - head * a.split.parts : 0;
    const int row0 = item.tile / (4 / SLABS) * FEW_ROWS, slab0 = item.tile % (4 / SLABS) * SLABS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, lh = lane >> 5;
    const float c2 = a.scale_log2;
    unsigned char *const ktile = lds + wave * FEW_WAVE_LDS, *const vtile = ktile + FEW_WAVE_LDS / 2;

    // A subtile is 32 consecutive keys of the cached ones, or of the current block (fewer at the end of
    // either).  They are read through buffer descriptors that end with the last cached key (with a block table: with
    // the region) and the block's last row; rows behind that read as zero, touch no memory and are masked.
    // A subtile's place is a scalar offset: descriptors and lane offsets are worked out once (a descriptor for every
    // subtile and copy was half of a step's scalar instructions).
    const int cached_keys = TABLE ? a.blocks.count * n : a.C;
    const int cached_subs = (cached_keys + 31) >> 5;
    const int all_subs = cached_subs + ((a.nb + 31) >> 5);
    const int first_sub = SPLIT ? part_begin(all_subs, a.split.parts, part) : 0, subs = SPLIT ? part_begin(all_subs, a.split.parts, part + 1) : all_subs;
    const int own_sub = first_sub + wave;
    auto keys_from = [&](int sub) IFX_INLINE -> int { return sub < cached_subs ? cached_keys - 32 * sub : a.nb - 32 * (sub - cached_subs); };
    const uintptr_t kc = (uintptr_t)a.kc + (uintptr_t)head * (uintptr_t)a.k_tokens * KEYB;
    const uintptr_t vc = (uintptr_t)a.vt + (uintptr_t)head * (uintptr_t)a.v_tokens * KEYB;
    const uintptr_t kb = (uintptr_t)a.kb + (uintptr_t)head * (BF_D * 2), vb = (uintptr_t)a.vb + (uintptr_t)head * (BF_D * 2);
    const int pitch = H * (BF_D * 2);
    const int l16 = lane & 15, g = lane >> 4;
    const int blk_bytes = a.nb > 0 ? (a.nb - 1) * pitch + BF_D * 2 : 0;
    const __amdgpu_buffer_rsrc_t rs_k = __builtin_amdgcn_make_buffer_rsrc((void *)kc, 0, TABLE ? (int)(a.k_tokens * KEYB) : a.C * KEYB, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_v = __builtin_amdgcn_make_buffer_rsrc((void *)vc, 0, TABLE ? (int)(a.v_tokens * KEYB) : a.C * KEYB, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_kb = __builtin_amdgcn_make_buffer_rsrc((void *)kb, 0, blk_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_vb = __builtin_amdgcn_make_buffer_rsrc((void *)vb, 0, blk_bytes, 0x00020000);
    constexpr int NOWHERE = 1 << 30;  // a scalar offset behind every descriptor's end

    // With a table a subtile may begin and end inside blocks and hold several (a subtile per block left
    // 8-token blocks with three quarters of every product empty: 60 listed ones, 64 heads: 15.7 us, now 8.5;
    // 13.0 with one key group).
    // Blocks are multiples of 8 tokens, so each of its four granules lies in one: four scalar byte
    // offsets into the head's regions, 2^30 past the last key (beyond any region, reads as zero).
    // 64 entries of the list from tab_first on are kept one per lane, a lookup is a lane read; a wavefront
    // walks its subtiles in order, so the 64 move along a longer list.
    struct granules {
        int at[4];
    };
    int tab = 0, tab_first = 0;
    auto load_entries = [&](int e) IFX_INLINE {
        tab_first = e;
        if (e + lane < a.blocks.count) {  // (two plain indexed reads, see ifx_attn_bf16.hpp)
            if (a.blocks.list != nullptr)
                tab = a.blocks.list[e + lane];
            else
                tab = a.blocks.first[e + lane];
        }
    };
    if constexpr (TABLE) load_entries(0);
    const int block_granules = n >> 3;
    auto granules_of = [&](int sub, bool some) IFX_INLINE -> granules {
        granules r = {};
        if constexpr (TABLE) {
            if (sub >= cached_subs) return r;
            if (!some) return {{NOWHERE, NOWHERE, NOWHERE, NOWHERE}};
            int e = 4 * sub / block_granules, w = 4 * sub - e * block_granules;
            if (e + 3 >= tab_first + 64) load_entries(e);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                r.at[k] = e < a.blocks.count ? (__builtin_amdgcn_readlane(tab, e - tab_first) + 8 * w) * KEYB : NOWHERE;
                if (++w == block_granules) {
                    w = 0;
                    ++e;
                }
            }
        }
        return r;
    };
    // K: row r (256 bytes), 16-byte chunk c at place c ^ (r % 16); codes: 128-byte rows, place c ^ (r % 8)
    int k_lane[4], kb_lane[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int chunk = (l16 ^ (4 * x + g)) << 4;
        k_lane[x] = FP8 ? (lane >> 3) * KEYB + (((lane & 7) ^ (lane >> 3)) << 4) : g * KEYB + chunk;
        kb_lane[x] = g * pitch + chunk;
    }
    // (some == false: instructions that touch no memory, so that the wait counts know what is in flight)
    auto copy_k = [&](int sub, const granules &from, bool some) IFX_INLINE {
        if (sub < cached_subs) {
            const int at = TABLE ? 0 : some ? 32 * sub * KEYB : NOWHERE;  // (a table's offsets say so themselves)
#pragma unroll
            for (int x = 0; x < COPIES; ++x) {
                // (not const: with arguments that depend on FP8 the host pass rejects the builtin's size, silently)
                int off_v, off_s;
                off_v = k_lane[x & 3];
                off_s = at + (!TABLE ? 1024 * x : FP8 ? from.at[x & 3] : from.at[x >> 1] + 1024 * (x & 1));
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_k, (lptr_t)(ktile + 1024 * x), 16, off_v, off_s, 0, 0);
            }
            return;
        }
        const int at = some ? 32 * (sub - cached_subs) * pitch : NOWHERE;
#pragma unroll
        for (int x = 0; x < 8; ++x)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_kb, (lptr_t)(ktile + 1024 * x), 16, kb_lane[x & 3], at + 4 * x * pitch, 0, 0);
    };
    // V: cached granules straight into registers (a lane's 8 keys of a dimension are 16 contiguous bytes,
    // 8 as codes); rows of the current block into LDS, chunk c of row r's slabs at place c ^ 4 (r % 4) (two slabs:
    // c ^ 4 (r / 2 % 2)), so that four rows lie in four quarters of the banks.  V_LOADS instructions either way.
    typedef uint32_t raw_u32x4 __attribute__((__vector_size__(16)));
    typedef uint32_t raw_u32x2 __attribute__((__vector_size__(8)));
    typedef typename std::conditional<FP8, raw_u32x2, raw_u32x4>::type stored_v;
    stored_v Vc[V_LOADS];
    auto row_swizzle = [&](int r4) IFX_INLINE -> int { return SLABS == 4 ? r4 : SLABS == 2 ? r4 >> 1 : 0; };  // r4: the row modulo 4
    const int v_lane = lq * (KEYB / 16) + (TABLE ? 0 : lh * (8 * KEYB));
    const int vb_row = lane / V_CHUNKS, vb_lane = vb_row * pitch + 64 * slab0 + (((lane % V_CHUNKS) ^ (row_swizzle(vb_row & 3) << 2)) << 4);
    auto load_v = [&](int sub, const granules &from, bool some) IFX_INLINE {
        if (sub < cached_subs) {
            const int at = (TABLE ? 0 : some ? 32 * sub * KEYB : NOWHERE) + slab0 * (2 * KEYB);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                // lanes 0 .. 31: granule 2 t, lanes 32 .. 63: the next
                const int off_v = TABLE ? v_lane + (lh ? from.at[2 * t + 1] : from.at[2 * t]) : v_lane;
                const int step = at + (TABLE ? 0 : t * (16 * KEYB));
#pragma unroll
                for (int sl = 0; sl < SLABS; ++sl) {
                    if constexpr (FP8)
                        Vc[t * SLABS + sl] = __builtin_amdgcn_raw_buffer_load_b64(rs_v, off_v, step + sl * (2 * KEYB), 0);
                    else
                        Vc[t * SLABS + sl] = __builtin_amdgcn_raw_buffer_load_b128(rs_v, off_v, step + sl * (2 * KEYB), 0);
                }
            }
            return;
        }
        const int at = some ? 32 * (sub - cached_subs) * pitch : NOWHERE;
#pragma unroll
        for (int x = 0; x < V_LOADS; ++x)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_vb, (lptr_t)(vtile + 1024 * x), 16, vb_lane, at + (64 / V_CHUNKS) * x * pitch, 0, 0);
    };

    if (own_sub < subs) {
        const granules from = granules_of(own_sub, true);
        copy_k(own_sub, from, true);
        load_v(own_sub, from, true);
    }
    bf16x8 Q[8];
    {
        const int qi = row0 + lq;
        const bf16x8 *qp = reinterpret_cast<const bf16x8 *>(a.q + ((int64_t)(qi < n ? qi : n - 1) * H + head) * BF_D);
#pragma unroll
        for (int s = 0; s < 8; ++s) Q[s] = qp[2 * s + lh];
    }

    // operand addresses (see ifx_attn_bf16.hpp)
    const int pkey = (lq & 16) | ((lq & 4) << 1) | ((lq & 8) >> 1) | (lq & 3);
    const int kz = lh ^ (pkey & 15);
    int vtoff[SLABS];
    {
        const int base = (8 * (g >> 1) + (l16 >> 2)) * V_ROW + (2 * (g & 1) + ((l16 & 3) >> 1)) * 16 + 8 * (l16 & 1);
#pragma unroll
        for (int sl = 0; sl < SLABS; ++sl) vtoff[sl] = base + ((sl ^ row_swizzle(l16 >> 2)) << 6);
    }
    auto widen8 = [&](const raw_u32x2 &c) IFX_INLINE -> bf16x8 {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        u32x4 r;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            r[2 * w] = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)c[w], 1.0f, false));
            r[2 * w + 1] = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)c[w], 1.0f, true));
        }
        return __builtin_bit_cast(bf16x8, r);
    };

    f32x16 O[SLABS];
#pragma unroll
    for (int sl = 0; sl < SLABS; ++sl)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[sl][r] = 0.0f;
    float m_used = BF_NO_REFERENCE;  // reference of the exponentials (scaled log2 units)
    // this lane's share of the row sum: of the weights as rounded to bf16, which is what the PV product
    // uses (the output's denominator), and, where the log-sum-exp is asked for, of the fp32 exponentials
    float l_acc[4] = {0.f, 0.f, 0.f, 0.f}, e_acc[4] = {0.f, 0.f, 0.f, 0.f};
    const bool with_lse = a.lse != nullptr;

    for (int sub = own_sub; sub < subs; sub += FEW_WAVES) {
        const bool more = sub + FEW_WAVES < subs;
        const int next = more ? sub + FEW_WAVES : sub;
        const bool cached = sub < cached_subs;
        const int keys = keys_from(sub);
        bf16x8 A[8];
        // K: only V's loads, issued behind it, may still be on their way
        __builtin_amdgcn_s_waitcnt(0x0F70 | V_LOADS);
        if (FP8 && cached) {
            raw_u32x2 c[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) c[s] = *reinterpret_cast<const raw_u32x2 *>(ktile + pkey * 128 + ((s ^ (pkey & 7)) << 4) + lh * 8);
#pragma unroll
            for (int s = 0; s < 8; ++s) A[s] = widen8(c[s]);
        } else {
#pragma unroll
            for (int s = 0; s < 8; ++s) A[s] = *reinterpret_cast<const bf16x8 *>(ktile + pkey * 256 + (((2 * s) ^ kz) << 4));
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the operands are in registers, the tile is free
        __builtin_amdgcn_sched_barrier(0);
        const granules from = granules_of(next, more);
        copy_k(next, from, more);
        __builtin_amdgcn_s_setprio(1);  // (MFMAs first: 5 % faster)
        f32x16 S = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 8; ++s) S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[s], Q[s], S, 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);

        // register r of S is key 16 (r / 8) + 8 lh + r % 8 of the subtile
        if (keys < 32) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (16 * (r >> 3) + 8 * lh + (r & 7) >= keys) S[r] = -INFINITY;
        }
        auto raise = [&]() IFX_INLINE {
            float t = S[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) t = fmaxf(t, S[r]);
            t = max_across_halves(t) * c2;
            const float m_next = t > m_used ? t + BF_HEADROOM : m_used;  // (a large reference would cost the log-sum-exp bits)
            const float alpha = __builtin_amdgcn_exp2f(m_used - m_next);  // 1 where unchanged, 0 at the start
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                l_acc[e] *= alpha;
                e_acc[e] *= alpha;
            }
#pragma unroll
            for (int sl = 0; sl < SLABS; ++sl)
#pragma unroll
                for (int r = 0; r < 16; ++r) O[sl][r] *= alpha;
            m_used = m_next;
        };
        bf16x8 P[2];
        f32x8 E[2];
        auto exps = [&]() IFX_INLINE {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int e = 0; e < 8; ++e) E[t][e] = __builtin_amdgcn_exp2f(fmaf(S[8 * t + e], c2, -m_used));
                P[t] = __builtin_convertvector(E[t], bf16x8);
            }
        };
        bool redo = sub == own_sub;  // no reference yet
        if (!redo) {
            exps();
            // a score a whole unit above the reference: an exponential of 2 or more, i.e. a top exponent bit
            const u32x4 x = __builtin_bit_cast(u32x4, P[0]), y = __builtin_bit_cast(u32x4, P[1]);
            const uint32_t o = (x[0] | x[1] | x[2]) | (x[3] | y[0] | y[1]) | (y[2] | y[3]);
            redo = __any((o & 0x40004000u) != 0u);
        }
        if (__builtin_expect(redo, 0)) {
            raise();
            exps();
        }
        bf16x8 V[V_LOADS];
        if (cached) {
#pragma unroll
            for (int o = 0; o < V_LOADS; ++o) {
                if constexpr (FP8)
                    V[o] = widen8(Vc[o]);
                else
                    V[o] = __builtin_bit_cast(bf16x8, Vc[o]);
            }
        } else {
            __builtin_amdgcn_s_waitcnt(0x0F70 | COPIES);  // only the K copies issued in this step may still be on their way
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int sl = 0; sl < SLABS; ++sl) {
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lptr_t)(vtile + vtoff[sl] + (16 * t) * V_ROW));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lptr_t)(vtile + vtoff[sl] + (16 * t + 4) * V_ROW));
                    typedef short s16x8 __attribute__((ext_vector_type(8)));
                    V[t * SLABS + sl] = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the tile is free
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int sl = 0; sl < SLABS; ++sl) O[sl] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(V[t * SLABS + sl], P[t], O[sl], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_v(next, from, more);
#pragma unroll
        for (int r = 0; r < 16; ++r) l_acc[r & 3] += (float)P[r >> 3][r & 7];
        if (with_lse) {
#pragma unroll
            for (int r = 0; r < 16; ++r) e_acc[r & 3] += E[r >> 3][r & 7];
        }
    }

    // ---- put the wavefronts' shares together: partial outputs, references and sums through LDS
    const float l_half = (l_acc[0] + l_acc[1]) + (l_acc[2] + l_acc[3]);
    const float l_own = l_half + __shfl_xor(l_half, 32);
    const float e_half = (e_acc[0] + e_acc[1]) + (e_acc[2] + e_acc[3]);
    const float e_own = e_half + __shfl_xor(e_half, 32);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the copies behind the last subtile have landed
    __syncthreads();
    constexpr int LD = few_ld(SLABS);
    float *const partial = reinterpret_cast<float *>(lds);
    f32x4 *const stats = reinterpret_cast<f32x4 *>(lds + FEW_WAVES * FEW_ROWS * LD * 4);
    {
        // register r of O[sl] is d = 32 sl + 8 (r / 4) + 4 lh + r % 4 of query lq
        float *dst = partial + (wave * FEW_ROWS + lq) * LD + 4 * lh;
#pragma unroll
        for (int sl = 0; sl < SLABS; ++sl)
#pragma unroll
            for (int r = 0; r < 16; r += 4)
                *reinterpret_cast<f32x4 *>(dst + 32 * sl + 2 * r) = f32x4{O[sl][r], O[sl][r + 1], O[sl][r + 2], O[sl][r + 3]};
        if (lh == 0) stats[wave * FEW_ROWS + lq] = f32x4{m_used, l_own, e_own, 0.f};
    }
    __syncthreads();
    // row of the tile, QUADS times 4 of its output dimensions (one slab: half the threads)
    constexpr int QUADS = SLABS == 4 ? 2 : 1, PER_ROW = 8 * SLABS / QUADS;
    const int rr = SPLIT ? tid & 31 : tid / PER_ROW, c = SPLIT ? tid >> 5 : tid % PER_ROW;
    const int i = row0 + rr;
    if (!SPLIT && (i >= n || rr >= FEW_ROWS)) return;
    float M = BF_NO_REFERENCE;
#pragma unroll
    for (int s = 0; s < FEW_WAVES; ++s) M = fmaxf(M, stats[s * FEW_ROWS + rr][0]);
    float sum = 0.f, sum_e = 0.f;
    f32x4 o[QUADS];
#pragma unroll
    for (int k = 0; k < QUADS; ++k) o[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < FEW_WAVES; ++s) {
        const f32x4 ml = stats[s * FEW_ROWS + rr];
        const float w = __builtin_amdgcn_exp2f(ml[0] - M);  // 0 for a wavefront without keys
        sum += w * ml[1];
        sum_e += w * ml[2];
        const f32x4 *src = reinterpret_cast<const f32x4 *>(partial + (s * FEW_ROWS + rr) * LD + 4 * QUADS * c);
#pragma unroll
        for (int k = 0; k < QUADS; ++k) {
            const f32x4 x = src[k];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[k][e] += w * x[e];
        }
    }
    if constexpr (SPLIT) {
        // where the accumulators of a 32-row wavefront would hold them: dimensions 8 c .. + 3 in lane rr, + 4 .. + 7 in lane rr + 32
        const int64_t unit = split_unit_of(a.split, head, part, item.tile);
        f32x4 *const dst = a.partial + unit * SPLIT_UNIT_CHUNKS + c * 64 + rr;
        dst[0] = o[0];
        dst[32] = o[QUADS - 1];
        if (c == 0) a.stats[unit * 32 + rr] = f32x4{M, sum, sum_e, 0.f};
        return;
    }
    if (with_lse && c == 0 && slab0 == 0) a.lse[(int64_t)i * H + head] = (M + __builtin_amdgcn_logf(sum_e)) * 0.6931471805599453f;
    const float inv = 1.0f / sum;
    __bf16 *const op = a.out + ((int64_t)i * H + head) * BF_D + 32 * slab0 + 4 * QUADS * c;
    if constexpr (QUADS == 2) {
        f32x8 both = __builtin_shufflevector(o[0], o[1], 0, 1, 2, 3, 4, 5, 6, 7);
        both *= inv;
        *reinterpret_cast<bf16x8 *>(op) = __builtin_convertvector(both, bf16x8);
    } else {
        o[0] *= inv;
        *reinterpret_cast<bf16x4 *>(op) = __builtin_convertvector(o[0], bf16x4);
    }
}

}  // namespace ifx
