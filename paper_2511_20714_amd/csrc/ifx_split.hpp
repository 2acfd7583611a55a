// Puts together the partial results of attention whose keys were dealt to several workgroups
// (attn_bf16_kernel's SPLIT instances): out = sum_p w_p O_p / sum_p w_p l_p, w_p = 2^(m_p - max m).
//
// A launch of its own behind the attention kernel: the stream's order is the only synchronisation.  (Letting the
// last workgroup of a tile do it was measured on stand-ins of 256 workgroups with 16 KiB each: 6.4 us for the
// two launches, 15 with agent-scope stores and a counter, 60 with plain stores and a release fence, which
// writes back the whole L2.)  Bound by the memory-side cache's latency and rate: the partials of 1560 rows x 12 heads in
// three parts are 29 MB, 7.3 us (wavefronts 64 % of their cycles at wait counts); 1560 x 1 in five 4.0.
#pragma once
#include "ifx_attn_bf16.hpp"

namespace ifx {

struct combine_args {
    const f32x4 *partial;
    const f32x4 *stats;
    __bf16 *out;  // [n, H, 128]
    float *lse;   // [n, H] or nullptr
    int n, H;
    attn_split split;
};

constexpr int COMBINE_MOST_WAVES = 4, COMBINE_MOST_BATCH = 4;
inline int combine_waves(int parts) { return parts <= COMBINE_MOST_BATCH ? 1 : COMBINE_MOST_WAVES; }
inline int combine_batch(int parts)
{
    const int each = (parts + combine_waves(parts) - 1) / combine_waves(parts);
    return each < COMBINE_MOST_BATCH ? each : COMBINE_MOST_BATCH;
}

// A workgroup = one slab of 32 dimensions of one unit's 32 rows, the parts dealt to its wavefronts (up to four: one
// wavefront, which exchanges nothing); lanes hold what the accumulators held.  BATCH: parts that a wavefront has on their way at
// once, as many as it takes up to four: 16 parts of four wavefronts (four of every wavefront's one or two before, some loaded four times: 30 layers of 1560 x 12 x 10920
// 3260 -> 3245 us, 800 x 12 x 6400 43.4 -> 42.9, 400 x 2 x 3200 13.1 -> 13.0, x 1 12.4 -> 12.2).  Streaming the partial results past
// the caches gains nothing.  The sums are taken in a fixed order, whichever workgroup finished first.
template <int BATCH>
__global__ __launch_bounds__(64 * COMBINE_MOST_WAVES) void combine_kernel(const combine_args a)
{
    __shared__ float shared[COMBINE_MOST_WAVES - 1][19][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int lq = lane & 31, lh = lane >> 5;
    const int unit = blockIdx.x >> 2, sl = blockIdx.x & 3;
    const int split_head = unit / a.split.row_tiles, tile = unit - split_head * a.split.row_tiles;
    const int64_t first = split_unit_of(a.split, split_head, 0, tile), step = a.split.row_tiles;
    const f32x4 *const st = a.stats + first * 32 + lq;
    const f32x4 *const src = a.partial + first * SPLIT_UNIT_CHUNKS + sl * 256 + lane;
    float m = BF_NO_REFERENCE, l = 0.f, sum_e = 0.f;
    f32x16 R;
#pragma unroll
    for (int r = 0; r < 16; ++r) R[r] = 0.f;
    auto add = [&](float m_other, float l_other, float e_other, auto &&value) IFX_INLINE {
        const float m_next = fmaxf(m, m_other);
        const float w = __builtin_amdgcn_exp2f(m - m_next), w_other = __builtin_amdgcn_exp2f(m_other - m_next);  // 0: no key that counts
        m = m_next;
        l = w * l + w_other * l_other;
        sum_e = w * sum_e + w_other * e_other;
#pragma unroll
        for (int r = 0; r < 16; ++r) R[r] = w * R[r] + w_other * value(r);
    };
    for (int p0 = wave; p0 < a.split.parts; p0 += BATCH * waves) {
        f32x4 v[BATCH][4];
        f32x4 ml[BATCH];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const int p = p0 + b * waves < a.split.parts ? p0 + b * waves : p0;
            ml[b] = st[p * step * 32];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[b][r] = src[p * step * SPLIT_UNIT_CHUNKS + 64 * r];
        }
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
            if (p0 + b * waves < a.split.parts) add(ml[b][0], ml[b][1], ml[b][2], [&](int r) IFX_INLINE { return v[b][r >> 2][r & 3]; });
    }
    if (wave > 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) shared[wave - 1][r][lane] = R[r];
        shared[wave - 1][16][lane] = m;
        shared[wave - 1][17][lane] = l;
        shared[wave - 1][18][lane] = sum_e;
    }
    __syncthreads();
    if (wave > 0) return;
    for (int w = 0; w < waves - 1; ++w) add(shared[w][16][lane], shared[w][17][lane], shared[w][18][lane], [&](int r) IFX_INLINE { return shared[w][r][lane]; });
    const int head = a.split.whole_heads + split_head, qi = tile * 32 + lq;
    if (a.lse != nullptr && sl == 0 && lh == 0 && qi < a.n)
        a.lse[(int64_t)qi * a.H + head] = (m + __builtin_amdgcn_logf(sum_e)) * 0.6931471805599453f;
    store_slab(a.out + ((int64_t)(qi < a.n ? qi : a.n - 1) * a.H + head) * BF_D + 32 * sl, R, 1.0f / l, lh, qi < a.n);
}

// (parts >= 2)
inline void (*combine_kernel_of(int parts))(const combine_args)
{
    switch (combine_batch(parts)) {
    case 2: return combine_kernel<2>;
    case 3: return combine_kernel<3>;
    default: return combine_kernel<4>;
    }
}

}  // namespace ifx
