"""GPU parity of fp32 attention whose keys are dealt to several workgroups per row tile (8 and 4 wavefronts each, padded
head dimensions, ragged rows and keys, listed blocks that fill subtiles or are gathered, no current block), and of the
kernel that takes its products apart into bf16 pieces."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_20714_amd import binding as ifx
from paper_2511_20714_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,H,D,cap,blocks,with_block,parts", [
    (256, 2, 64, 3, None, True, 8),
    (250, 2, 40, 5, None, True, 8),
    (100, 3, 72, 12, [11, 3, 0, 5, 7, 1, 2, 9, 8], False, 7),               # blocks of six subtiles and four keys
    (400, 4, 128, 4, None, True, 5),                                       # 500 workgroups of 4 wavefronts
    (17, 2, 24, 150, list(range(149, -1, -1)), True, 37),                  # a subtile of one key in every block
    (5, 3, 64, 400, list(range(0, 400, 2)) + list(range(1, 400, 2)), True, 15),  # subtiles gathered from several blocks
    (1560, 6, 128, 2, [1, 0], True, 3),                                    # 588 row tiles
])
def test_f32_key_parts(gpu_device, n, H, D, cap, blocks, with_block, parts):
    dev = gpu_device
    listed = cap if blocks is None else len(blocks)
    subs = listed * n if blocks is None or n < 16 else listed * ((n + 15) // 16) * 16  # of 16 keys; blocks of 16 and more begin one of their own
    assert ifx.ifx_attention_f32_key_parts(n, H, D, subs + (((n + 15) // 16) * 16 if with_block else 0), blocks is not None) == (parts, 16)
    with ifx.KVCache(1, H, D, cap * n, n, ifx.IFX_F32) as cache:
        oc = oracle.BlockCacheOracle(cap)
        for b in range(cap):
            _, k, v = synth.draw_qkv(71, b, 0, 0, n, H, D, torch.float32, dev)
            cache.commit(0, k, v)
            oc.commit(synth.to_f64_numpy(k), synth.to_f64_numpy(v))
        q, k, v = synth.draw_qkv(71, 999, 0, 0, n, H, D, torch.float32, dev)
        if not with_block:
            k = v = None
        out = torch.full((n + 1, H, D), float("nan"), device=dev)
        lse = torch.full((n + 1, H), float("nan"), device=dev)
        cache.attention_blocks(0, q, k, v, blocks, out[:n], lse[:n])
        torch.cuda.synchronize()
        assert torch.isfinite(out[:n]).all() and torch.isfinite(lse[:n]).all() and torch.isnan(out[n]).all() and torch.isnan(lse[n]).all()
        kc, vc = oc.logical() if blocks is None else oc.logical([(b, 1) for b in blocks])
        r = np.unique(np.concatenate([np.arange(min(n, 20)), np.arange(max(0, n - 20), n), np.random.default_rng(1).integers(0, n, 20)]))
        rows, heads = np.repeat(r, H), np.tile(np.arange(H), len(r))
        want, want_lse = oracle.attention_rows(synth.to_f64_numpy(q), kc, vc, None if k is None else synth.to_f64_numpy(k),
                                               None if v is None else synth.to_f64_numpy(v), rows, heads)
        assert np.abs(synth.to_f64_numpy(out[:n])[rows, heads] - want).max() <= 1e-5
        assert np.abs(synth.to_f64_numpy(lse[:n])[rows, heads] - want_lse).max() <= 2e-5


def rows_of(n, H):
    r = np.unique(np.concatenate([np.arange(12), np.arange(n - 12, n), np.random.default_rng(1).integers(0, n, 12)]))
    return np.repeat(r, H), np.tile(np.arange(H), len(r))


@pytest.mark.parametrize("n,H,D,cap,with_block,whole", [
    (1560, 3, 128, 1, True, False),
    (1000, 8, 40, 4, True, False),      # padded to 64; 8 rows past a wavefront's, 8 keys past a tile
    (705, 8, 72, 5, False, False),      # to 128; one row, one key over
    (520, 16, 64, 4, True, False),      # workgroups of 6 and 5 wavefronts
    (250, 130, 128, 2, True, True),     # no parts: 130 workgroups
])
def test_f32_in_pieces(gpu_device, n, H, D, cap, with_block, whole):
    """256-row workgroups: no element further from the oracle than the bound of the other kernel."""
    dev = gpu_device
    parts, rows = ifx.ifx_attention_f32_key_parts(n, H, D, cap * n + (n if with_block else 0))
    assert rows == 256 and (parts == 1) == whole
    hs = np.array([0, H - 1])
    with ifx.KVCache(1, H, D, cap * n, n, ifx.IFX_F32) as cache:
        ks, vs = [], []
        for b in range(cap):
            _, k, v = synth.draw_qkv(73, b, 0, 0, n, H, D, torch.float32, dev)
            cache.commit(0, k, v)
            ks.append(k), vs.append(v)
        q, k, v = synth.draw_qkv(73, 999, 0, 0, n, H, D, torch.float32, dev)
        out = torch.full((n + 1, H, D), float("nan"), device=dev)
        lse = torch.full((n + 1, H), float("nan"), device=dev)
        cache.attention_blocks(0, q, k if with_block else None, v if with_block else None, None, out[:n], lse[:n])
        torch.cuda.synchronize()
    if with_block:
        ks.append(k), vs.append(v)
    assert torch.isfinite(out[:n]).all() and torch.isfinite(lse[:n]).all() and torch.isnan(out[n]).all() and torch.isnan(lse[n]).all()
    rows, heads = rows_of(n, 2)
    want, want_lse = oracle.attention_rows(synth.to_f64_numpy(q)[:, hs], np.concatenate([synth.to_f64_numpy(k)[:, hs] for k in ks]),
                                           np.concatenate([synth.to_f64_numpy(v)[:, hs] for v in vs]), None, None, rows, heads)
    assert np.abs(synth.to_f64_numpy(out[:n])[rows, hs[heads]] - want).max() <= 1e-5
    assert np.abs(synth.to_f64_numpy(lse[:n])[rows, hs[heads]] - want_lse).max() <= 2e-5


@pytest.mark.parametrize("what", ["tiny values", "large values", "tiny queries, large keys", "-inf keys", "overflowing keys"])
def test_f32_in_pieces_beyond_bf16s_ease(gpu_device, what):
    """Values whose pieces are subnormal or near the largest number, queries and keys of opposite scales, keys whose
    scores are -inf (an infinite element, or a finite product that overflows): as fp32 arithmetic has them."""
    dev, n, H, D, cap = gpu_device, 1560, 3, 128, 1
    assert ifx.ifx_attention_f32_key_parts(n, H, D, 2 * n)[1] == 256
    (_, k0, v0), (q, k1, v1) = (synth.draw_qkv(79, b, 0, 0, n, H, D, torch.float32, dev) for b in (0, 999))
    vscale, count = 1.0, np.arange(2 * n)
    if what == "tiny values":
        vscale = 2.0 ** -110  # last pieces down to 2^-128 of elements near 1
    elif what == "large values":
        vscale = 2.0 ** 112  # sums of 3120 weights of up to e^2 stay below 2^127
    elif what == "tiny queries, large keys":
        q, k0, k1 = q * 2.0 ** -100, k0 * 2.0 ** 100, k1 * 2.0 ** 100
    else:
        q = q.clone()
        q[..., 0] = q[..., 0].abs() + 0.5
        if what == "overflowing keys":
            q[..., 0] *= 2.0 ** 70
            k0, k1 = k0.clone(), k1.clone()
            k0[..., 0] = k1[..., 0] = 0.0
        for k, lo, hi in ((k0, 5, 70), (k0, 128, 1000), (k1, 0, 64), (k1, n - 41, n)):
            k[lo:hi, :, 0] = -float("inf") if what == "-inf keys" else -2.0 ** 64
        count = np.r_[0:5, 70:128, 1000:n, n + 64:2 * n - 41]
    v0, v1 = v0 * vscale, v1 * vscale
    with ifx.KVCache(1, H, D, n, n, ifx.IFX_F32) as cache:
        cache.commit(0, k0, v0)
        out, lse = torch.empty_like(q), torch.empty((n, H), device=dev)
        cache.attention_blocks(0, q, k1, v1, None, out, lse)
        torch.cuda.synchronize()
    rows, heads = rows_of(n, H)
    q64 = synth.to_f64_numpy(q)
    if what == "overflowing keys":
        q64[..., 0] = 0.0
    want, want_lse = oracle.attention_rows(q64, np.concatenate([synth.to_f64_numpy(k0), synth.to_f64_numpy(k1)])[count],
                                           np.concatenate([synth.to_f64_numpy(v0), synth.to_f64_numpy(v1)])[count], None, None, rows, heads)
    assert np.abs(synth.to_f64_numpy(out)[rows, heads] - want).max() <= 1e-5 * vscale
    assert np.abs(synth.to_f64_numpy(lse)[rows, heads] - want_lse).max() <= 2e-5


@pytest.mark.parametrize("what", ["values near the smallest", "keys near the smallest", "queries near the smallest"])
def test_f32_in_pieces_of_every_size(gpu_device, what):
    """Elements as small as fp32 has them, rows that a few keys dominate (queries x 4): the tolerance of elements near 1.  An
    element of 2^-124 held to 2^-134 (a bf16's last subnormal place) is off by up to 1e-3."""
    dev, n, H, D = gpu_device, 1560, 3, 128
    assert ifx.ifx_attention_f32_key_parts(n, H, D, 2 * n)[1] == 256
    (_, k0, v0), (q, k1, v1) = (synth.draw_qkv(97, b, 0, 0, n, H, D, torch.float32, dev) for b in (0, 999))
    q, vscale, scale = 4.0 * q, 1.0, 1.0 / np.sqrt(D)
    if what == "values near the smallest":
        vscale = 2.0 ** -124
    elif what == "keys near the smallest":
        k0, k1, q, scale = k0 * 2.0 ** -122, k1 * 2.0 ** -122, q * 2.0 ** 60, scale * 2.0 ** 62
    else:
        q, k0, k1, scale = q * 2.0 ** -122, k0 * 2.0 ** 60, k1 * 2.0 ** 60, scale * 2.0 ** 62
    v0, v1 = v0 * vscale, v1 * vscale
    with ifx.KVCache(1, H, D, n, n, ifx.IFX_F32, softmax_scale=float(scale)) as cache:
        cache.commit(0, k0, v0)
        out, lse = torch.empty_like(q), torch.empty((n, H), device=dev)
        cache.attention_blocks(0, q, k1, v1, None, out, lse)
        torch.cuda.synchronize()
    rows, heads = rows_of(n, H)
    want, want_lse = oracle.attention_rows(synth.to_f64_numpy(q), synth.to_f64_numpy(k0), synth.to_f64_numpy(v0), synth.to_f64_numpy(k1),
                                           synth.to_f64_numpy(v1), rows, heads, scale=float(np.float32(scale)))
    assert np.abs(synth.to_f64_numpy(out)[rows, heads] - want).max() <= 1e-5 * vscale
    assert np.abs(synth.to_f64_numpy(lse)[rows, heads] - want_lse).max() <= 4e-5


def test_f32_in_pieces_values_near_the_largest(gpu_device):
    """718 of 750 keys score 1.9, the first 32 nothing: against the largest score the sum of weighted values is 722 x 2^118, below
    2^128; against a first reference of 0 it is 4800 x 2^118."""
    dev, n, H, D, cap = gpu_device, 250, 130, 128, 2
    assert ifx.ifx_attention_f32_key_parts(n, H, D, (cap + 1) * n) == (1, 256)
    q, k0, k1 = (torch.zeros((n, H, D), device=dev) for _ in range(3))
    v = torch.full((n, H, D), 2.0 ** 118, device=dev)
    q[..., 0] = 1.0
    k0[32:, :, 0] = k1[..., 0] = 1.9
    with ifx.KVCache(1, H, D, cap * n, n, ifx.IFX_F32, softmax_scale=1.0) as cache:
        cache.commit(0, k0, v)
        cache.commit(0, k1, v)
        out, lse = torch.empty_like(q), torch.empty((n, H), device=dev)
        cache.attention_blocks(0, q, k1, v, None, out, lse)
        torch.cuda.synchronize()
    assert (out / 2.0 ** 118 - 1).abs().max() <= 2e-6
    assert np.abs(synth.to_f64_numpy(lse) - np.log(32 + 718 * np.exp(float(np.float32(1.9))))).max() <= 2e-6


@pytest.mark.parametrize("n,H,D,cap", [(1560, 3, 128, 1), (250, 130, 128, 2)])  # in 12 parts, whole
def test_f32_in_pieces_log_sum_exp(gpu_device, n, H, D, cap):
    """Half a unit in the last place of a number from 8 on is 4.8e-7; the scores' own rounding adds as much at most.  A logarithm
    rounded before the reference is added to it comes out up to 1.5e-6 off."""
    dev = gpu_device
    assert ifx.ifx_attention_f32_key_parts(n, H, D, (cap + 1) * n)[1] == 256
    blocks = [synth.draw_qkv(101, b, 0, 0, n, H, D, torch.float32, dev) for b in range(cap + 1)]
    with ifx.KVCache(1, H, D, cap * n, n, ifx.IFX_F32) as cache:
        for _, k, v in blocks[:cap]:
            cache.commit(0, k, v)
        q, k, v = blocks[cap]
        out, lse = torch.empty_like(q), torch.empty((n, H), device=dev)
        cache.attention_blocks(0, q, k, v, None, out, lse)
        torch.cuda.synchronize()
    keys = torch.cat([b[1] for b in blocks]).double().cpu()
    for h in range(0, H, 13):
        want = torch.logsumexp(q[:, h].double().cpu() @ keys[:, h].T.contiguous() * float(np.float32(1) / np.sqrt(np.float32(D))), -1)
        assert (lse[:, h].double().cpu() - want).abs().max() <= 1e-6, h


@pytest.mark.parametrize("what", ["infinite keys", "infinite queries", "values near the largest"])
def test_f32_in_pieces_time_of_other_inputs(gpu_device, what):
    """Scores and sums taken again in fp32: 2 to 4 times an ordinary call; a lane at a time it was 70 times one."""
    dev, n, H, D = gpu_device, 1560, 12, 128
    assert ifx.ifx_attention_f32_key_parts(n, H, D, 2 * n)[1] == 256
    (q, k0, v0), (_, k1, v1) = (synth.draw_qkv(103, b, 0, 0, n, H, D, torch.float32, dev) for b in (0, 1))
    odd = [x.clone() for x in (q, k0, v0)]
    if what == "values near the largest":
        odd[2] *= 2.0 ** 100
    else:
        odd[0][..., 0] = odd[0][..., 0].abs() + 0.5
        odd[1 if what == "infinite keys" else 0][::7, :, 0] = -float("inf")
    out = torch.empty_like(q)

    def best_of(queries, keys, values):
        with ifx.KVCache(1, H, D, n, n, ifx.IFX_F32) as cache:
            cache.commit(0, keys, values)
            times = []
            for _ in range(6):
                start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                start.record()
                cache.attention(0, queries, k1, v1, out)
                stop.record()
                torch.cuda.synchronize()
                times.append(start.elapsed_time(stop))
        return min(times)

    assert best_of(*odd) <= 12 * best_of(q, k0, v0)


def test_f32_in_pieces_weights_near_the_smallest(gpu_device):
    """Values that read single weights out: e^-80 has its last pieces below a bf16's range, e^-89 is subnormal (22 bits)."""
    dev, n, H, D = gpu_device, 1560, 3, 64
    assert ifx.ifx_attention_f32_key_parts(n, H, D, 2 * n)[1] == 256
    q, k0, k1, v0, v1 = (torch.zeros((n, H, D), device=dev) for _ in range(5))
    q[..., 0] = 8.0  # times the scale: 1
    faint = {5: -80.0, 700: -86.0, 1559: -89.0}
    for d, (j, s) in enumerate(faint.items()):
        k0[j, :, 0], v0[j, :, d] = s, 2.0 ** 60
        k1[j, :, 0], v1[j, :, 8 + d] = s, 2.0 ** 60
    with ifx.KVCache(1, H, D, n, n, ifx.IFX_F32) as cache:
        cache.commit(0, k0, v0)
        out = torch.empty_like(q)
        cache.attention(0, q, k1, v1, out)
        torch.cuda.synchronize()
    got = synth.to_f64_numpy(out)
    want = np.zeros(D)
    for d, s in enumerate(faint.values()):
        want[d] = want[8 + d] = np.exp(s) * 2.0 ** 60 / (2 * n - 6)
    # half a unit in the last place of 86 log2 e is 2^-18: 2.6e-6 of e^-86; the other steps 5e-7
    assert (np.abs(got - want) <= 4e-6 * want).all()


def test_f32_streams_without_an_area(gpu_device):
    """Two streams of a cache have memory for parts; the third runs the call whole, on the kernel of 16-row tiles: the
    same but for fp32's rounding."""
    dev, n, H, D = gpu_device, 1560, 3, 128
    assert ifx.ifx_attention_f32_key_parts(n, H, D, 2 * n) == (12, 256)
    with ifx.KVCache(1, H, D, n, n, ifx.IFX_F32) as cache:
        _, k, v = synth.draw_qkv(89, 0, 0, 0, n, H, D, torch.float32, dev)
        cache.commit(0, k, v)
        q, kb, vb = synth.draw_qkv(89, 999, 0, 0, n, H, D, torch.float32, dev)
        torch.cuda.synchronize()
        outs = []
        for _ in range(3):
            outs.append(torch.empty_like(q))
            with torch.cuda.stream(torch.cuda.Stream()):
                cache.attention(0, q, kb, vb, outs[-1])
        torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    assert (outs[0] - outs[2]).abs().max() <= 1e-5


@pytest.mark.parametrize("n,H,D,cap,parts", [
    (552, 2, 128, 8, 39),   # four tiles of keys to a workgroup, 18 wavefronts of rows in three
    (736, 6, 72, 2, 14),    # four or five
    (656, 4, 64, 5, 21),    # five or six; workgroups of 7 wavefronts
    (576, 4, 40, 8, 21),    # seven or eight, padded to 64
    (248, 33, 128, 2, 6),   # four, and none cached in the last part
])
def test_f32_in_pieces_step_by_step(gpu_device, n, H, D, cap, parts):
    """Few tiles, even and odd numbers of them, for wavefronts that run a step apart."""
    dev = gpu_device
    assert ifx.ifx_attention_f32_key_parts(n, H, D, (cap + 1) * n) == (parts, 256)
    hs = np.array([0, H - 1])
    blocks = [synth.draw_qkv(97, b, 0, 0, n, H, D, torch.float32, dev) for b in range(cap + 1)]
    with ifx.KVCache(1, H, D, cap * n, n, ifx.IFX_F32) as cache:
        for _, k, v in blocks[:cap]:
            cache.commit(0, k, v)
        q = blocks[cap][0]
        out, lse = torch.full((n + 1, H, D), float("nan"), device=dev), torch.full((n + 1, H), float("nan"), device=dev)
        cache.attention_blocks(0, *blocks[cap], None, out[:n], lse[:n])
        torch.cuda.synchronize()
    assert torch.isfinite(out[:n]).all() and torch.isfinite(lse[:n]).all() and torch.isnan(out[n]).all() and torch.isnan(lse[n]).all()
    rows, heads = rows_of(n, 2)
    want, want_lse = oracle.attention_rows(synth.to_f64_numpy(q)[:, hs], np.concatenate([synth.to_f64_numpy(b[1])[:, hs] for b in blocks]),
                                           np.concatenate([synth.to_f64_numpy(b[2])[:, hs] for b in blocks]), None, None, rows, heads)
    assert np.abs(synth.to_f64_numpy(out[:n])[rows, hs[heads]] - want).max() <= 1e-5
    assert np.abs(synth.to_f64_numpy(lse[:n])[rows, hs[heads]] - want_lse).max() <= 2e-5
