"""GPU parity of the fp32 attention kernel at the edges of its tiling: 16-row tiles, 16-key subtiles
dealt to 4 or 8 wavefronts, head_dim padded to a multiple of 32, key runs that end inside a subtile
(whole cache, listed blocks, current block)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_20714_amd import binding as ifx
from paper_2511_20714_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,H,D,cap,commits,blocks,with_block", [
    (1, 1, 8, 4, 3, None, True),        # one row, four keys: seven of eight wavefronts without a key
    (15, 2, 40, 2, 3, None, True),      # head_dim 40 in 64, ragged rows and keys
    (16, 3, 64, 3, 3, [2, 0], False),   # exact tiles, a selection out of order, no current block
    (17, 2, 72, 3, 4, [1, 2], True),    # head_dim 72 in 96; every listed block ends one key into a subtile
    (33, 5, 96, 2, 2, None, True),
    (129, 3, 128, 2, 3, [1], True),
    (8, 1, 128, 70, 72, list(range(69, -1, -1)), True),   # more listed blocks than a wavefront has lanes
    (1, 4, 8, 200, 203, list(range(199, -1, -1)), True),  # one key per entry and subtile: the entries at hand move along the list
    (16, 1, 40, 130, 131, list(range(0, 130, 2)) + list(range(1, 130, 2)), False),
    # listed blocks shorter than a subtile: rows gathered from several blocks, at every head_dim the kernel is built for
    (3, 2, 24, 150, 151, list(range(0, 150, 2)) + list(range(1, 150, 2)), True),
    (5, 3, 64, 66, 70, list(range(65, -1, -1)), False),
    (7, 2, 96, 9, 10, [8, 0, 3], True),
    (15, 2, 128, 70, 71, list(range(1, 70)), True),
    (13, 300, 72, 3, 5, [2, 0], True),      # 300 workgroups: 4 wavefronts each
    (1, 1, 128, 2, 3, [1], True),
    (1370, 3, 128, 1, 1, None, True),   # 258 workgroups: the first size with 4 wavefronts each
    (1366, 3, 32, 1, 0, None, True),    # 258 of the smallest head_dim, no cached keys
])
def test_f32_attention_at_tile_edges(gpu_device, n, H, D, cap, commits, blocks, with_block):
    dev = gpu_device
    with ifx.KVCache(1, H, D, cap * n, n, ifx.IFX_F32) as cache:
        oc = oracle.BlockCacheOracle(cap)
        for b in range(commits):
            _, k, v = synth.draw_qkv(61, b, 0, 0, n, H, D, torch.float32, dev)
            cache.commit(0, k, v)
            oc.commit(synth.to_f64_numpy(k), synth.to_f64_numpy(v))
        q, k, v = synth.draw_qkv(61, 999, 0, 0, n, H, D, torch.float32, dev)
        if not with_block:
            k = v = None
        out = torch.full((n, H, D), float("nan"), device=dev)
        lse = torch.full((n, H), float("nan"), device=dev)
        cache.attention_blocks(0, q, k, v, blocks, out, lse)
        torch.cuda.synchronize()
        assert torch.isfinite(out).all() and torch.isfinite(lse).all()
        kc, vc = oc.logical() if blocks is None else oc.logical([(b, 1) for b in blocks])
        r = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 40), n), np.random.default_rng(1).integers(0, n, 40)]))
        rows, heads = np.repeat(r, H), np.tile(np.arange(H), len(r))
        want, want_lse = oracle.attention_rows(synth.to_f64_numpy(q), kc, vc, None if k is None else synth.to_f64_numpy(k),
                                               None if v is None else synth.to_f64_numpy(v), rows, heads)
        assert np.abs(synth.to_f64_numpy(out)[rows, heads] - want).max() <= 1e-5
        assert np.abs(synth.to_f64_numpy(lse)[rows, heads] - want_lse).max() <= 2e-5


@pytest.mark.parametrize("n,H,D,commits", [
    (256, 2, 64, 3),    # 8 wavefronts: some of them first see keys that count nothing
    (48, 3, 128, 1),
    (1370, 3, 64, 1),   # 4 wavefronts
    (256, 2, 40, 3),    # head_dim padded to 64: the padding must not meet the infinite element
    (100, 3, 72, 2),    # to 96
    (33, 1, 8, 1),      # to 32
])
def test_f32_keys_with_scores_of_minus_infinity(gpu_device, n, H, D, commits):
    """A key whose score is -inf for every query (an element of -inf against positive query elements)
    has weight 0, whatever share of a wavefront's keys it makes up: the result is that of the other
    keys.  Runs of such keys that fill subtiles, a wavefront's first subtile, a whole block."""
    dev = gpu_device
    blocks = [synth.draw_qkv(67, b, 0, 0, n, H, D, torch.float32, dev) for b in range(commits)] + [synth.draw_qkv(67, 999, 0, 0, n, H, D, torch.float32, dev)]
    q = blocks[-1][0].clone()
    q[..., 0] = q[..., 0].abs() + 0.5
    keys, values = (np.concatenate([synth.to_f64_numpy(b[i]) for b in blocks]) for i in (1, 2))
    r = np.unique(np.concatenate([np.arange(min(n, 20)), np.arange(n - 20, n)]))
    rows, heads = np.repeat(r, H), np.tile(np.arange(H), len(r))
    for lo, hi in ((5, 6), (16, 32), (32, min(64, 2 * n)), (16, n), (n, 2 * n), (2 * n - 20, 2 * n)):
        with ifx.KVCache(1, H, D, commits * n, n, ifx.IFX_F32) as cache:
            for b in range(commits + 1):
                k = blocks[b][1].clone()
                k[max(0, lo - b * n):max(0, hi - b * n), :, 0] = -float("inf")
                if b < commits:
                    cache.commit(0, k, blocks[b][2])
            out = torch.full((n, H, D), float("nan"), device=dev)
            lse = torch.full((n, H), float("nan"), device=dev)
            cache.attention_blocks(0, q, k, blocks[-1][2], None, out, lse)
            torch.cuda.synchronize()
        count = np.r_[0:lo, hi:len(keys)]
        want, want_lse = oracle.attention_rows(synth.to_f64_numpy(q), keys[count], values[count], None, None, rows, heads)
        assert np.abs(synth.to_f64_numpy(out)[rows, heads] - want).max() <= 1e-5, (lo, hi)
        assert np.abs(synth.to_f64_numpy(lse)[rows, heads] - want_lse).max() <= 2e-5, (lo, hi)
