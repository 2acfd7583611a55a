"""GPU parity of bf16 attention where its keys are dealt to one, two or eight groups of wavefronts:
row counts on both sides of every switch, key runs that end inside a tile or a subtile or leave a
group without a key, listed blocks, no current block, scores beyond the norm bound."""
import numpy as np
import pytest
import torch

from paper_2511_20714_amd import binding as ifx
from paper_2511_20714_amd import synth

from gpu_util import OracleCacheF, OracleCacheFP8, assert_attention_close, f64, to_np_exact
import oracle

pytestmark = pytest.mark.gpu

CASES = [
    # eight groups (32-row workgroups): H * ceil(n / 32) <= 256
    (8, 1, 2, 1, None, True),        # 16 keys: seven wavefronts without a key
    (8, 3, 70, 72, list(range(69, -1, -1)), True),  # more listed blocks than a wavefront has lanes, 8 keys each
    (40, 2, 3, 5, [2, 0], False),    # blocks that end 8 keys into a subtile, no current block
    (72, 5, 3, 3, None, True),
    (264, 28, 2, 2, None, True),     # 252 workgroups
    (1024, 8, 1, 0, None, True),     # 256, no cached keys
    # two groups (128-row workgroups)
    (1032, 8, 1, 1, None, True),     # 264 row wavefronts: the first past eight groups
    (32, 257, 2, 2, None, True),     # phases of 64 and 32 keys, no partial tile; the second leaves a group without keys
    (40, 130, 2, 2, None, True),     # 80 cached keys: one tile and 16; 40 of the block: no whole tile
    (72, 90, 3, 5, [1, 2], True),    # selection on a wrapped ring
    (64, 131, 66, 66, list(range(65, 0, -1)), False),  # 65 listed blocks: two passes of the table
    (1560, 12, 1, 1, None, True),
    (264, 85, 1, 0, None, True),     # 255 workgroups, no cached keys
    (264, 135, 1, 1, None, True),    # 270 workgroups of 256 rows, 405 of 128
    # one group (256-row workgroups)
    (264, 86, 1, 1, None, True),     # 258 workgroups of 128 rows, 172 of 256
    (200, 150, 2, 3, [1], True),
    (64, 700, 1, 1, None, True),     # whole tiles only, one in each phase
    (40, 700, 2, 2, [1, 0], False),
]


@pytest.mark.parametrize("dtype", [ifx.IFX_BF16, ifx.IFX_FP8_E4M3])
@pytest.mark.parametrize("n,H,cap,commits,blocks,with_block", CASES)
def test_key_groups_at_every_switch(gpu_device, n, H, cap, commits, blocks, with_block, dtype):
    dev, D = gpu_device, 128
    rng = np.random.default_rng(7)
    r = np.unique(np.concatenate([np.arange(min(n, 10)), np.arange(max(0, n - 10), n), rng.integers(0, n, 12)]))
    hs = np.unique(np.concatenate([[0, H - 1], rng.integers(0, H, 4)]))
    rows, heads = np.repeat(r, len(hs)), np.tile(hs, len(r))
    for gain in (1.0, 5.0):  # under the norm bound, and past it
        with ifx.KVCache(1, H, D, cap * n, n, dtype) as cache:
            oc = OracleCacheFP8(cap) if dtype == ifx.IFX_FP8_E4M3 else OracleCacheF(cap, torch.bfloat16)
            for b in range(commits):
                _, k, v = synth.draw_qkv(83, b, 0, 0, n, H, D, torch.bfloat16, dev, rms_norm=True)
                cache.commit(0, k, v)
                oc.commit(k, v)
            q, k, v = synth.draw_qkv(83, 999, 0, 0, n, H, D, torch.bfloat16, dev, rms_norm=True, logit_gain=gain)
            if not with_block:
                k = v = None
            # canary rows behind both outputs
            out = torch.full((n + 3, H, D), float("nan"), dtype=torch.bfloat16, device=dev)
            lse = torch.full((n + 3, H), float("nan"), device=dev)
            cache.attention_blocks(0, q, k, v, blocks, out[:n], lse[:n])
            torch.cuda.synchronize()
            assert torch.isfinite(out[:n].float()).all() and torch.isfinite(lse[:n]).all()
            assert torch.isnan(out[n:].float()).all() and torch.isnan(lse[n:]).all()
            if blocks is None:
                kc, vc = oc.logical()
            else:
                kc, vc = (oracle.bf16_bits_to_f64(x) for x in oc.raw.logical(blocks=blocks))
            sel = lambda x: None if x is None else x[:, hs]
            want, want_lse = oracle.attention_rows(f64(q)[:, hs], sel(kc), sel(vc), None if k is None else f64(k)[:, hs],
                                                   None if v is None else f64(v)[:, hs], rows, np.tile(np.arange(len(hs)), len(r)))
            assert_attention_close(to_np_exact(out)[rows, heads].astype(np.float64), want, ifx.IFX_BF16, f"gain {gain}")
            # a sum of weights rounded to bf16 (past the norm bound) is off by 2^-9 at most, one taken in fp32 by rounding alone
            assert np.abs(f64(lse)[rows, heads] - want_lse).max() <= 4e-3


@pytest.mark.parametrize("dtype", [ifx.IFX_BF16, ifx.IFX_FP8_E4M3])
@pytest.mark.parametrize("n,H,cap", [
    (264, 2, 2),     # eight groups
    (8, 3, 9),       # whole blocks that count nothing
    (1560, 12, 1),   # two groups
    (264, 135, 1),   # two groups, two rounds of workgroups
    (200, 150, 2),   # one group
])
def test_keys_with_scores_of_minus_infinity(gpu_device, n, H, cap, dtype):
    """Keys whose score is -inf for every query (finite elements whose product overflows) have weight
    0, whatever share of a group's keys they make up: the result is that of the other keys."""
    dev, D = gpu_device, 128
    rng = np.random.default_rng(5)
    hs = np.unique(np.concatenate([[0, H - 1], rng.integers(0, H, 2)]))
    r = np.unique(np.concatenate([np.arange(min(n, 10)), np.arange(n - 8, n), rng.integers(0, n, 10)]))
    rows, heads = np.repeat(r, len(hs)), np.tile(np.arange(len(hs)), len(r))
    blocks = [synth.draw_qkv(29, b, 0, 0, n, H, D, torch.bfloat16, dev, rms_norm=True) for b in range(cap + 1)]
    big = 2.0 ** 8 if dtype == ifx.IFX_FP8_E4M3 else 2.0 ** 64  # the largest codes are 448
    q = blocks[cap][0].clone()
    q[..., 0] = 3.0e38 if dtype == ifx.IFX_FP8_E4M3 else 2.0 ** 70
    Lk = (cap + 1) * n
    for lo, hi in ((5, 6), (32, 64), (n, 2 * n), (32, Lk - n), (Lk - 40 if n > 40 else Lk - 5, Lk)):
        if lo >= hi:
            continue
        oc = OracleCacheFP8(cap) if dtype == ifx.IFX_FP8_E4M3 else OracleCacheF(cap, torch.bfloat16)
        with ifx.KVCache(1, H, D, cap * n, n, dtype) as cache:
            for b in range(cap + 1):
                k = blocks[b][1].clone()
                k[..., 0] = 0.0  # the keys that count do not meet the huge query element
                k[max(0, lo - b * n):max(0, hi - b * n), :, 0] = -big
                if b < cap:
                    cache.commit(0, k, blocks[b][2])
                    oc.commit(k[:, hs], blocks[b][2][:, hs])
            out = torch.full((n, H, D), float("nan"), dtype=torch.bfloat16, device=dev)
            lse = torch.full((n, H), float("nan"), device=dev)
            cache.attention_blocks(0, q, k, blocks[cap][2], None, out, lse)
            torch.cuda.synchronize()
        kc, vc = oc.logical()
        count = np.r_[0:lo, hi:Lk]
        q0 = f64(q)[:, hs]
        q0[..., 0] = 0.0
        want, want_lse = oracle.attention_rows(q0, np.concatenate([kc, f64(k)[:, hs]])[count], np.concatenate([vc, f64(blocks[cap][2])[:, hs]])[count],
                                               None, None, rows, heads)
        assert_attention_close(to_np_exact(out)[rows, hs[heads]].astype(np.float64), want, ifx.IFX_BF16, f"{lo}..{hi}")
        # (sums of weights rounded to bf16 are off by 2^-9 at most)
        assert np.abs(f64(lse)[rows, hs[heads]] - want_lse).max() <= 4e-3, (lo, hi)
