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

# (key groups, n, heads, cap, commits, listed blocks, with the current block)
CASES = [
    # eight groups (32-row workgroups): H * ceil(n / 32) <= 256
    (8, 8, 1, 2, 1, None, True),        # 16 keys: seven wavefronts without a key
    (8, 8, 3, 70, 72, list(range(69, -1, -1)), True),  # more listed blocks than a wavefront has lanes, 8 keys each
    (8, 8, 5, 200, 203, list(range(199, -1, -1)), True),  # the entries at hand move along the list, twice and more
    (8, 40, 3, 140, 141, list(range(0, 140, 2)) + list(range(1, 140, 2)), False),  # two subtiles per entry
    (8, 16, 40, 5, 6, [3, 0, 4, 1], True),  # two listed blocks to a subtile
    (8, 24, 3, 67, 67, list(range(66, 0, -1)), True),  # blocks that straddle subtiles
    (8, 56, 3, 4, 6, [3, 1, 2], False),
    (8, 264, 2, 70, 71, list(range(69, -1, -1)), True),
    (8, 40, 2, 3, 5, [2, 0], False),    # blocks that end 8 keys into a subtile, no current block
    (8, 72, 5, 3, 3, None, True),
    (8, 264, 28, 2, 2, None, True),     # 252 workgroups
    (8, 1024, 8, 1, 0, None, True),     # 256, no cached keys
    # up to here tiles of up to 64 workgroups are shared by four, of up to 128 by two; the same forms where two share, and where none do
    (8, 8, 100, 200, 203, list(range(199, -1, -1)), True),
    (8, 24, 70, 67, 67, list(range(66, 0, -1)), True),
    (8, 40, 45, 3, 5, [2, 0], False),
    (8, 8, 130, 200, 203, list(range(199, -1, -1)), True),
    (8, 24, 140, 67, 67, list(range(66, 0, -1)), True),
    (8, 40, 70, 3, 5, [2, 0], False),
    (8, 8, 129, 2, 1, None, True),      # seven wavefronts without a key
    # two groups (128-row workgroups)
    (2, 1032, 8, 1, 1, None, True),     # 264 row wavefronts: the first past eight groups
    (2, 168, 43, 2, 2, None, True),     # the fewest rows a head, 6 wavefronts of them; a phase of 5 tiles and 16 keys
    (2, 200, 40, 1, 2, None, True),     # 3 tiles and 8 keys: the last tile leaves a group without keys
    (2, 200, 40, 3, 5, [1, 2], True),   # selection on a wrapped ring
    (2, 192, 48, 66, 66, list(range(65, 0, -1)), False),  # 65 listed blocks: two passes of the table, whole tiles
    (2, 1560, 12, 1, 1, None, True),
    (2, 264, 85, 1, 0, None, True),     # 255 workgroups, no cached keys
    (2, 264, 135, 1, 1, None, True),    # 272 workgroups of 256 rows, 408 of 128
    (2, 1160, 52, 1, 1, [0], True),     # 264 workgroups of 256 rows, 520 of 128
    # one group (256-row workgroups)
    (1, 264, 86, 1, 1, None, True),     # 258 workgroups of 128 rows, 172 of 256
    (1, 200, 150, 2, 3, [1], True),
    (1, 64, 700, 1, 1, None, True),     # whole tiles only, one in each phase
    (1, 40, 700, 2, 2, [1, 0], False),
    (1, 32, 257, 2, 2, None, True),     # phases of one tile and of half a tile
    (1, 40, 130, 2, 2, None, True),     # 80 cached keys: one tile and 16; 40 of the block: no whole tile
    (1, 72, 90, 3, 5, [1, 2], True),
    (1, 64, 131, 66, 66, list(range(65, 0, -1)), False),  # 65 listed blocks: two passes of the table
]


@pytest.mark.parametrize("dtype", [ifx.IFX_BF16, ifx.IFX_FP8_E4M3])
@pytest.mark.parametrize("groups,n,H,cap,commits,blocks,with_block", CASES)
def test_key_groups_at_every_switch(gpu_device, groups, n, H, cap, commits, blocks, with_block, dtype):
    dev, D = gpu_device, 128
    assert ifx.ifx_attention_key_groups(n, H) == groups
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
                oc.commit(k[:, hs], v[:, hs])
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
            want, want_lse = oracle.attention_rows(f64(q)[:, hs], kc, vc, None if k is None else f64(k)[:, hs],
                                                   None if v is None else f64(v)[:, hs], rows, np.tile(np.arange(len(hs)), len(r)))
            assert_attention_close(to_np_exact(out)[rows, heads].astype(np.float64), want, ifx.IFX_BF16, f"gain {gain}")
            # eight groups, and rows under the norm bound (which needs cached keys): from fp32 exponentials, off by the
            # rounding of scores and sums (up to 5 x 11 in log2 units here, 2^-24 of that in a product, a sum and a power
            # of two); otherwise from weights rounded to bf16, off by 2^-9 at most
            exact = groups == 8 or (gain == 1.0 and commits > 0)
            assert np.abs(f64(lse)[rows, heads] - want_lse).max() <= (2e-5 if exact else 4e-3)


@pytest.mark.parametrize("dtype", [ifx.IFX_BF16, ifx.IFX_FP8_E4M3])
@pytest.mark.parametrize("groups,n,H,cap", [
    (8, 264, 2, 2),
    (8, 8, 3, 9),       # whole blocks that count nothing
    (8, 264, 8, 2),     # 72 and 135 row tiles, of two workgroups and of one
    (8, 8, 100, 9),
    (8, 264, 15, 2),
    (8, 8, 130, 9),
    (2, 1560, 12, 1),
    (2, 264, 135, 1),   # two rounds of workgroups
    (1, 200, 150, 2),
])
def test_keys_with_scores_of_minus_infinity(gpu_device, groups, n, H, cap, dtype):
    """Keys whose score is -inf for every query (finite elements whose product overflows) have weight
    0, whatever share of a group's keys they make up: the result is that of the other keys."""
    dev, D = gpu_device, 128
    assert ifx.ifx_attention_key_groups(n, H) == groups
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


@pytest.mark.parametrize("dtype", [ifx.IFX_BF16, ifx.IFX_FP8_E4M3])
@pytest.mark.parametrize("groups,n,H", [(2, 168, 43), (1, 8, 300)])
def test_long_block_lists_in_the_table_kernels(gpu_device, groups, n, H, dtype):
    """Lists that take one, two and three passes of the block table, with a last pass of 1, 2 and 4
    entries, scrambled on a wrapped ring, with and without the current block (eight groups have no
    passes)."""
    dev, D, cap = gpu_device, 128, 130
    assert ifx.ifx_attention_key_groups(n, H) == groups
    hs = np.array([0, H // 2, H - 1])
    r = np.unique(np.concatenate([np.arange(min(n, 6)), np.arange(n - 6, n), np.arange(0, n, 29)]))
    rows, heads = np.repeat(r, len(hs)), np.tile(np.arange(len(hs)), len(r))
    oc = OracleCacheFP8(cap) if dtype == ifx.IFX_FP8_E4M3 else OracleCacheF(cap, torch.bfloat16)
    with ifx.KVCache(1, H, D, cap * n, n, dtype) as cache:
        for b in range(cap + 7):
            _, k, v = synth.draw_qkv(43, b, 0, 0, n, H, D, torch.bfloat16, dev, rms_norm=True)
            cache.commit(0, k, v)
            oc.commit(k[:, hs], v[:, hs])
        q, k, v = synth.draw_qkv(43, 999, 0, 0, n, H, D, torch.bfloat16, dev, rms_norm=True)
        rng = np.random.default_rng(11)
        for count in (63, 64, 126, 127, 128, 130):
            picks = rng.permutation(cap)[:count].tolist()
            for kk, vv in ((k, v), (None, None)):
                out = torch.full((n, H, D), float("nan"), dtype=torch.bfloat16, device=dev)
                lse = torch.full((n, H), float("nan"), device=dev)
                cache.attention_blocks(0, q, kk, vv, picks, out, lse)
                torch.cuda.synchronize()
                kc, vc = (oracle.bf16_bits_to_f64(x) for x in oc.raw.logical(blocks=picks))
                want, want_lse = oracle.attention_rows(f64(q)[:, hs], kc, vc, None if kk is None else f64(kk)[:, hs],
                                                       None if vv is None else f64(vv)[:, hs], rows, heads)
                label = f"{count} listed blocks, block={kk is not None}"
                assert_attention_close(to_np_exact(out)[rows, hs[heads]].astype(np.float64), want, ifx.IFX_BF16, label)
                assert np.abs(f64(lse)[rows, hs[heads]] - want_lse).max() <= 2e-5, label  # under the norm bound: see above


@pytest.mark.parametrize("dtype", [ifx.IFX_BF16, ifx.IFX_FP8_E4M3])
@pytest.mark.parametrize("groups", [1, 2])
def test_random_calls_of_the_larger_kernels(gpu_device, groups, dtype):
    """A seeded sweep of calls that two groups and one group take: rows, heads, ring state, key set,
    rows on both sides of the norm bound in one workgroup."""
    dev, D = gpu_device, 128
    rng = np.random.default_rng(1000 * groups + dtype)
    done = 0
    while done < 20:
        n, H = 8 * int(np.exp(rng.uniform(0, np.log(170)))), int(np.exp(rng.uniform(np.log(8), np.log(320))))
        if ifx.ifx_attention_key_groups(n, H) != groups or n * H > 60000:
            continue
        done += 1
        cap = int(rng.integers(1, 5))
        commits = int(rng.integers(0, 2 * cap + 1))
        resident = min(cap, commits)
        picks = None if rng.random() < 0.5 else rng.permutation(resident)[:int(rng.integers(0, resident + 1))].tolist()
        with_block = commits == 0 or picks == [] or rng.random() < 0.7
        hs = np.unique(np.concatenate([[0, H - 1], rng.integers(0, H, 2)]))
        r = np.unique(np.concatenate([np.arange(min(n, 8)), np.arange(n - 8, n), rng.integers(0, n, 24)]))
        rows, heads = np.repeat(r, len(hs)), np.tile(np.arange(len(hs)), len(r))
        oc = OracleCacheFP8(cap) if dtype == ifx.IFX_FP8_E4M3 else OracleCacheF(cap, torch.bfloat16)
        with ifx.KVCache(1, H, D, cap * n, n, dtype) as cache:
            for b in range(commits):
                _, k, v = synth.draw_qkv(done, b, 0, 0, n, H, D, torch.bfloat16, dev, rms_norm=True)
                cache.commit(0, k, v)
                oc.commit(k[:, hs], v[:, hs])
            q, k, v = synth.draw_qkv(done, 999, 0, 0, n, H, D, torch.bfloat16, dev, rms_norm=True)
            q = q.clone()
            for w in range(0, n, 32):
                q[w:w + 32] *= float(rng.choice([1.0, 1.0, 3.0, 8.0]))
            if not with_block:
                k = v = None
            out = torch.full((n + 2, H, D), float("nan"), dtype=torch.bfloat16, device=dev)
            cache.attention_blocks(0, q, k, v, picks, out[:n])
            torch.cuda.synchronize()
        assert torch.isfinite(out[:n].float()).all() and torch.isnan(out[n:].float()).all()
        kc, vc = (None, None) if resident == 0 or picks == [] else (oracle.bf16_bits_to_f64(x) for x in oc.raw.logical(**({} if picks is None else {"blocks": picks})))
        want, _ = oracle.attention_rows(f64(q)[:, hs], kc, vc, None if k is None else f64(k)[:, hs], None if v is None else f64(v)[:, hs], rows, heads)
        label = f"n {n} heads {H} cap {cap} commits {commits} picks {picks} block {with_block}"
        assert_attention_close(to_np_exact(out)[rows, hs[heads]].astype(np.float64), want, ifx.IFX_BF16, label, input_scale=8.0)
