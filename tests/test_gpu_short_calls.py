"""GPU parity of short calls: 32-row tiles whose output dimensions are shared by four, two or one workgroups; and, with one and
two key groups, whose first tiles are asked for before anything else is known: one to four tiles of cached keys or of
the block alone, listed blocks, more key norms than the first loads take."""
import numpy as np
import pytest
import torch

from paper_2511_20714_amd import binding as ifx
from paper_2511_20714_amd import synth

from gpu_util import OracleCacheF, OracleCacheFP8, assert_attention_close, f64, to_np_exact
import oracle

pytestmark = pytest.mark.gpu


def check(dev, dtype, n, H, cap, blocks, with_block, gain):
    """Rows at either end and some others of the first and last head against the oracle, log-sum-exp and canary rows too."""
    hs = np.unique([0, H - 1])
    oc = OracleCacheFP8(max(cap, 1)) if dtype == ifx.IFX_FP8_E4M3 else OracleCacheF(max(cap, 1), torch.bfloat16)
    with ifx.KVCache(1, H, 128, max(cap, 1) * n, n, dtype) as cache:
        for b in range(cap):
            _, k, v = synth.draw_qkv(91, b, 0, 0, n, H, 128, torch.bfloat16, dev, rms_norm=True)
            cache.commit(0, k, v)
            oc.commit(k[:, hs], v[:, hs])
        q, k, v = synth.draw_qkv(91, 999, 0, 0, n, H, 128, torch.bfloat16, dev, rms_norm=True, logit_gain=gain)
        if not with_block:
            k = v = None
        out = torch.full((n + 3, H, 128), float("nan"), dtype=torch.bfloat16, device=dev)
        lse = torch.full((n + 3, H), float("nan"), device=dev)
        cache.attention_blocks(0, q, k, v, blocks, out[:n], lse[:n])
        torch.cuda.synchronize()
    assert torch.isfinite(out[:n].float()).all() and torch.isfinite(lse[:n]).all()
    assert torch.isnan(out[n:].float()).all() and torch.isnan(lse[n:]).all()
    r = np.unique(np.concatenate([np.arange(min(n, 8)), np.arange(max(n - 8, 0), n), np.random.default_rng(5).integers(0, n, 12)]))
    rows, heads = np.repeat(r, len(hs)), np.tile(np.arange(len(hs)), len(r))
    kc, vc = oc.logical() if blocks is None else (oracle.bf16_bits_to_f64(x) for x in oc.raw.logical(blocks=blocks))
    want, want_lse = oracle.attention_rows(f64(q)[:, hs], kc, vc, None if k is None else f64(k)[:, hs], None if v is None else f64(v)[:, hs], rows, heads)
    assert_attention_close(to_np_exact(out)[rows, hs[heads]].astype(np.float64), want, ifx.IFX_BF16, f"{n} x {H}, {cap} blocks, gain {gain}")
    return np.abs(f64(lse)[rows, hs[heads]] - want_lse).max()


@pytest.mark.parametrize("dtype", [ifx.IFX_BF16, ifx.IFX_FP8_E4M3])
@pytest.mark.parametrize("n,H,cap,blocks,with_block", [
    (8, 1, 0, None, True), (8, 3, 9, [7, 0, 3, 8], True), (40, 5, 1, None, False), (264, 2, 2, None, True), (264, 2, 5, [4, 0, 2], False),
    (32, 64, 3, None, True), (512, 4, 1, None, True),                # 64 tiles: four workgroups each
    (32, 65, 3, [2, 1], True), (1032, 3, 0, None, True), (32, 128, 2, None, False), (264, 14, 3, None, True),  # two
    (32, 129, 3, None, True), (264, 15, 2, [1, 0], True),            # one
])
def test_shared_row_tiles(gpu_device, n, H, cap, blocks, with_block, dtype):
    """A step or less for every wavefront, some without a key, half-filled tiles; the log-sum-exp is from fp32 exponentials."""
    keys = n * (cap if blocks is None else len(blocks))
    assert ifx.ifx_attention_key_groups(n, H) == 8 and ifx.ifx_attention_key_parts(n, H, keys, with_block)[0] == 1
    for gain in (1.0, 5.0):
        assert check(gpu_device, dtype, n, H, cap, blocks, with_block, gain) <= 2e-5


@pytest.mark.parametrize("dtype", [ifx.IFX_BF16, ifx.IFX_FP8_E4M3])
@pytest.mark.parametrize("groups,n,H,cap,blocks,with_block", [
    (1, 8, 257, 0, None, True), (1, 72, 100, 0, None, True), (1, 136, 64, 0, None, True),   # one, two and three tiles of the block alone
    (1, 8, 257, 1, None, False), (1, 8, 257, 9, [8, 0, 4], True), (1, 136, 64, 2, None, True),
    (1, 8, 257, 600, None, True),                                                            # 600 key norms
    (2, 264, 30, 0, None, True), (2, 168, 43, 1, None, True), (2, 264, 30, 3, [2, 0], False), (2, 520, 16, 1, None, False),
])
def test_first_tiles(gpu_device, groups, n, H, cap, blocks, with_block, dtype):
    assert ifx.ifx_attention_key_groups(n, H) == groups
    for gain in (1.0, 5.0):  # under the norm bound, and past it
        # past it a row's sum is of weights rounded to bf16: off by 2^-9
        assert check(gpu_device, dtype, n, H, cap, blocks, with_block, gain) <= (2e-5 if gain == 1.0 and cap else 4e-3)
