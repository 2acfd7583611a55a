"""Commit and read-back, bit for bit, at the edges of their launches: blocks of one granule or one
row, heads and rows that leave workgroups without work, head dims whose rows do not fill a workgroup
(fp32), more resident blocks than one launch takes, a wrapped ring in both orders, canary rows."""
import pytest
import torch

from paper_2511_20714_amd import binding as ifx
from paper_2511_20714_amd import synth

from gpu_util import TORCH_DTYPE, OracleCacheF, OracleCacheFP8, expected_ids

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,H,D,cap,commits", [
    (ifx.IFX_BF16, 8, 1, 128, 3, 4),
    (ifx.IFX_BF16, 8, 600, 128, 2, 3),      # one K workgroup per head
    (ifx.IFX_BF16, 72, 5, 128, 67, 70),     # 67 resident blocks: two launches
    (ifx.IFX_BF16, 2056, 3, 128, 1, 2),
    (ifx.IFX_FP8_E4M3, 8, 2, 128, 66, 69),
    (ifx.IFX_FP8_E4M3, 264, 7, 128, 2, 2),
    (ifx.IFX_F32, 1, 1, 8, 3, 5),
    (ifx.IFX_F32, 33, 3, 40, 66, 68),       # rows of 10 chunks, 25 a round
    (ifx.IFX_F32, 300, 2, 96, 2, 3),
    (ifx.IFX_F32, 64, 700, 128, 1, 1),
])
def test_read_back_at_the_edges(gpu_device, dtype, n, H, D, cap, commits):
    dev, L = gpu_device, 2
    tdtype = TORCH_DTYPE.get(dtype, torch.bfloat16)
    with ifx.KVCache(L, H, D, cap * n, n, dtype) as cache:
        oracles = [OracleCacheFP8(cap) if dtype == ifx.IFX_FP8_E4M3 else OracleCacheF(cap, tdtype) for _ in range(L)]
        for b in range(commits):
            blocks = [synth.draw_qkv(19, b, 0, layer, n, H, D, tdtype, dev)[1:] for layer in range(L)]
            if b % 2:
                cache.commit_layers(0, [k for k, _ in blocks], [v for _, v in blocks])
            else:
                for layer, (k, v) in enumerate(blocks):
                    cache.commit(layer, k, v)
            for layer, (k, v) in enumerate(blocks):
                oracles[layer].commit(k, v)
        for layer in range(L):
            C, raw = cache.len(layer), oracles[layer].raw
            for logical in (True, False):
                k, v = (torch.full((C + 2, H, D), 7.0, dtype=tdtype, device=dev) for _ in range(2))
                cache.read(layer, k[:C], v[:C], logical)
                torch.cuda.synchronize()
                want_k, want_v = raw.logical()
                if not logical:  # slot s holds the block with the ordinal the deque model puts there
                    order = [raw.ordinals.index(o) for o in expected_ids(raw, cap) if o >= 0]
                    want_k, want_v = ([x[b * n:(b + 1) * n] for b in order] for x in (want_k, want_v))
                    want_k, want_v = (b"".join(p.tobytes() for p in x) for x in (want_k, want_v))
                else:
                    want_k, want_v = want_k.tobytes(), want_v.tobytes()
                assert synth.raw_bytes(k[:C]) == want_k and synth.raw_bytes(v[:C]) == want_v, (layer, logical)
                assert (k[C:] == 7.0).all() and (v[C:] == 7.0).all()


@pytest.mark.parametrize("dtype,n,H,D,L,cap", [
    (ifx.IFX_BF16, 1032, 9, 128, 34, 2),
    (ifx.IFX_FP8_E4M3, 1032, 9, 128, 45, 3),
    (ifx.IFX_F32, 1033, 9, 40, 54, 2),      # rows of 10 chunks; ragged last round
])
def test_copies_past_the_caches(gpu_device, dtype, n, H, D, L, cap):
    """A commit that moves more than 300 MiB, and the read-backs but the first that go over layers which together move more than
    that, stream: bit for bit what one layer's commits and read-backs, which do not, leave."""
    dev = gpu_device
    tdtype = TORCH_DTYPE.get(dtype, torch.bfloat16)
    io, held = (4, 4) if dtype == ifx.IFX_F32 else (2, 1 if dtype == ifx.IFX_FP8_E4M3 else 2)
    assert L * n * H * D * 2 * (io + held) > 300 << 20 and L * cap * n * H * D * 2 * held > 150 << 20
    blocks = [[synth.draw_qkv(23, b, 0, layer, n, H, D, tdtype, dev)[1:] for layer in range(L)] for b in range(2)]
    order = [0, 1] * cap  # more commits than the ring holds
    with ifx.KVCache(L, H, D, cap * n, n, dtype) as cache, ifx.KVCache(1, H, D, cap * n, n, dtype) as one:
        for b in order[:cap + 1]:
            cache.commit_layers(0, [k for k, _ in blocks[b]], [v for _, v in blocks[b]])
        for layer in (0, 1, L - 1):
            one.reset()
            for b in order[:cap + 1]:
                one.commit(0, *blocks[b][layer])
            got, want = ([torch.full((cap * n + 2, H, D), 7.0, dtype=tdtype, device=dev) for _ in range(2)] for _ in range(2))
            cache.read(layer, *(t[:cap * n] for t in got))
            one.read(0, *(t[:cap * n] for t in want))
            torch.cuda.synchronize()
            for g, w in zip(got, want):
                assert synth.raw_bytes(g) == synth.raw_bytes(w), layer
