"""The work this library is timed on: block attention against a KV cache, cache commits, read-back
and the merge of partial results, each through the public binding as a generation loop calls it.

A case is a dict of plain values:
  kind "attend"  a block's attention over `layers` layers (and, with `commit`, the commit of the
                 block that ends its last denoising step), at a cache of `cached` resident blocks;
  kind "handover" a new video's first block committed in every layer and read back whole;
  kind "merge"   two partial attention results over disjoint key sets combined.
"""
import math

import torch

from paper_2511_20714_amd import binding as ifx
from paper_2511_20714_amd import synth

DTYPES = {"fp32": ifx.IFX_F32, "bf16": ifx.IFX_BF16, "fp8": ifx.IFX_FP8_E4M3}
TENSOR = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.bfloat16}
ELEM = {"fp32": 4, "bf16": 2, "fp8": 1}  # bytes of a cached element
SINK, WINDOW = 1, 3  # "sink_window": the oldest resident block and the newest three

# the largest listed case, 4 n Lk D H = 1.19e13: no drawn case costs more
MOST_FLOPS = 4.0 * 10800 * 54000 * 128 * 40


def attend(name, dtype, heads, head_dim, block, cached, layers=1, gain=1.0, keys="all", lse=False, commit=False):
    case = {"kind": "attend", "dtype": dtype, "heads": heads, "head_dim": head_dim, "block": block, "cached": cached,
            "layers": layers, "gain": gain, "keys": keys, "lse": lse, "commit": commit}
    return {"name": name, **case} if name else case


def handover(name, dtype, heads, head_dim, block, layers):
    case = {"kind": "handover", "dtype": dtype, "heads": heads, "head_dim": head_dim, "block": block, "layers": layers}
    return {"name": name, **case} if name else case


def merge(name, dtype, heads, head_dim, block):
    case = {"kind": "merge", "dtype": dtype, "heads": heads, "head_dim": head_dim, "block": block}
    return {"name": name, **case} if name else case


def listed():
    return [
        # the benchmark's step: one 1.3B-class layer (12 heads, blocks of 3 latent frames) over a full
        # ring of 6 blocks, key length 32760, then the block's commit, which evicts the oldest
        attend("layer_32k_step", "bf16", 12, 128, 4680, 6, commit=True),
        # the largest: one 14B-class layer at 720p, key length 54000
        attend("layer_720p_54k", "bf16", 40, 128, 10800, 4),
        # the same 1.3B-class layer on the compressed cache, ring of 7
        attend("layer_37k_fp8", "fp8", 12, 128, 4680, 7),
        # long-horizon generation with a sliding window: a sink block and the newest three of a wrapped ring
        attend("layer_sink_window", "bf16", 12, 128, 4680, 7, keys="sink_window", lse=True),
        # rows dominated by a few keys: scores beyond what the norm bound covers (no QK normalisation, learned gains)
        attend("layer_18k_peaked", "bf16", 12, 128, 4680, 3, gain=4.0),
        # the first block of a video: no cached keys yet
        attend("first_block", "bf16", 12, 128, 4680, 0),
        # frame-by-frame generation: one denoising step over 30 layers at blocks of one latent frame, and its commit
        attend("frame_step_30_layers", "bf16", 12, 128, 1560, 6, layers=30, commit=True),
        # the smallest: a few hundred tokens and two heads, where launches and latency count
        attend("small_call", "bf16", 2, 128, 264, 2),
        # the fp32 configuration: 2 heads x 64, key length 1024
        attend("fp32_small_step", "fp32", 2, 64, 256, 3, commit=True),
        # fp32 as the check of a bf16 model's layer
        attend("fp32_layer", "fp32", 12, 128, 1560, 1),
        # a new video's first block: all layers committed in one call, then every layer's contents handed over
        handover("commit_handover_30_layers", "bf16", 12, 128, 4680, 30),
        # ring attention: two ranks' partial results of one layer combined
        merge("merge_layer", "bf16", 12, 128, 4680),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _block(rng, lo, hi):
    """Block sizes are multiples of 8 (bf16 caches ask for it), odd multiples as well as even ones."""
    return max(lo, min(hi, 8 * round(_log_uniform(rng, lo, hi) / 8)))


def draw(rng):
    kind = rng.choice(["bf16", "bf16", "bf16", "peaked", "fp8", "window", "layers", "fp32", "handover", "merge"])
    heads = round(_log_uniform(rng, 1, 40))
    block = _block(rng, 64, 10800)
    cached = rng.randint(0, 7)
    if kind in ("bf16", "peaked", "fp8"):
        while 4.0 * block * block * (cached + 1) * 128 * heads > MOST_FLOPS:
            cached -= 1
        return attend(None, "fp8" if kind == "fp8" else "bf16", heads, 128, block, cached, gain=round(rng.uniform(3.5, 8.0), 2) if kind == "peaked" else 1.0,
                      lse=rng.random() < 0.25, commit=cached > 0 and rng.random() < 0.25)
    if kind == "window":
        return attend(None, rng.choice(["bf16", "fp8"]), heads, 128, block, rng.randint(5, 7) if block < 6000 else 5, keys="sink_window", lse=True)
    if kind == "layers":
        block, heads, cached = _block(rng, 64, 3600), round(_log_uniform(rng, 2, 40)), rng.randint(1, 7)
        layers = rng.randint(2, 30)
        while layers > 2 and layers * block * heads * (cached + 10) > 4e7:
            layers -= 1
        return attend(None, rng.choice(["bf16", "bf16", "fp8"]), heads, 128, block, cached, layers=layers, commit=True)
    if kind == "fp32":
        return attend(None, "fp32", round(_log_uniform(rng, 1, 16)), rng.choice([40, 64, 72, 96, 128, 128]), _block(rng, 64, 1600),
                      rng.randint(0, 4), lse=rng.random() < 0.25, commit=False)
    if kind == "handover":
        block = _block(rng, 64, 4680)
        layers = max(1, min(rng.randint(1, 30), int(3e6 / (block * heads))))
        return handover(None, rng.choice(["bf16", "bf16", "fp8", "fp32"]), heads, 128, block, layers)
    dtype = rng.choice(["bf16", "bf16", "fp32"])
    return merge(None, dtype, heads, 128 if dtype == "bf16" else rng.choice([40, 64, 72, 96, 128]), block)


def _blocks(case, seed, block, layer):
    """(q, k, v) of one block of one layer: RMS-normalised q and k as a QK-normed DiT has them (fp32: plain N(0,1))."""
    return synth.draw_qkv(seed, block, 0, layer, case["block"], case["heads"], case["head_dim"], TENSOR[case["dtype"]],
                          torch.device("cuda"), rms_norm=case["dtype"] != "fp32", logit_gain=case.get("gain", 1.0))


def prepare(case, seed):
    n, H, D = case["block"], case["heads"], case["head_dim"]
    tensor, dev = TENSOR[case["dtype"]], torch.device("cuda")
    if case["kind"] == "merge":
        g = torch.Generator(device=dev).manual_seed(seed)
        out_a, out_b = (torch.randn(n, H, D, generator=g, device=dev).to(tensor) for _ in range(2))
        # log-sum-exps of normalised scores over some thousand keys, the two sides of one size
        lse_a, lse_b = (9.0 + 0.5 * torch.randn(n, H, generator=g, device=dev) for _ in range(2))
        return {"case": case, "a": (out_a, lse_a), "b": (out_b, lse_b), "out": torch.empty_like(out_a), "lse": torch.empty_like(lse_a)}
    L = case["layers"]
    if case["kind"] == "handover":
        cache = ifx.KVCache(L, H, D, n, n, DTYPES[case["dtype"]])
        sets = [_blocks(case, seed, 0, l)[1:] for l in range(L)]
        return {"case": case, "cache": cache, "k": [s[0] for s in sets], "v": [s[1] for s in sets],
                "k_out": torch.empty((L, n, H, D), dtype=tensor, device=dev), "v_out": torch.empty((L, n, H, D), dtype=tensor, device=dev)}
    cached = case["cached"]
    cache = ifx.KVCache(L, H, D, max(cached, 1) * n, n, DTYPES[case["dtype"]])
    # a sliding window is met after the ring has gone round
    commits = cached + 2 if case["keys"] == "sink_window" else cached
    for b in range(commits):
        for l in range(L):
            _, k, v = _blocks(case, seed, b, l)
            cache.commit(l, k, v)
    sets = [_blocks(case, seed, 1000 + i, 0) for i in range(max(L, 2))]
    return {"case": case, "cache": cache, "sets": sets, "pass": 0, "out": torch.empty((L, n, H, D), dtype=tensor, device=dev),
            "lse": torch.empty((L, n, H), dtype=torch.float32, device=dev) if case["lse"] else None}


def run(state):
    case = state["case"]
    n, H, D = case["block"], case["heads"], case["head_dim"]
    if case["kind"] == "merge":
        ifx.ifx_attention_merge(*state["a"], *state["b"], state["out"], state["lse"], n * H, D, DTYPES[case["dtype"]])
        return state["out"], state["lse"]
    cache, L = state["cache"], case["layers"]
    if case["kind"] == "handover":
        cache.reset()
        cache.commit_layers(0, state["k"], state["v"])
        for l in range(L):
            cache.read(l, state["k_out"][l], state["v_out"][l])
        return state["k_out"], state["v_out"]
    sets, i = state["sets"], state["pass"]
    state["pass"] = i + 1
    ks, vs = [], []
    for l in range(L):
        q, k, v = sets[(i + l) % len(sets)]
        out = state["out"][l]
        if case["keys"] == "sink_window":
            cache.attention_ranges(l, q, k, v, [(0, SINK), (case["cached"] - WINDOW, WINDOW)], out, state["lse"][l])
        elif case["lse"]:
            cache.attention_blocks(l, q, k, v, None, out, state["lse"][l])
        else:
            cache.attention(l, q, k, v, out)
        ks.append(k)
        vs.append(v)
    if case["commit"]:
        if L == 1:
            cache.commit(0, ks[0], vs[0])
        else:
            cache.commit_layers(0, ks, vs)
    return (state["out"], state["lse"]) if case["lse"] else state["out"]


def work(case):
    n, H, D = case["block"], case["heads"], case["head_dim"]
    row = H * D * (4 if case["dtype"] == "fp32" else 2)  # bytes of a token in the caller's tensors
    if case["kind"] == "merge":
        return {"bytes": 3 * n * row + 3 * n * H * 4, "flops": 3 * n * H * D}
    held = 2 * H * D * ELEM[case["dtype"]]  # bytes of a token's K and V in the cache
    L = case["layers"]
    if case["kind"] == "handover":  # block read, cache written; cache read, block written
        return {"bytes": L * n * (2 * (2 * row) + 2 * held), "flops": 0}
    keys = (SINK + WINDOW if case["keys"] == "sink_window" else case["cached"]) * n
    per_layer = n * 2 * row + keys * held + n * 2 * row  # q and out, the cached keys, the block's own
    if case["lse"]:
        per_layer += n * H * 4
    if case["commit"]:
        per_layer += n * 2 * row + n * held
    return {"bytes": L * per_layer, "flops": L * 4 * n * (keys + n) * D * H}


def tolerance(case):
    """About four times the relative errors measured against the same operation in 64 bits."""
    if case["kind"] == "handover":
        return "exact"  # data movement (and one fixed rounding rule)
    fp32 = case["dtype"] == "fp32"
    if case["kind"] == "merge":  # bf16: 1.5e-5 against the 64-bit result rounded to bf16; a value then differs by one unit in the last place
        return {"rel": 1e-6, "max": 1e-5} if fp32 else {"rel": 1e-4, "max": 2e-2}
    # fp32: 6e-7 ... 1.2e-6, largest element 7e-6; bf16 and fp8: 2.0e-3 ... 2.4e-3, largest element 1.1e-2
    # (each row's weights and outputs are rounded to bf16; rows dominated by one key show more in single elements)
    return {"rel": 5e-6, "max": 5e-5} if fp32 else {"rel": 1e-2, "max": 0.1}
