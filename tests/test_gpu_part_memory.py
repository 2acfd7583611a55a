"""The memory for partial results of calls whose keys come in parts: from stream to stream, while other streams are at work, beside
a capture, under host threads; and the same calls without it, on a third stream or captured."""
import threading

import pytest
import torch

from paper_2511_20714_amd import binding as ifx
from paper_2511_20714_amd import synth

pytestmark = pytest.mark.gpu

# (dtype, n, heads, head_dim, blocks, rows of a workgroup)
CALLS = [
    (ifx.IFX_BF16, 1000, 3, 128, 9, 32),
    (ifx.IFX_BF16, 1000, 5, 128, 9, 256),
    (ifx.IFX_BF16, 520, 104, 128, 12, 256),  # 85 heads whole, the others' keys in parts
    (ifx.IFX_F32, 256, 2, 64, 3, 16),
    (ifx.IFX_F32, 1560, 3, 128, 1, 256),
]
SLEEP = 20_000_000  # cycles: some 10 ms


class Calls:
    def __init__(self, dtype, n, H, D, cap, rows, dev):
        tensor = torch.float32 if dtype == ifx.IFX_F32 else torch.bfloat16
        if dtype == ifx.IFX_F32:
            parts, of = ifx.ifx_attention_f32_key_parts(n, H, D, (cap + 1) * n)
        else:
            parts, _, of = ifx.ifx_attention_key_parts(n, H, cap * n)
        assert parts > 1 and of == rows
        self.cache = ifx.KVCache(1, H, D, cap * n, n, dtype)
        for b in range(cap):
            self.cache.commit(0, *synth.draw_qkv(5, b, 0, 0, n, H, D, tensor, dev, rms_norm=True)[1:])
        self.inputs = synth.draw_qkv(5, 999, 0, 0, n, H, D, tensor, dev, rms_norm=True)
        # another order of sums in fp32; two independent roundings of each row's weights
        self.bound = 2e-6 if dtype == ifx.IFX_F32 else 6e-3
        torch.cuda.synchronize()

    def empty(self):
        return torch.full_like(self.inputs[0], float("nan"))

    def run(self, stream, out, times=1):
        with torch.cuda.stream(stream):
            for _ in range(times):
                self.cache.attention(0, *self.inputs, out)

    def close(self, a, b):
        return ((a.float() - b.float()).norm() <= self.bound * b.float().norm()).item()


@pytest.fixture(params=CALLS, ids=lambda c: "-".join(map(str, c)))
def calls(request, gpu_device):
    c = Calls(*request.param, gpu_device)
    with c.cache:
        yield c


def test_streams_one_after_another(calls):
    want, got = calls.empty(), calls.empty()
    calls.run(torch.cuda.Stream(), want)
    torch.cuda.synchronize()
    for i in range(5):
        calls.run(torch.cuda.Stream(), got.fill_(float("nan")), 9)
        torch.cuda.synchronize()
        assert torch.equal(got, want), i


def test_streams_at_work_keep_theirs(calls):
    want, got, mine = calls.empty(), calls.empty(), [calls.empty() for _ in range(2)]
    busy, third = [torch.cuda.Stream() for _ in range(2)], torch.cuda.Stream()
    calls.run(busy[0], want)
    torch.cuda.synchronize()
    for s, o in zip(busy, mine):
        with torch.cuda.stream(s):
            torch.cuda._sleep(SLEEP)
        calls.run(s, o)
    calls.run(third, got, 12)
    assert not busy[0].query() and not busy[1].query()
    torch.cuda.synchronize()
    assert torch.equal(mine[0], want) and torch.equal(mine[1], want)
    assert calls.close(got, want)
    calls.run(third, got.fill_(float("nan")))
    torch.cuda.synchronize()
    assert torch.equal(got, want)


def test_captured_beside_other_streams(calls):
    """Replays of a captured call, which has no memory of its own; a host thread makes calls on a third stream, which look for
    memory, while the capture is under way."""
    want, got, graphed = calls.empty(), calls.empty(), calls.empty()
    streams = [torch.cuda.Stream() for _ in range(4)]
    for s in streams[:2]:
        calls.run(s, want)
    torch.cuda.synchronize()
    static = [t.clone() for t in calls.inputs]
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    other = threading.Thread(target=calls.run, args=(streams[2], got, 12))
    with torch.cuda.graph(graph, stream=streams[3]):
        calls.cache.attention(0, *static, graphed)
        other.start()
        other.join()
        calls.cache.attention(0, *static, graphed)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    for i in range(3):
        graphed.fill_(float("nan"))
        static[0].copy_(calls.inputs[0] * (1 - 0.25 * i))
        graph.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[2]):
            calls.cache.attention(0, *static, got)
        torch.cuda.synchronize()
        assert calls.close(graphed, got), i


def test_two_host_threads(calls):
    want = calls.empty()
    streams, outs = [torch.cuda.Stream() for _ in range(2)], [calls.empty() for _ in range(2)]
    calls.run(streams[0], want)
    torch.cuda.synchronize()
    threads = [threading.Thread(target=calls.run, args=(s, o, 30)) for s, o in zip(streams, outs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert torch.equal(outs[0], want) and torch.equal(outs[1], want)
