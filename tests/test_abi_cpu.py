"""CPU-side checks: the library loads and exports everything include/ifx.h
declares; the slot bookkeeping matches a deque model; calls that need a device
fail loudly (there is no CPU fallback)."""
import collections
import os
import re

import pytest

from paper_2511_20714_amd import binding as ifx

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "ifx.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ifx_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = ifx.lib()
    names = declared_symbols()
    assert len(names) >= 20
    for name in names:
        assert hasattr(lib, name), name
    # and the binding wraps each of them under the same name
    for name in names:
        assert callable(getattr(ifx, name)), name


def test_header_is_plain_c():
    import subprocess, tempfile
    with tempfile.TemporaryDirectory() as d:
        src = os.path.join(d, "t.c")
        open(src, "w").write('#include "ifx.h"\nint main(void){return IFX_OK;}\n')
        subprocess.check_call(["gcc", "-std=c99", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-c", src,
                               "-o", os.path.join(d, "t.o")])


@pytest.mark.parametrize("cap", [1, 2, 7, 16])
def test_ring_matches_deque_model(cap):
    ring = ifx.ifx_ring_create(cap)
    try:
        model = collections.deque(maxlen=cap)
        slot_of = {}
        assert ifx.ifx_ring_block_ids(ring) == [-1] * cap
        for t in range(3 * cap + 5):
            assert ifx.ifx_ring_next_slot(ring) == t % cap
            slot = ifx.ifx_ring_commit(ring)
            if len(model) == cap:
                slot_of.pop(model[0])
            # a free slot, or the slot of the block that just fell out
            assert slot not in slot_of.values()
            model.append(t)
            slot_of[t] = slot
            assert ifx.ifx_ring_committed(ring) == t + 1
            assert ifx.ifx_ring_resident(ring) == len(model)
            ids = ifx.ifx_ring_block_ids(ring)
            want = [-1] * cap
            for o, s in slot_of.items():
                want[s] = o
            assert ids == want
            for i, o in enumerate(model):
                assert ifx.ifx_ring_slot_of_logical(ring, i) == slot_of[o]
            assert ifx.ifx_ring_slot_of_logical(ring, len(model)) == -1
            assert ifx.ifx_ring_slot_of_logical(ring, -1) == -1
        ifx.ifx_ring_reset(ring)
        assert ifx.ifx_ring_resident(ring) == 0 and ifx.ifx_ring_block_ids(ring) == [-1] * cap
    finally:
        ifx.ifx_ring_destroy(ring)


@pytest.mark.parametrize("in_place", [False, True])
def test_ring_grow_matches_a_growing_window_model(in_place):
    """ifx_ring_grow against a plain list model: the resident blocks keep their numbers and order;
    moved: they sit in slots 0, 1, ... oldest first right after the grow; in place: every block
    stays in the slot it had; either way the new slots are used next and only then the oldest
    block is evicted again; a slot never holds two resident blocks; slots in use are a prefix."""
    import random
    rng = random.Random(7 + in_place)
    for trial in range(40):
        cap = rng.randint(1, 5)
        ring = ifx.ifx_ring_create(cap)
        try:
            committed = []  # ordinals, all of them
            gone = 0        # how many of them are evicted
            slot_of = {}
            for step in range(80):
                if rng.random() < 0.12:
                    new_cap = cap + rng.randint(1, 4)
                    ifx.ifx_ring_grow(ring, new_cap, in_place)
                    old_cap, cap = cap, new_cap
                    resident = committed[gone:]
                    if not in_place:
                        slot_of = {o: i for i, o in enumerate(resident)}  # re-laid, oldest first
                    # the next commit takes a new slot, unless the old capacity was not full yet
                    assert ifx.ifx_ring_next_slot(ring) == len(resident)
                    with pytest.raises(ifx.IfxError):
                        ifx.ifx_ring_grow(ring, cap, in_place)
                    del old_cap
                else:
                    slot = ifx.ifx_ring_commit(ring)
                    if len(committed) - gone == cap:
                        assert slot == slot_of.pop(committed[gone])  # the oldest block's slot is the one reused
                        gone += 1
                    else:
                        assert slot == len(committed) - gone  # slots in use are a prefix
                    assert slot not in slot_of.values()
                    slot_of[len(committed)] = slot
                    committed.append(len(committed))
                resident = committed[gone:]
                assert ifx.ifx_ring_committed(ring) == len(committed)
                assert ifx.ifx_ring_resident(ring) == len(resident)
                want = [-1] * cap
                for o in resident:
                    want[slot_of[o]] = o
                assert ifx.ifx_ring_block_ids(ring) == want
                assert sorted(slot_of.values()) == list(range(len(resident)))
                for i, o in enumerate(resident):
                    assert ifx.ifx_ring_slot_of_logical(ring, i) == slot_of[o]
                assert ifx.ifx_ring_slot_of_logical(ring, len(resident)) == -1
        finally:
            ifx.ifx_ring_destroy(ring)


def test_reserve_is_checked_before_any_device_work():
    h = ifx.ifx_kv_cache_create(1, 2, 128, 128)
    try:
        lib = ifx.lib()
        assert lib.ifx_kv_cache_reserve(h, 64) == ifx.IFX_ERR_INVALID_ARG  # below the capacity
        assert lib.ifx_kv_cache_reserve(None, 256) == ifx.IFX_ERR_INVALID_ARG
        assert lib.ifx_kv_cache_reserve(h, 200) == ifx.IFX_OK
        assert lib.ifx_kv_cache_configure(h, 64, ifx.IFX_BF16, 0.0) == ifx.IFX_ERR_INVALID_ARG  # 200 % 64
    finally:
        ifx.ifx_kv_cache_destroy(h)


def test_ring_rejects_bad_capacity():
    with pytest.raises(ifx.IfxError):
        ifx.ifx_ring_create(0)


def test_create_rejects_bad_sizes():
    for args in [(0, 2, 64, 128), (1, 0, 64, 128), (1, 2, 0, 128), (1, 2, 64, 0), (1, 2, 64, -5)]:
        with pytest.raises(ifx.IfxError):
            ifx.ifx_kv_cache_create(*args)


def test_calls_before_configure_fail():
    h = ifx.ifx_kv_cache_create(2, 2, 128, 64)
    try:
        lib = ifx.lib()
        assert lib.ifx_kv_cache_len(h, 0) == ifx.IFX_ERR_NOT_CONFIGURED
        assert lib.ifx_kv_cache_commit(h, 0, 16, 16, None) == ifx.IFX_ERR_NOT_CONFIGURED
        assert lib.ifx_block_attention(h, 0, 16, 16, 16, 16, None) == ifx.IFX_ERR_NOT_CONFIGURED
        assert "configure" in ifx.ifx_last_error()
        assert lib.ifx_kv_cache_configure(h, 48, ifx.IFX_BF16, 0.0) == ifx.IFX_ERR_INVALID_ARG  # 64 % 48
        assert lib.ifx_kv_cache_configure(h, 64, 7, 0.0) == ifx.IFX_ERR_INVALID_ARG
        assert lib.ifx_kv_cache_configure(None, 64, 0, 0.0) == ifx.IFX_ERR_INVALID_ARG
    finally:
        ifx.ifx_kv_cache_destroy(h)
    ifx.ifx_kv_cache_destroy(None)


def test_no_cpu_fallback_without_a_device():
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    with pytest.raises(ifx.IfxError) as e:
        ifx.KVCache(1, 2, 64, 1024, 256, ifx.IFX_F32)
    assert e.value.code == ifx.IFX_ERR_HIP


def test_current_stream_with_and_without_torchs_raw_handle(monkeypatch):
    """stream=None is the current stream of the current device, whether or not this torch has the
    private function that gives its handle directly."""
    torch = pytest.importorskip("torch")
    import types

    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    assert ifx._stream(None) == 103
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert ifx._stream(None) == 77
    assert ifx._stream(5) == 5 and ifx._stream(types.SimpleNamespace(cuda_stream=9)) == 9


def test_bench_refuses_more_than_one_gpu():
    """bench.py is a one-GPU benchmark: any other --gpus value ends with a message, before any GPU work."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "one GPU" in (r.stderr + r.stdout)


def test_oracle_is_not_imported_by_the_product():
    """The package must not reach for the oracle (test infrastructure) or for working files."""
    pkg = os.path.join(ROOT, "paper_2511_20714_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hpp", ".hip", ".h")):
                text = open(os.path.join(dirpath, f)).read()
                assert "import oracle" not in text and "from oracle" not in text, f
                assert "_work" not in text, f


@pytest.mark.parametrize("heads", [1, 2, 3, 5, 7, 8, 9, 11, 12, 13, 16, 17, 24, 40])
def test_attention_launch_items_tile_every_head(heads):
    """The bf16 attention launch: the workgroups' (head, query rows) items, decoded by the function
    the kernel itself uses, cover rows 0 .. n - 1 of every head exactly once, in wavefronts of 32
    rows, at most 8 per workgroup and dealt evenly (counts differ by at most one, no workgroup
    is empty unless it exits); a head's workgroups sit on as few XCDs as its share allows."""
    for n in (8, 32, 72, 200, 256, 264, 2056, 4680, 10800):
        grid = ifx.ifx_attention_launch_grid(n, heads)
        q_tiles = -(-n // 256)
        assert grid % 8 == 0 and grid >= heads * q_tiles
        covered = collections.defaultdict(list)  # head -> [(row0, waves)]
        xcds = collections.defaultdict(set)
        tiles = collections.defaultdict(set)
        for w in range(grid):
            head, q_tile, row0, waves, xcd = ifx.ifx_attention_launch_item(n, heads, w)
            assert xcd == w % 8
            if waves == 0:
                continue
            assert 0 <= head < heads and 1 <= waves <= 8 and row0 % 32 == 0
            assert q_tile not in tiles[head]
            tiles[head].add(q_tile)
            covered[head].append((row0, waves))
            xcds[head].add(xcd)
        assert sorted(covered) == list(range(heads))
        for head, items in covered.items():
            items.sort()
            assert len(items) == q_tiles
            nxt = 0
            for row0, waves in items:
                assert row0 == nxt, (n, heads, head)
                nxt = row0 + 32 * waves
            assert n <= nxt < n + 32  # the last wavefront holds the last row
            counts = [wv for _, wv in items]
            assert max(counts) - min(counts) <= 1
        # whole heads live on one XCD each, eight at a time; the rest on as few as an even split needs
        left = heads % 8
        for head in range(heads):
            if head < heads - left:
                assert len(xcds[head]) == 1
            elif 8 % left == 0:
                assert len(xcds[head]) <= 8 // left


def test_attention_launch_shape_rejects_bad_arguments():
    with pytest.raises(ifx.IfxError):
        ifx.ifx_attention_launch_grid(0, 12)
    with pytest.raises(ifx.IfxError):
        ifx.ifx_attention_launch_grid(4680, 0)
    grid = ifx.ifx_attention_launch_grid(4680, 12)
    assert grid == 232  # 8 x (19 workgroups of a whole head + 10 of a shared one); 228 of them have rows
    with pytest.raises(ifx.IfxError):
        ifx.ifx_attention_launch_item(4680, 12, grid)
    with pytest.raises(ifx.IfxError):
        ifx.ifx_attention_launch_item(4680, 12, -1)
    busy = [ifx.ifx_attention_launch_item(4680, 12, w) for w in range(grid)]
    assert sum(1 for it in busy if it[3] > 0) == 228
    assert sorted(it[3] for it in busy if it[0] == 0 and it[3] > 0) == [7] * 5 + [8] * 14


@pytest.mark.parametrize("groups,shapes", [
    # 32-row workgroups as long as they are one round on 256 CUs
    (8, [(8, 1), (8, 256), (32, 256), (264, 28), (1560, 5), (8192, 1)]),
    # up to 160 rows a head: a head's workgroups are the same, or read its keys once more, with two groups
    (1, [(8, 257), (32, 257), (32, 600), (64, 131), (104, 250), (128, 65), (128, 300), (136, 64), (160, 300)]),
    # 128-row workgroups in one round
    (2, [(168, 43), (192, 128), (256, 128), (264, 85), (520, 16), (1560, 6), (1560, 12), (4680, 6)]),
    (1, [(168, 130), (256, 200), (264, 86), (520, 64), (4680, 7), (4680, 12)]),
    # in two rounds, where 256-row workgroups take two as well
    (2, [(264, 135), (264, 170), (520, 100), (1560, 39), (10800, 6)]),
    # in three: only from 37 wavefronts of rows on, and up to 680 workgroups
    (2, [(1160, 52), (1160, 68), (1560, 40), (4680, 14), (4680, 18), (10800, 8)]),
    (1, [(192, 300), (256, 300), (264, 200), (392, 135), (520, 130), (1032, 57), (1152, 58), (1560, 58), (4680, 20), (10800, 40)]),
])
def test_key_groups_where_they_pay(groups, shapes):
    """Where a call's keys are dealt to groups: on either side of every line of the rule."""
    for n, heads in shapes:
        assert ifx.ifx_attention_key_groups(n, heads) == groups, (n, heads)
    for bad in ((0, 12), (4680, 0), (-8, 3)):
        with pytest.raises(ifx.IfxError):
            ifx.ifx_attention_key_groups(*bad)


@pytest.mark.parametrize("n,heads,cached,parts,whole,rows", [
    (1560, 12, 9360, 3, 0, 256), (1560, 12, 1560, 1, 12, 128), (4680, 2, 28080, 6, 0, 256), (1560, 3, 9360, 12, 0, 256), (4000, 1, 24000, 16, 0, 256),
    (1560, 1, 9360, 5, 0, 32), (1560, 2, 9360, 2, 0, 32), (264, 2, 1848, 8, 0, 32), (264, 2, 1056, 1, 2, 32), (264, 2, 528, 1, 2, 32), (1000, 8, 3000, 1, 8, 32),
    (4680, 12, 28080, 1, 12, 256),  # 228 workgroups
    (4680, 14, 14040, 8, 13, 256), (4680, 18, 14040, 1, 18, 128), (10800, 7, 21600, 3, 5, 256), (10800, 6, 21600, 1, 6, 128),  # 266, 342, 301, 258
    (4680, 28, 9360, 6, 26, 256), (1560, 37, 9360, 1, 37, 128), (1560, 40, 9360, 8, 36, 256), (1560, 40, 1560, 1, 40, 128), (10800, 40, 43200, 1, 40, 256),
])
def test_key_parts_where_they_pay(n, heads, cached, parts, whole, rows):
    """To how many workgroups a row tile's keys are dealt, on either side of every line of the rule."""
    assert ifx.ifx_attention_key_parts(n, heads, cached) == (parts, whole, rows)
    for bad in ((0, 12, 8), (8, 0, 8), (8, 1, -1), (8, 1, (1 << 30) + 1)):
        with pytest.raises(ifx.IfxError):
            ifx.ifx_attention_key_parts(*bad)


@pytest.mark.parametrize("n,heads,cached,bf16,fp8", [
    (1000, 1, 1000, 1, 1), (400, 2, 1600, 1, 1), (304, 4, 1520, 1, 1), (160, 12, 1760, 1, 1),                          # up to 8 steps
    (216, 1, 1728, 1, 7), (448, 2, 1792, 1, 8), (680, 1, 1360, 1, 8), (224, 2, 2016, 9, 9), (1000, 1, 2000, 8, 8), (1560, 1, 1560, 5, 5), (1000, 2, 2000, 4, 4),
    (760, 3, 1520, 1, 1), (760, 3, 2280, 1, 3), (752, 4, 3008, 1, 2),                                                  # two to a tile
    (760, 3, 3040, 3, 3), (1424, 2, 2848, 2, 2), (464, 6, 4176, 2, 2), (1000, 3, 4000, 2, 2), (528, 7, 3696, 2, 2), (528, 8, 3696, 1, 1),
])
def test_shared_row_tiles_or_parts(n, heads, cached, bf16, fp8):
    """32-row tiles shared by workgroups, or their keys in parts: on either side of the lines of both caches; what a cache holds
    for partial results has room for either."""
    assert ifx.ifx_attention_key_parts(n, heads, cached)[::2] == (bf16, 32) and ifx.ifx_attention_fp8_key_parts(n, heads, cached)[::2] == (fp8, 32)
    holds = ifx.ifx_attention_area_bytes(n, heads, 128, ifx.IFX_FP8_E4M3, cached // n)
    assert max(bf16, fp8) == 1 or max(bf16, fp8) * heads * ((n + 31) // 32) * (16384 + 512) <= holds
    with pytest.raises(ifx.IfxError):
        ifx.ifx_attention_fp8_key_parts(0, heads, cached)


@pytest.mark.parametrize("n,heads,head_dim,keys,listed,parts,rows", [
    (256, 2, 64, 1024, False, 8, 16), (256, 2, 64, 256, False, 1, 16), (64, 1, 128, 320, False, 1, 16), (400, 4, 128, 2000, False, 5, 16),
    (800, 3, 128, 1600, False, 5, 16), (400, 10, 128, 1200, False, 1, 16), (100, 16, 64, 500, False, 1, 16),
    (1560, 2, 128, 7800, True, 5, 16), (1560, 6, 128, 4680, True, 3, 16), (1560, 12, 128, 3120, True, 1, 16),
    (1560, 2, 128, 7800, False, 18, 256), (1560, 12, 128, 3120, False, 3, 256), (1560, 16, 128, 1560, False, 2, 256), (700, 16, 72, 2100, False, 5, 256),
    (1560, 40, 128, 3120, False, 1, 256),
])
def test_f32_key_parts_where_they_pay(n, heads, head_dim, keys, listed, parts, rows):
    """Which fp32 kernel, and to how many workgroups a row tile's keys are dealt."""
    assert ifx.ifx_attention_f32_key_parts(n, heads, head_dim, keys, listed) == (parts, rows)
    for bad in ((0, 1, 8, 8), (8, 0, 8, 8), (8, 1, 0, 8), (8, 1, 136, 8), (8, 1, 8, -1)):
        with pytest.raises(ifx.IfxError):
            ifx.ifx_attention_f32_key_parts(*bad)


@pytest.mark.parametrize("head_dim", [8, 64, 72, 128])
def test_f32_parts_fit_their_memory(head_dim):
    """At every number of resident blocks, over all of them or listed ones, with the block and without: the parts of an fp32
    call leave at most as many rows (of head_dim rounded up to 32 fp32 numbers, a maximum and a sum) as a stream's memory holds."""
    row_bytes = 4 * ((head_dim + 31) // 32 * 32) + 8
    in_parts = 0
    shapes = [(n, heads, cap) for n in (*range(64, 1601, 56), 1080, 1568) for heads in range(1, 17) for cap in (1, 3, 4)]
    shapes += [(816, 2, 4), (240, 13, 8), (472, 6, 2), (464, 2, 15), (512, 6, 4), (544, 5, 3), (7, 3, 300), (5, 1, 40), (1, 12, 700), (16, 2, 64), (17, 2, 150)]
    for n, heads, cap in shapes:
        tiles = (n + 15) // 16
        holds = ifx.ifx_attention_area_bytes(n, heads, head_dim, ifx.IFX_F32, cap)
        for resident in (range(cap + 1) if cap < 100 else (0, 1, 2, 17, cap // 2, cap - 1, cap)):
            for block_subs in (0, tiles):
                dense, own = (resident * n + 15) // 16 + block_subs, resident * tiles + block_subs
                for subs, listed in ((dense, False), (own, True), (dense if n < 16 else own, True)):
                    parts, _ = ifx.ifx_attention_f32_key_parts(n, heads, head_dim, 16 * subs, listed)
                    if parts > 1:
                        in_parts += 1
                        assert parts * heads * tiles * 16 * row_bytes <= holds, (n, heads, cap, resident, block_subs, listed, parts)
    assert in_parts > 1000


@pytest.mark.parametrize("n,heads,cap", [(264, 2, 7), (1560, 1, 6), (1560, 12, 6), (4680, 14, 3), (10800, 7, 2), (200, 40, 6), (8, 3, 40)])
def test_parts_fit_their_memory(n, heads, cap):
    """The same of bf16 and fp8 calls: units of 32 rows, 16 KiB and 16 bytes a row."""
    holds = ifx.ifx_attention_area_bytes(n, heads, 128, ifx.IFX_BF16, cap)
    assert holds == ifx.ifx_attention_area_bytes(n, heads, 128, ifx.IFX_FP8_E4M3, cap)
    for resident in range(cap + 1):
        for with_block in (False, True):
            parts, whole, _ = ifx.ifx_attention_key_parts(n, heads, resident * n, with_block)
            assert parts == 1 or parts * (heads - whole) * ((n + 31) // 32) * (16384 + 512) <= holds
    for bad in ((0, 1, 128, 1, 1), (8, 0, 128, 1, 1), (8, 1, 64, 1, 1), (8, 1, 128, 7, 1), (8, 1, 128, 1, -1), (8, 1, 136, 0, 1), (8, 1, 128, 1, 1 << 28)):
        with pytest.raises(ifx.IfxError):
            ifx.ifx_attention_area_bytes(*bad)


@pytest.mark.parametrize("heads", [1, 2, 3, 5, 7, 8, 9, 12, 13, 17, 40, 130, 257])
@pytest.mark.parametrize("groups", [1, 2, 8])
def test_attention_group_items_tile_every_head(heads, groups):
    """The launches with one, two and eight key groups, decoded by the functions the kernels use: the
    workgroups' items cover rows 0 .. n - 1 of every head exactly once, at most 8, 4 or 1 wavefronts'
    worth of rows apiece; with eight groups a head's tiles sit on neighbouring XCDs."""
    most = {1: 8, 2: 4, 8: 1}[groups]
    for n in (8, 32, 40, 128, 136, 200, 264, 1032, 1560, 4680):
        if heads > 40 and n > 264:
            continue
        grid = ifx.ifx_attention_group_grid(n, heads, groups)
        assert grid % 8 == 0
        covered = collections.defaultdict(list)
        xcds = collections.defaultdict(set)
        for w in range(grid):
            head, tile, row0, waves, xcd = ifx.ifx_attention_group_item(n, heads, groups, w)
            assert xcd == w % 8
            if groups == 1:
                assert ifx.ifx_attention_launch_item(n, heads, w) == (head, tile, row0, waves, xcd)
            if waves == 0:
                continue
            assert 0 <= head < heads and 1 <= waves <= most and row0 % 32 == 0
            covered[head].append((row0, waves, tile))
            xcds[head].add(xcd)
        assert sorted(covered) == list(range(heads)), n
        for head, items in covered.items():
            items.sort()
            assert [tile for _, _, tile in items] == list(range(len(items)))
            nxt = 0
            for row0, waves, _ in items:
                assert row0 == nxt, (n, head)
                nxt = row0 + 32 * waves
            assert n <= nxt < n + 32  # the last wavefront's worth holds the last row
            if groups == 8:
                assert max(xcds[head]) - min(xcds[head]) + 1 == len(xcds[head])
    for bad in ((0, heads, groups), (8, 0, groups), (8, heads, 4)):
        with pytest.raises(ifx.IfxError):
            ifx.ifx_attention_group_grid(*bad)
    with pytest.raises(ifx.IfxError):
        ifx.ifx_attention_group_item(8, heads, groups, ifx.ifx_attention_group_grid(8, heads, groups))


def test_kernels_need_no_scratch_memory(tmp_path):
    """A kernel with spilled registers makes the runtime allocate scratch memory at its launch, behind
    the back of callers that may not allocate.  Only the block-table instances over an fp8 cache
    have any (a few registers, as the one-group instance always had)."""
    import shutil
    import subprocess

    llvm = "/opt/rocm/llvm/bin"
    tools = [os.path.join(llvm, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")]
    if not all(shutil.which(t) for t in tools):
        pytest.skip("no LLVM tools")
    objcopy, bundler, readelf = tools
    ifx.lib()
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    subprocess.check_call([objcopy, "--dump-section", ".hip_fatbin=" + fat, ifx.LIB_PATH, str(tmp_path / "copy")])
    subprocess.check_call([bundler, "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat, "--output=" + code])
    notes = subprocess.check_output([readelf, "--notes", code], text=True)
    kernels = re.findall(r"\.name:\s+(\S*kernel\S*)\n\s+\.private_segment_fixed_size:\s+(\d+)", notes)
    assert len(kernels) >= 20
    with_scratch = {name: int(size) for name, size in kernels if int(size)}
    assert all("attn_bf16_kernelILb1ELb1E" in name and size <= 40 for name, size in with_scratch.items()), with_scratch
