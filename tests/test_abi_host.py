"""CPU-side checks of the C ABI: the library loads, exports what prism.h
declares, rejects bad arguments, and its host planner covers every
(request, kv head, row, key) exactly once."""
import ctypes
import os
import re
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2605_08581_amd import binding as B
from paper_2605_08581_amd import workload as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2605_08581_amd import build
        build.build()
    return B.load()


def test_library_exports_every_declared_symbol(lib):
    from paper_2605_08581_amd import sched as S
    declared = set()
    for name, exports in (("prism.h", B.EXPORTS), ("prism_sched.h", S.EXPORTS)):
        header = open(os.path.join(ROOT, "include", name)).read()
        body = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
        found = set(re.findall(r"\b(prism_[a-z_]+)\s*\(", body))
        assert found == set(exports), name
        declared |= found
    assert sorted(os.listdir(os.path.join(ROOT, "include"))) == ["prism.h", "prism_sched.h"]
    for name in declared:
        assert hasattr(lib, name), name
    assert B.prism_version() == 200
    assert lib.prism_strerror(B.ERR_UNSUPPORTED).decode().startswith("unsupported")


def _shape(**kw):
    base = dict(num_q_heads=8, num_kv_heads=2, head_dim=128, num_pages=64, batch=2,
                max_blocks_per_req=8, softmax_scale=0.1)
    base.update(kw)
    return B.make_shape(**base)


def test_shape_errors(lib):
    P, S = [16, 0], [5, 7]
    for kw, code in [(dict(page_size=32), B.ERR_UNSUPPORTED), (dict(head_dim=96), B.ERR_UNSUPPORTED),
                     (dict(num_q_heads=7), B.ERR_INVALID_ARG), (dict(batch=0), B.ERR_INVALID_ARG),
                     (dict(softmax_scale=0.0), B.ERR_INVALID_ARG), (dict(num_pages=0), B.ERR_INVALID_ARG),
                     (dict(max_blocks_per_req=1), B.ERR_INVALID_ARG)]:
        with pytest.raises(B.PrismError) as e:
            B.prism_plan_dry_run(_shape(**kw), P, S)
        assert e.value.code == code, kw
    with pytest.raises(B.PrismError) as e:
        B.prism_plan_dry_run(_shape(), [16, -1], S)
    assert e.value.code == B.ERR_INVALID_ARG
    with pytest.raises(B.PrismError) as e:
        B.prism_plan_dry_run(_shape(), P, S, tile_rows=96)
    assert e.value.code == B.ERR_UNSUPPORTED
    assert lib.prism_plan_create(None, None, None, None, None) == B.ERR_INVALID_ARG
    assert lib.prism_kv_append(None, None, None, None, None, None, None) == B.ERR_INVALID_ARG
    assert lib.prism_prefix_prefill(*([None] * 9), 0, None) == B.ERR_INVALID_ARG
    assert lib.prism_prefix_attention(*([None] * 7), 0, None) == B.ERR_INVALID_ARG


def _check_cover(b, tile_rows, split_kv, min_split_keys=0):
    sh = B.shape_of(b)
    info, ws, items = B.prism_plan_dry_run(sh, b.prefix_len, b.suffix_len, tile_rows, split_kv,
                                           min_split_keys)
    G = b.geom.group
    tr = info.tile_rows
    assert info.tile_keys == 64 and info.num_items == len(items)
    cover = {}
    slots = set()
    die = {}
    for pos, (req, kvh, row0, kb, ke, slot, P, S) in enumerate(items.tolist()):
        if req < 0:
            continue                     # idle padding of the die interleave
        die.setdefault((req, kvh), set()).add(pos % 8)
        assert P == b.prefix_len[req] and S == b.suffix_len[req]
        assert row0 % tr == 0 and 0 <= row0 < S * G
        last_row = min(S * G, row0 + tr) - 1
        kv_len = P + last_row // G + 1
        assert 0 <= kb < ke <= kv_len and kb % 64 == 0
        cover.setdefault((req, kvh, row0), []).append((kb, ke, slot, kv_len))
        if slot >= 0:
            assert slot not in slots
            slots.add(slot)
    assert all(len(v) == 1 for v in die.values()), "one (request, kv head) must stay on one die"
    want = {(r, h, t * tr) for r in range(b.batch) for h in range(b.geom.num_kv_heads)
            for t in range(-(-int(b.suffix_len[r]) * G // tr))}
    assert set(cover) == want
    nsplit_items = 0
    for key, chunks in cover.items():
        chunks.sort()
        assert chunks[0][0] == 0 and chunks[-1][1] == chunks[0][3]
        for a, c in zip(chunks, chunks[1:]):
            assert a[1] == c[0], "key ranges of one row tile must tile the visible keys"
        if len(chunks) == 1:
            assert chunks[0][2] == -1
        else:
            assert all(c[2] >= 0 for c in chunks)
            assert [c[2] for c in chunks] == list(range(chunks[0][2], chunks[0][2] + len(chunks)))
            nsplit_items += len(chunks)
    assert info.num_split_items == nsplit_items == len(slots)
    # workspace: the work lists (64-byte items, 32-byte merge groups, each part
    # padded to 256 bytes), then one fp32 partial slot per split item
    up = lambda n: -(-n // 256) * 256
    assert ws == up(64 * info.num_items) + up(32 * info.num_reduce_groups) + len(slots) * tr * (b.geom.head_dim + 2) * 4
    S64, P64 = b.suffix_len.astype(np.int64), b.prefix_len.astype(np.int64)
    assert info.flops == 4 * b.geom.head_dim * b.geom.num_q_heads * int((S64 * P64 + S64 * (S64 + 1) // 2).sum())
    assert info.total_suffix == b.total_suffix
    return info


@pytest.mark.parametrize("index", [0, 1, 2, 4])
@pytest.mark.parametrize("tile_rows", [0, 64, 256])
def test_planner_covers_every_pair_once(lib, index, tile_rows):
    _check_cover(W.make_config(index), tile_rows, 0)


@pytest.mark.parametrize("seed", range(24))
def test_planner_random_waves(lib, seed):
    """Seeded random waves (empty requests, no prefix, single tokens, long and
    short mixes, every head grouping) under every tile shape and split policy:
    each (request, kv head, row, key) is covered exactly once."""
    rng = np.random.default_rng(1000 + seed)
    hkv = int(rng.choice([1, 2, 4, 5, 8]))
    geom = W.Geometry(hkv * int(rng.choice([1, 2, 3, 4, 8])), hkv, int(rng.choice([64, 128])))
    n = int(rng.integers(1, 12))
    prefix = [int(rng.choice([0, 16, 100, 1000, 5000])) * int(rng.integers(0, 3)) for _ in range(n)]
    suffix = [int(rng.choice([0, 1, 2, 31, 32, 33, 127, 128, 129, 700])) for _ in range(n)]
    if sum(suffix) == 0:
        suffix[0] = 5
    b = W.make_custom_batch("rnd", geom, prefix, suffix, seed=seed)
    tile_rows = int(rng.choice([0, 64, 128, 256]))
    split_kv = int(rng.choice([0, 1, 2, 9]))
    _check_cover(b, tile_rows, split_kv, min_split_keys=int(rng.choice([0, 64, 512])))


def test_planner_forced_and_disabled_split(lib):
    b = W.make_custom_batch("t", W.Geometry(8, 2, 128), [0, 100, 1000, 37], [5, 0, 300, 129], seed=1)
    assert _check_cover(b, 128, 1).num_split_items == 0
    assert _check_cover(b, 128, 3).num_split_items > 0
    assert _check_cover(b, 64, 0, min_split_keys=64).num_reduce_groups >= 0
    long_rag = _check_cover(W.make_config(4), 0, 0)
    assert long_rag.num_reduce_groups > 0, "long prefixes with few requests must be split"
    assert _check_cover(W.make_config(2), 0, 0).num_reduce_groups == 0


@pytest.mark.parametrize("d,rows", [(128, (1, 9)), (64, (1, 9)), (128, (33, 500)), (64, (33, 500))])
@pytest.mark.parametrize("least", [0, 64, 1280])
def test_pieces_are_not_too_short(lib, d, rows, least):
    rng = np.random.default_rng(11)
    cut = 0
    for _ in range(60):
        n = int(rng.integers(1, 9))
        b = W.make_custom_batch("even", W.Geometry(8, 4, d), rng.integers(0, 9000, n).tolist(),
                                rng.integers(rows[0], rows[1], n).tolist(), seed=1)
        _check_cover(b, 0, 0, least)
        items = B.prism_plan_dry_run(B.shape_of(b), b.prefix_len, b.suffix_len, min_split_keys=least)[2]
        tiles = {}
        for req, kvh, row0, kb, ke, slot, _, _ in items[items[:, 0] >= 0].tolist():
            if slot >= 0:
                tiles.setdefault((req, kvh, row0), {})[kb] = (ke + 63) // 64 - kb // 64
        for piece in tiles.values():
            lengths = [piece[kb] for kb in sorted(piece)]
            assert min(lengths if least else lengths[:-1]) >= (least or 256) // 64, lengths
        cut += len(tiles)
    assert cut > 0


@pytest.mark.parametrize("d,rows,batch,keys,stream", [
    (128, 18, 7, 60, False), (128, 18, 6, 60, True), (128, 9, 27, 60, False), (128, 16, 7, 640, False),
    (128, 16, 7, 720, True), (128, 32, 7, 1900, False), (128, 32, 7, 2100, True), (64, 16, 13, 190, False),
    (64, 16, 13, 280, True), (64, 32, 13, 960, False), (64, 32, 13, 1100, True), (64, 32, 12, 60, True),
    (128, 33, 1, 4000, False)])
def test_key_splitting_kernel_only_where_it_is_ahead(lib, d, rows, batch, keys, stream):
    """Up to 32 rows go to it while every (request, kv head) has a place on the chip, and beyond that
    only with long key ranges."""
    b = W.make_custom_batch("few", W.Geometry(40, 40, d), [keys - rows] * batch, [rows] * batch, seed=1)
    assert _check_cover(b, 0, 0).tile_rows == ((16 if rows <= 16 else 32) if stream else 128)


@pytest.mark.parametrize("heads,prefix,suffix,rows", [
    ((8, 8, 128), [0], [512], 16), ((8, 8, 128), [0], [513], 128), ((8, 8, 64), [0], [1024], 16), ((8, 8, 64), [0], [1025], 128),
    ((8, 2, 128), [200], [128], 16), ((8, 2, 128), [200], [129], 128), ((32, 8, 128), [1240], [40], 16),
    ((32, 8, 128), [1241], [40], 128), ((32, 8, 64), [1368], [40], 16), ((32, 8, 64), [1369], [40], 128),
    ((40, 40, 128), [100] * 2, [33, 17], 16), ((40, 40, 128), [100] * 2, [33, 49], 128), ((40, 40, 128), [100] * 4, [17] * 4, 32)],
    ids=["places128", "above128", "places64", "above64", "die", "above-die", "longest128", "longer128", "longest64", "longer64",
         "heads-over-dies", "more-than-places", "too-many-few-rows"])
def test_row_tiles_of_sixteen_while_they_find_places(lib, heads, prefix, suffix, rows):
    """Every tile a place at once, on its set's die, over ranges that four waves read alone; whole ranges."""
    b = W.make_custom_batch("tiles", W.Geometry(*heads), prefix, suffix, seed=1)
    info = _check_cover(b, 0, 0)
    assert info.tile_rows == rows and (rows > 16 or info.num_split_items == 0)


def test_row_tiles_of_sixteen_are_dealt_as_they_were_counted(lib):
    """Sets of as many key tiles, in 20 row tiles and in two, turn and turn about: 176 row tiles, 22 a die."""
    b = W.make_custom_batch("ties", W.Geometry(8, 1, 128), [80, 1270] * 8, [40, 4] * 8, seed=1)
    info, _, items = B.prism_plan_dry_run(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table)
    assert info.tile_rows == 16 and np.bincount(np.flatnonzero(items[:, 0] >= 0) % 8, minlength=8).tolist() == [22] * 8


@pytest.mark.parametrize("heads,prefix,suffix,pieces", [
    ((32, 8, 128), [639] * 2, [1] * 2, {64: 80, 128: 48, 256: 32}), ((32, 8, 64), [511] * 3, [4] * 3, {64: 120, 128: 72, 256: 48}),
    ((32, 8, 128), [1003], [37], {64: 240, 512: 160, 1024: 80})], ids=["decode", "few-rows-d64", "row-tiles"])
def test_smallest_piece_of_the_caller_is_used_where_the_default_leaves_ranges_whole(lib, heads, prefix, suffix, pieces):
    b = W.make_custom_batch("least", W.Geometry(*heads), prefix, suffix, seed=1)
    whole = _check_cover(b, 0, 0)
    assert whole.tile_rows == 16 and whole.num_split_items == 0
    for least, want in pieces.items():
        info = _check_cover(b, 0, 0, min_split_keys=least)
        assert info.tile_rows == 16 and info.num_items == want and info.num_split_items in (0, want)


@pytest.mark.parametrize("heads,prefix,suffix,groups,tile_rows", [
    ((8, 1, 64), [0], [4096], [-1], 0), ((8, 1, 64), [18612] * 3, [1648, 2400, 3297], [-1] * 3, 0), ((8, 2, 128), [373] * 3, [2685] * 3, [-1] * 3, 0),
    ((4, 1, 128), [512] * 5, [700, 300, 500, 600, 400], [0] * 5, 0), ((8, 1, 128), [0, 100], [400, 37], [-1] * 2, 64), ((4, 4, 64), [0, 100], [6200, 37], [-1] * 2, 0),
    ((8, 2, 128), [0, 9, 500, 16] * 3, [2100, 2050, 40, 2200] * 3, [-1] * 12, 0), ((8, 1, 128), [8192], [800], [-1], 0),
    ((8, 1, 64), [30000], [800], [-1], 0), ((8, 1, 128), [16384], [960], [-1], 0), ((8, 1, 64), [0], [800], [-1], 0)],
    ids=["one-request", "cut-too", "three", "sharers", "64-rows", "four-heads", "more-sets-than-dies", "57-tiles", "50-tiles",
         "60-tiles", "50-tiles-uncut"])
def test_sets_larger_than_a_die_are_dealt_out(lib, heads, prefix, suffix, groups, tile_rows):
    """More row tiles in one (cluster, kv head) set than one and a half for each CU of a die: every die has work
    and none more than a quarter above an eighth of the wave and one workgroup, and every key of every row tile
    belongs to one workgroup."""
    b = W.make_custom_batch("dealt", W.Geometry(*heads), prefix, suffix, seed=1, share_groups=groups)
    info, _, items = B.prism_plan_dry_run(B.shape_of(b), b.prefix_len, b.suffix_len, tile_rows=tile_rows, block_table=b.block_table)
    load, longest, ranges = np.zeros(8, np.int64), 0, {}
    for pos, (req, kvh, row0, kb, ke, *_) in enumerate(items.tolist()):
        if req >= 0:
            load[pos % 8] += (ke - kb + 63) // 64
            longest = max(longest, (ke - kb + 63) // 64)
            ranges.setdefault((req, kvh, row0), []).append((kb, ke))
    G, tr = b.geom.group, info.tile_rows
    want = {(r, h, row0): b.prefix_len[r] + (min(b.suffix_len[r] * G, row0 + tr) - 1) // G + 1 for r in range(b.batch)
            for h in range(b.geom.num_kv_heads) for row0 in range(0, int(b.suffix_len[r]) * G, tr)}
    assert set(ranges) == set(want)
    for key, pieces in ranges.items():
        pieces.sort()
        assert pieces[0][0] == 0 and pieces[-1][1] == want[key] and all(x[1] == y[0] for x, y in zip(pieces, pieces[1:]))
    assert load.min() > 0 and load.max() <= 1.25 * load.mean() + longest, load.tolist()


@pytest.mark.parametrize("heads,prefix,suffix,least,most", [
    ((8, 1, 64), [15838], [34], 8, 30), ((8, 2, 128), [224, 480], [750] * 2, 1, 1), ((8, 2, 128), [224, 480], [1116] * 2, 1, 3),
    ((8, 1, 128), [16384] * 2, [480] * 2, 7, 9), ((8, 2, 128), [8192] * 2, [1000] * 2, 4, 4), ((32, 8, 64), [2448] * 22, [12] * 22, 2, 5)],
    ids=["deep-merge", "full-tiles", "full-tiles-dealt-out", "sharers-dealt-out", "two-heads-dealt-out", "few-rows-d64"])
def test_cuts_weigh_the_merge(lib, heads, prefix, suffix, least, most):
    """Pieces of a row tile where the estimate has to see how deep the merge gets, how many rows of partials
    it moves, how many dies the wave reaches - two sets of 48 row tiles stay on theirs, sets of sharers with 60
    and more are dealt out - and that a key tile takes half the time at d = 64."""
    b = W.make_custom_batch("merge", W.Geometry(*heads), prefix, suffix, seed=1,
                            share_groups=[-1 if len(prefix) > 2 else 0] * len(prefix))
    items = B.prism_plan_dry_run(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table)[2]
    pieces = {}
    for req, kvh, row0, *_ in items[items[:, 0] >= 0].tolist():
        pieces[req, kvh, row0] = pieces.get((req, kvh, row0), 0) + 1
    assert least <= min(pieces.values()) and max(pieces.values()) <= most, sorted(pieces.values())


SCRATCH = 64 << 20                             # PRISM_STATIC_SCRATCH_BYTES


@pytest.mark.parametrize("prefix,suffix", [([21234, 27950, 30066], [394, 200, 307]),
                                           ([34959, 52451, 19008, 58356], [172, 398, 314, 113])])
@pytest.mark.parametrize("tile_rows", [0, 64, 256])
def test_automatic_cuts_fit_the_static_scratch(lib, prefix, suffix, tile_rows):
    """Waves whose pieces at four workgroups per CU would not fit it."""
    b = W.make_custom_batch("scratch", W.Geometry(32, 8, 128), prefix, suffix, seed=1)
    assert _check_cover(b, tile_rows, 0).num_split_items > 0
    assert B.prism_plan_dry_run(B.shape_of(b), b.prefix_len, b.suffix_len, tile_rows=tile_rows)[1] <= SCRATCH


def test_automatic_cuts_of_random_waves_fit_the_static_scratch(lib):
    rng = np.random.default_rng(7)
    for _ in range(400):
        n, hkv = int(rng.integers(2, 25)), int(rng.choice([1, 2, 8, 40]))
        prefix, suffix = rng.integers(16384, 65537, n), rng.integers(33, 401, n)
        sh = B.make_shape(hkv * int(rng.choice([1, 4])), hkv, 128, 1 << 16, n, 4200, 0.1)
        for tile_rows, width in ((0, 0), (256, 64)):
            ws = B.prism_plan_dry_run(sh, prefix, suffix, tile_rows=tile_rows, rows_per_wave=width)[1]
            assert ws <= SCRATCH, (sh.num_q_heads, hkv, prefix.tolist(), suffix.tolist(), tile_rows)


def test_placement_hint_keeps_prefix_sharers_on_one_die(lib):
    """With a host block table, requests whose tables start with the same page
    (a common cached prefix) run the same kv head on the same die."""
    b = W.make_config(2)
    sh = B.shape_of(b)
    _, _, items = B.prism_plan_dry_run(sh, b.prefix_len, b.suffix_len, block_table=b.block_table)
    _, _, plain = B.prism_plan_dry_run(sh, b.prefix_len, b.suffix_len)
    key = lambda it: tuple(sorted(map(tuple, it[it[:, 0] >= 0][:, :6].tolist())))
    assert key(items) == key(plain), "the hint may only reorder the work"
    first = {r: int(b.block_table[r, 0]) for r in range(b.batch) if b.prefix_len[r] >= 16}
    die = {}
    for pos, (req, kvh, *_rest) in enumerate(items.tolist()):
        if req >= 0 and req in first:
            die.setdefault((first[req], kvh), set()).add(pos % 8)
    assert len({k[0] for k in die}) < len(first), "the Zipf wave has requests with a common prefix"
    assert all(len(v) == 1 for v in die.values())


MIB = 1 << 20


@pytest.mark.parametrize("private,shared,flagged", [
    (32, [], False), (32 + 1 / 16, [], True), (64, [], True), (0, [(64, 2)], False),
    (2, [(8, 28)], False), (24, [(3, 10), (2, 3)], False), (24, [(4, 10), (5, 2)], True), (33, [(1, 2)], True)],
    ids=["at-the-line", "a-page-more", "private", "no-private", "many-sharers", "two-clusters-below", "two-clusters-above",
         "private-above"])
@pytest.mark.parametrize("geom", [W.Geometry(32, 8, 128), W.Geometry(40, 40, 64)], ids=["gqa128", "mha64"])
def test_pages_read_past_the_caches(lib, geom, private, shared, flagged):
    """The pages of requests that share none, if the wave's distinct pages (private: MiB of four requests'
    own; shared: MiB of a prefix and how many have it) are more than the 32 MiB of the dies' L2 caches."""
    token = 4 * geom.num_kv_heads * geom.head_dim                # bytes of K and V
    total = int(private * MIB / token)
    own = [total // 4] * 3 + [total - total // 4 * 3] if private else []
    prefix, groups = [n - 1 for n in own], [-1] * len(own)
    for g, (size, sharers) in enumerate(shared):
        prefix += [int(size * MIB / token) // 16 * 16] * sharers   # and a page each for the new token
        groups += [g] * sharers
    b = W.make_custom_batch("once", geom, prefix, [1] * len(prefix), seed=1, share_groups=groups)
    args = (B.shape_of(b), b.prefix_len, b.suffix_len)
    once = lambda **kw: B.prism_plan_dry_run_read_once(*args, **kw)
    info, _, items = B.prism_plan_dry_run(*args, block_table=b.block_table)
    assert info.tile_rows == 16
    assert np.array_equal(once(block_table=b.block_table), flagged & (items[:, 0] >= 0) & (items[:, 0] < len(own)))
    assert not once().any() and not once(block_table=b.block_table, tile_rows=128).any()


def test_append_inside_attention_needs_a_final_table(lib):
    """A table that is only a placement hint may differ from the one on the device: nothing but the order
    of the work follows from it.  Options that a caller has zeroed say just that."""
    b = W.make_custom_batch("hint", W.Geometry(4, 2, 128), [32, 48], [20, 200], seed=1)
    args = (B.shape_of(b), b.prefix_len, b.suffix_len)
    fused = lambda **kw: B.prism_plan_dry_run(*args, **kw)[0].append_in_attention
    assert fused(block_table=b.block_table) == 1
    assert fused(block_table=b.block_table, table_is_final=False) == 0
    assert fused() == 0
    assert fused(block_table=b.block_table, rows_per_wave=64) == 0
    table = b.block_table.copy()
    table[1, :3] = table[0, :3]                # a cached prefix that the same wave writes
    assert fused(block_table=table) == 0
    opt, info = B.PlanOptions(), B.PlanInfo()
    opt.block_table_host = b.block_table.ctypes.data
    lib.prism_plan_dry_run(ctypes.byref(args[0]), args[1].ctypes.data, args[2].ctypes.data, ctypes.byref(opt),
                           ctypes.byref(info), None, None, 0)
    assert info.num_items > 0 and info.append_in_attention == 0


def test_plan_needs_no_memory_for_pages_outside_the_wave(lib):
    """A pool of 2^30 pages: an array over it (4 GiB) does not fit the limit set here."""
    code = """
import resource
from paper_2605_08581_amd import binding as B, workload as W
b = W.make_custom_batch("x", W.Geometry(4, 2, 128), [0, 37, 500], [40, 1, 7], seed=1)
sh = B.shape_of(b)
plan = lambda: B.prism_plan_dry_run(sh, b.prefix_len, b.suffix_len, block_table=b.block_table)
plan()
now = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (now + (256 << 20),) * 2)
sh.num_pages = 1 << 30
print(plan()[0].num_items)
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0 and int(r.stdout) > 0, r.stderr[-2000:]


def test_validate_flags_bad_tables(lib):
    b = W.make_custom_batch("t", W.Geometry(4, 2, 64), [32, 32, 5], [20, 9, 30], seed=2,
                            share_groups=[0, 0, -1])
    sh = B.shape_of(b)
    assert B.prism_validate(sh, b.prefix_len, b.suffix_len, b.block_table) == B.PRISM_OK
    bt = b.block_table.copy()
    bt[0, 0] = b.num_pages                     # out of range
    assert B.prism_validate(sh, b.prefix_len, b.suffix_len, bt) == B.ERR_TABLE
    bt = b.block_table.copy()
    bt[1, 2] = bt[0, 2]                        # two requests append into one page
    assert B.prism_validate(sh, b.prefix_len, b.suffix_len, bt) == B.ERR_TABLE
    bt = b.block_table.copy()
    bt[2, 1] = bt[0, 0]                        # an append lands in a cached page
    assert B.prism_validate(sh, b.prefix_len, b.suffix_len, bt) == B.ERR_TABLE
    bt = b.block_table.copy()
    bt[0, 3] = bt[0, 2]                        # one request maps two blocks to one page
    assert B.prism_validate(sh, b.prefix_len, b.suffix_len, bt) == B.ERR_TABLE
    assert B.prism_validate(sh, [32, 32, 5000], b.suffix_len, b.block_table) == B.ERR_INVALID_ARG


def test_measure_peaks_rejects_bad_arguments(lib):
    m, h = ctypes.c_double(), ctypes.c_double()
    assert lib.prism_measure_peaks(None, 1 << 30, 1, ctypes.byref(m), ctypes.byref(h), None) == B.ERR_INVALID_ARG
    assert lib.prism_measure_peaks(ctypes.c_void_p(4096), 16, 1, ctypes.byref(m), ctypes.byref(h), None) == B.ERR_INVALID_ARG
    assert lib.prism_measure_peaks(ctypes.c_void_p(4096), 1 << 30, 0, ctypes.byref(m), ctypes.byref(h), None) == B.ERR_INVALID_ARG
    assert lib.prism_measure_peaks(ctypes.c_void_p(4096), 1 << 30, 1, None, ctypes.byref(h), None) == B.ERR_INVALID_ARG


@pytest.mark.parametrize("k_off,v_off", [(8, 0), (0, 2), (4, 4)])
@pytest.mark.parametrize("suffix", [[3, 1], [200, 40]], ids=["few-rows", "tiles"])
def test_pools_off_the_16_byte_grid_are_refused(lib, suffix, k_off, v_off):
    """Refused before anything is launched: the addresses here belong to nobody."""
    b = W.make_custom_batch("off", W.Geometry(4, 2, 64), [32, 5], suffix, seed=2)
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len)
    at, n = ctypes.c_void_p(1 << 20), plan.prism_plan_workspace_bytes()
    k, v = ctypes.c_void_p((1 << 20) + k_off), ctypes.c_void_p((1 << 20) + v_off)
    assert lib.prism_prefix_attention(plan._h, at, k, v, at, at, at, n, None) == B.ERR_INVALID_ARG
    assert lib.prism_prefix_prefill(plan._h, at, at, at, k, v, at, at, at, n, None) == B.ERR_INVALID_ARG
    assert lib.prism_prefix_prefill_static(plan._h, at, at, at, k, v, at, at, None) == B.ERR_INVALID_ARG
    plan.close()


@pytest.mark.parametrize("make", [lambda n: torch.empty(-(-n // 4), dtype=torch.float32),
                                  lambda n: torch.empty(-(-n // 4) * 2, dtype=torch.float32)[::2],
                                  lambda n: torch.empty(n, dtype=torch.uint8)],
                         ids=["few-wide-elements", "strided", "host"])
def test_workspace_of_another_kind_is_refused(lib, make):
    """Large enough in bytes, so the library would take the pointer: the tensors, here all on the host,
    must be checked before it sees the call."""
    b = W.make_custom_batch("ws", W.Geometry(4, 2, 64), [32, 5], [20, 9], seed=2)
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, split_kv=2)
    n, ws = plan.prism_plan_workspace_bytes(), make(plan.prism_plan_workspace_bytes())
    assert n > 0 and ws.numel() * ws.element_size() >= n
    t = W.make_tensors(b, "cpu")
    table, out = torch.from_numpy(b.block_table), torch.empty_like(t["q"])
    with pytest.raises(ValueError):
        plan.prism_prefix_attention(t["q"], t["k_pool"], t["v_pool"], table, out, ws)
    with pytest.raises(ValueError):
        plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], table, out, ws)
    plan.close()


def test_layer_call_that_torch_refuses_raises():
    """Without a device torch has no current stream: an exception in Python, and not the end of the process."""
    code = """
from paper_2605_08581_amd import binding as B, workload as W
b = W.make_custom_batch("x", W.Geometry(2, 2, 64), [16], [5], seed=1)
plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len)
for call, n in ((plan.prism_prefix_attention, 5), (plan.prism_prefix_prefill, 7)):
    try:
        call(*[None] * n)
    except Exception as e:
        print("raised")
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", CUDA_VISIBLE_DEVICES="")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.split() == ["raised"] * 2, r.stderr[-2000:]
