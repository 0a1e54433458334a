"""GPU parity of the kernel for few rows per kv head (its waves split the keys):
row blocks of 16, both head dims, prefixes that end inside a page (rows of one
page come from the pool and from the packed arrays), split keys with the merge
by the last workgroup, and the append done by the attention workgroups."""
import numpy as np
import pytest
import torch

from paper_2605_08581_amd import binding as B
from paper_2605_08581_amd import workload as W

from gpu_util import check_close, full_parity, widen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,suffix", [(1, [1, 15, 16]), (4, [1, 4, 3]), (1, [17, 32, 1]), (8, [2, 4, 1]),
                                          (1, [33, 64, 63]), (5, [12, 7, 1])],
                         ids=["16", "g4x16", "32", "g8x32", "64", "g5x60"])
def test_row_blocks_and_page_edges(oracle_lib, group, suffix, d):
    """Up to 16 and 32 rows, and 33 to 64 (the prefill kernel again); cached lengths 0, inside a page, on a page edge,
    around the 32-key tile and far past it; sequences of a single key."""
    prefix = [0, 37, 1500] if suffix[0] > 1 else [1000, 16, 31]
    b = W.make_custom_batch("stream", W.Geometry(2 * group, 2, d), prefix + [0], suffix + [1], seed=61)
    info = full_parity(oracle_lib, b)
    rows = max(suffix) * group
    assert info.tile_rows == (16 if rows <= 16 else 32 if rows <= 32 else 128)
    full_parity(oracle_lib, b, split_kv=3)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,prefix,suffix", [
    (1, [0, 37, 1100], [17, 33, 20]), (4, [1003], [37]), (5, [0, 16, 250], [13, 7, 1]), (3, [31, 640], [47, 16]),
    (8, [5], [61]), (1, [0], [256])], ids=["mha", "one-request", "g5", "g3", "g8", "one-place-each"])
def test_more_rows_in_tiles_of_sixteen(oracle_lib, group, prefix, suffix, d):
    """Waves that find a place for every row tile at once: tiles that begin and end inside a token's group of
    heads, last tiles of one row, new rows appended by the tile that owns their token, keys cut by the caller."""
    b = W.make_custom_batch("row-tiles", W.Geometry(4 * group, 4, d), prefix, suffix, seed=67)
    assert full_parity(oracle_lib, b).tile_rows == 16
    full_parity(oracle_lib, b, entry="separate")
    full_parity(oracle_lib, b, split_kv=3)


@pytest.mark.parametrize("geom", [W.Geometry(8, 8, 128), W.Geometry(32, 8, 128), W.Geometry(8, 1, 64)],
                         ids=["mha128", "gqa128", "mqa64"])
def test_wave_larger_than_the_chip(oracle_lib, geom):
    """Enough workgroups for two waves each, ragged lengths, split by the planner; two calls in a
    row on one workspace (the arrival counters must be back at zero)."""
    rng = np.random.default_rng(3)
    n = 48
    b = W.make_custom_batch("many", geom, rng.integers(1, 1800, n).tolist(), [1] * n, seed=62)
    t = W.make_tensors(b, "cuda")
    host = {k: W.bf16_bits(v) for k, v in t.items()}
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table)
    ws = torch.empty(plan.prism_plan_workspace_bytes(), dtype=torch.uint8, device="cuda")
    bt = torch.from_numpy(b.block_table).cuda()
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  b.block_table, b.prefix_len, b.suffix_len)
    ref = oracle_lib.attention(host["q"], kp, vp, b.block_table, b.prefix_len, b.suffix_len, b.softmax_scale)
    for _ in range(2):
        out = torch.full_like(t["q"], float("nan"))
        plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], bt, out, ws)
        torch.cuda.synchronize()
        check_close(widen(W.bf16_bits(out)), ref, b.name)
    plan.close()
    assert np.array_equal(W.bf16_bits(t["k_pool"]), kp) and np.array_equal(W.bf16_bits(t["v_pool"]), vp)


@pytest.mark.parametrize("geom,suffix,rows", [
    (W.Geometry(8, 8, 128), 1, 16), (W.Geometry(8, 8, 128), 4, 16), (W.Geometry(40, 8, 128), 1, 16),
    (W.Geometry(40, 8, 128), 4, 32), (W.Geometry(16, 16, 64), 1, 16), (W.Geometry(16, 16, 64), 4, 16),
    (W.Geometry(32, 8, 64), 8, 32)],
    ids=["mha128-one", "mha128-four", "g5x128-one", "g5x128-four", "mha64-one", "mha64-four", "g4x64-eight"])
def test_waves_larger_than_the_l2_caches(oracle_lib, geom, suffix, rows):
    """Just above and below 32 MiB of different pages, beyond which those of one request alone are read
    past the caches: shared and private prefixes in one wave, some ending inside a page."""
    token = 4 * geom.num_kv_heads * geom.head_dim   # bytes of K and V
    line = (32 << 20) // token
    groups = [-1] * 6 + [0, 0, 0, 1, 1, -1]
    own = [r for r, g in enumerate(groups) if g < 0]
    each = line // 10
    prefix = [each - 7] * 6 + [each // 16 * 16] * 6
    make = lambda: W.make_custom_batch("once", geom, prefix, [suffix] * 12, seed=66, share_groups=groups)
    shared = {int(p) for r in range(12) if r not in own
              for p in make().block_table[r, :-(-(prefix[r] + suffix) // 16)]}
    for total in (line + 200, line - 200):
        prefix[0] += total - sum(prefix[r] + suffix for r in own) - 16 * len(shared)
        b = make()
        args = (B.shape_of(b), b.prefix_len, b.suffix_len)
        items = B.prism_plan_dry_run(*args, block_table=b.block_table)[2]
        once = B.prism_plan_dry_run_read_once(*args, block_table=b.block_table)
        assert np.array_equal(once, np.isin(items[:, 0], own) & (total > line))
        assert full_parity(oracle_lib, b).tile_rows == rows


@pytest.mark.parametrize("suffix", [[20, 20], [150, 40]], ids=["stream", "tile"])
@pytest.mark.parametrize("hint", [True, False], ids=["table", "no-table"])
def test_prefix_pages_written_by_the_same_wave(oracle_lib, suffix, hint):
    """The second request's cached prefix is what the first one appends in this
    very call: attention must then see the appended rows."""
    geom = W.Geometry(2, 2, 128)
    b = W.make_custom_batch("in-wave", geom, [32, 48], suffix, seed=63)
    table = b.block_table.copy()
    table[1, :3] = table[0, :3]                    # positions 32..47 of request 0 are new tokens
    t = W.make_tensors(b, "cuda")
    host = {k: W.bf16_bits(v) for k, v in t.items()}
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=table if hint else None)
    ws = torch.empty(plan.prism_plan_workspace_bytes(), dtype=torch.uint8, device="cuda")
    out = torch.full_like(t["q"], float("nan"))
    plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"],
                              torch.from_numpy(table).cuda(), out, ws)
    torch.cuda.synchronize()
    plan.close()
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  table, b.prefix_len, b.suffix_len)
    assert np.array_equal(W.bf16_bits(t["k_pool"]), kp) and np.array_equal(W.bf16_bits(t["v_pool"]), vp)
    ref = oracle_lib.attention(host["q"], kp, vp, table, b.prefix_len, b.suffix_len, b.softmax_scale)
    check_close(widen(W.bf16_bits(out)), ref, b.name)


def test_slots_past_the_sequence_hold_nan(oracle_lib):
    """Unused slots of the last page must not reach the products, whether the
    new rows come from the packed arrays or from the pool."""
    b = W.make_custom_batch("nan", W.Geometry(4, 4, 128), [32, 5], [21, 2], seed=64)

    def mutate(t):
        for r in range(b.batch):
            T = int(b.prefix_len[r] + b.suffix_len[r])
            pg = int(b.block_table[r, (T - 1) // 16])
            t["k_pool"][pg, :, T % 16:, :] = float("nan")
            t["v_pool"][pg, :, T % 16:, :] = float("inf")
    full_parity(oracle_lib, b, mutate=mutate)
    full_parity(oracle_lib, b, mutate=mutate, entry="separate")
