"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2605_08581_amd import binding as B
from paper_2605_08581_amd import workload as W

from gpu_util import check_close, full_parity, run_hip, widen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.load()


def test_tiny_config_all_rows(oracle_lib):
    full_parity(oracle_lib, W.make_config(0))


# (tile_rows, rows_per_wave): every kernel shape the planner can pick
SHAPES = [(64, 32), (128, 32), (256, 32), (128, 64), (256, 64)]
SHAPE_IDS = [f"{t}x{w}" for t, w in SHAPES]


@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
@pytest.mark.parametrize("geom", [W.Geometry(4, 4, 64), W.Geometry(8, 2, 128), W.Geometry(6, 6, 128),
                                   W.Geometry(8, 1, 64)], ids=["mha64", "gqa4x128", "mha128", "mqa8x64"])
def test_ragged_lengths_all_rows(oracle_lib, geom, shape):
    """Prefixes and suffixes that end inside pages and tiles, an empty request,
    a request with no cached prefix, and a single-token one."""
    prefix = [0, 16, 37, 200, 64, 129, 0]
    suffix = [70, 0, 19, 33, 130, 65, 1]
    b = W.make_custom_batch("ragged", geom, prefix, suffix, seed=5, share_groups=[-1, 0, -1, 0, 0, -1, -1])
    full_parity(oracle_lib, b, tile_rows=shape[0], rows_per_wave=shape[1])


@pytest.mark.parametrize("shape", SHAPES, ids=SHAPE_IDS)
@pytest.mark.parametrize("geom", [W.Geometry(2, 2, 128), W.Geometry(8, 2, 128), W.Geometry(4, 4, 64)],
                         ids=["mha128", "gqa4x128", "mha64"])
def test_long_prefixes_run_the_steady_state_loop(oracle_lib, geom, shape):
    """Cached prefixes of 1 000 to 2 600 tokens: dozens of unmasked key tiles
    before the causal diagonal, so the unrolled steady-state loop of every
    kernel shape (ring slots fixed in the code, copies interleaved with the
    math) runs several trips, then hands over to the masked tail.  Ragged
    suffixes leave some waves of a workgroup without rows."""
    prefix = [1024, 2600, 1500, 1040]
    suffix = [300, 40, 129, 64]
    b = W.make_custom_batch("steady", geom, prefix, suffix, seed=15, share_groups=[0, -1, 0, -1])
    full_parity(oracle_lib, b, tile_rows=shape[0], rows_per_wave=shape[1])


@pytest.mark.parametrize("tile_rows", [64, 128, 256])
@pytest.mark.parametrize("geom", [W.Geometry(2, 2, 128), W.Geometry(3, 1, 64)], ids=["mha128", "gqa3x64"])
def test_tiles_around_the_diagonal(oracle_lib, geom, tile_rows):
    """Odd and even numbers of key tiles before, at and after the end of the cached
    prefix, and last tiles of which a wave's rows see 1, 31, 32 and 33 keys or all."""
    lengths = [(0, 31), (0, 33), (0, 64), (16, 17), (48, 81), (64, 128), (96, 65), (128, 1), (128, 32), (160, 97),
               (191, 130), (192, 192), (250, 70), (257, 255), (320, 160), (400, 321)]
    b = W.make_custom_batch("diagonal", geom, [p for p, _ in lengths], [s for _, s in lengths], seed=16)
    full_parity(oracle_lib, b, tile_rows=tile_rows)
    full_parity(oracle_lib, b, tile_rows=tile_rows, entry="separate")


@pytest.mark.parametrize("tile_rows", [64, 128, 256])
@pytest.mark.parametrize("geom", [W.Geometry(3, 1, 128), W.Geometry(2, 2, 64)], ids=["g3x128", "mha64"])
@pytest.mark.parametrize("split_kv", [1, 3])
@pytest.mark.parametrize("copies", [1, 70], ids=["alone", "shared"])
def test_out_anywhere_in_a_larger_buffer(geom, tile_rows, split_kv, copies):
    """Rows are stored whole, or by pieces where a wave has few or its workgroup a compute unit to itself,
    wherever out starts; nothing beside it is touched, and the values do not depend on it: blocks that end after 1, 31,
    32 and 33 rows, with one workgroup to a compute unit and more."""
    b = W.make_custom_batch("out", geom, [0, 70, 300, 16] * copies, [11, 31, 32, 97] * copies, seed=17)
    t = W.make_tensors(b, "cuda")
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table, tile_rows=tile_rows, split_kv=split_kv)
    ws = torch.empty(max(256, plan.prism_plan_workspace_bytes()), dtype=torch.uint8, device="cuda")
    bt = torch.from_numpy(b.block_table).cuda()
    n, results = t["q"].numel(), []
    for start in (0, 4, 1):
        buf = torch.full((n + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
        plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], bt,
                                  buf[start:start + n].view(t["q"].shape), ws)
        torch.cuda.synchronize()
        assert bool((buf[:start] == 7.0).all()) and bool((buf[start + n:] == 7.0).all())
        results.append(W.bf16_bits(buf[start:start + n]))
    plan.close()
    assert np.array_equal(results[0], results[1]) and np.array_equal(results[0], results[2])


def test_rows_of_a_wave_over_four_gigabytes():
    """Token rows of 140 MB: the 32 query rows of one wave lie over more bytes than 32 bits count."""
    heads, S, d = 550_000, 33, 128
    b = W.make_custom_batch("wide", W.Geometry(heads, heads, d), [0], [S], seed=18)
    gen = torch.Generator(device="cuda").manual_seed(18)
    normal = lambda *n: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, k, v = (normal(S, heads, d) for _ in range(3))
    pools = [torch.zeros(b.num_pages, heads, W.PAGE_SIZE, d, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table)
    assert plan.prism_plan_get_info().tile_rows == 128 and 31 * heads * d * 2 > 2 ** 32
    ws = torch.empty(max(256, plan.prism_plan_workspace_bytes()), dtype=torch.uint8, device="cuda")
    out = torch.full_like(q, float("nan"))
    plan.prism_prefix_prefill(q, k, v, *pools, torch.from_numpy(b.block_table).cuda(), out, ws)
    torch.cuda.synchronize()
    plan.close()
    some = torch.cat([torch.tensor([0, 1, heads // 2, heads - 1]), torch.arange(7, heads, 9973)]).cuda()
    x, y, z = (t[:, some].transpose(0, 1).float().contiguous() for t in (q, k, v))
    scores = (x @ y.transpose(1, 2).contiguous()) * b.softmax_scale
    scores.masked_fill_(torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    check_close(out[:, some].transpose(0, 1).double().cpu().numpy(), (scores.softmax(-1) @ z).double().cpu().numpy(), "wide")
    pages = torch.from_numpy(b.block_table[0, :3].astype(np.int64)).cuda()
    for pool, new in zip(pools, (k, v)):
        rows = pool[:, some].index_select(0, pages).permute(0, 2, 1, 3).reshape(-1, len(some), d)
        assert torch.equal(rows[:S], new[:, some]) and not rows[S:].any()


@pytest.mark.parametrize("shape", [(128, 32), (128, 64), (256, 64)], ids=["128x32", "128x64", "256x64"])
@pytest.mark.parametrize("split_kv", [2, 3, 7])
def test_split_kv_matches_oracle(oracle_lib, split_kv, shape):
    b = W.make_custom_batch("split", W.Geometry(8, 2, 128), [500, 0, 1000, 77], [40, 300, 7, 150], seed=6)
    info = full_parity(oracle_lib, b, split_kv=split_kv, tile_rows=shape[0], rows_per_wave=shape[1])
    assert info.num_reduce_groups > 0


@pytest.mark.parametrize("requests", [3, 48, 49], ids=["small", "few", "many"])
@pytest.mark.parametrize("split_kv", [4, 5, 8, 9, 17])
@pytest.mark.parametrize("geom", [W.Geometry(6, 2, 128), W.Geometry(4, 4, 64)], ids=["gqa3x128", "mha64"])
def test_merge_of_few_and_of_many_rows(oracle_lib, geom, split_kv, requests):
    """Up to 768 workgroups at one row per thread (48 requests of one tile) a merge
    reads up to four, eight or sixteen partials at once, beyond them four: below, at
    and above those numbers."""
    prefix = [64 * split_kv - 60 + r % 30 for r in range(requests)]      # one key tile a piece
    b = W.make_custom_batch("merge", geom, prefix, [11 + r % 10 for r in range(requests)], seed=17)
    info = full_parity(oracle_lib, b, split_kv=split_kv, tile_rows=64)
    assert info.num_reduce_groups == requests * geom.num_kv_heads
    assert info.num_split_items == split_kv * info.num_reduce_groups


def test_split_and_unsplit_agree():
    b = W.make_custom_batch("split", W.Geometry(4, 4, 128), [900, 130], [100, 260], seed=7)
    t = W.make_tensors(b, "cuda")
    a, _ = run_hip(b, {k: v.clone() for k, v in t.items()}, split_kv=1)
    c, info = run_hip(b, {k: v.clone() for k, v in t.items()}, split_kv=4)
    assert info.num_split_items > 0
    # both are bf16 roundings of fp32 results that differ only in summation
    # order: at most one bf16 ulp (2^-7 relative at the top binade) apart
    dmax = float((a.double() - c.double()).abs().max())
    amax = float(a.double().abs().max())
    assert dmax <= 2.0 ** -7 * amax, (dmax, amax)


@pytest.mark.parametrize("shape", [(128, 32), (128, 64), (256, 64)], ids=["128x32", "128x64", "256x64"])
@pytest.mark.parametrize("scale,name", [(1.0, "unit"), (4.0, "sharp")])
def test_unscaled_and_sharp_inputs(oracle_lib, scale, name, shape):
    """q,k,v ~ N(0,1) (logits of order 1, outputs of order 0.1-1, so the
    absolute tolerance bites) and q,k ~ 4 N(0,1) (logit std 16: the max
    subtraction matters)."""
    geom = W.Geometry(4, 2, 128)
    b = W.make_custom_batch(name, geom, [96, 0, 333], [100, 257, 31], seed=8, value_scale=1.0)

    def mutate(t):
        for k in ("q", "k_suffix", "k_pool"):
            t[k].mul_(scale)
    full_parity(oracle_lib, b, mutate=mutate, tile_rows=shape[0], rows_per_wave=shape[1])


@pytest.mark.parametrize("shape", [(128, 32), (128, 64), (256, 64)], ids=["128x32", "128x64", "256x64"])
def test_slots_past_the_sequence_are_ignored(oracle_lib, shape):
    """The last page's unused slots (and unrelated pages) hold NaN/Inf bit
    patterns; results must not change."""
    geom = W.Geometry(4, 4, 128)
    b = W.make_custom_batch("nan", geom, [32, 0], [21, 70], seed=9)

    def mutate(t):
        for r in range(b.batch):
            T = int(b.prefix_len[r] + b.suffix_len[r])
            pg = int(b.block_table[r, (T - 1) // 16])
            if T % 16:
                t["k_pool"][pg, :, T % 16:, :] = float("nan")
                t["v_pool"][pg, :, T % 16:, :] = float("inf")
    full_parity(oracle_lib, b, mutate=mutate, tile_rows=shape[0], rows_per_wave=shape[1])


@pytest.mark.parametrize("seed", range(16))
def test_random_small_waves(oracle_lib, seed):
    """Seeded random waves: head grouping, head dim, lengths (empty requests,
    no prefix, single tokens, lengths around the tile and page edges), page
    sharing, kernel shape and split policy all drawn at random; every row
    against the oracle, both pools against the page-table writer."""
    rng = np.random.default_rng(7000 + seed)
    hkv = int(rng.choice([1, 2, 3, 4]))
    geom = W.Geometry(hkv * int(rng.choice([1, 2, 4, 5])), hkv, int(rng.choice([64, 128])))
    n = int(rng.integers(1, 7))
    prefix = [int(rng.choice([0, 16, 37, 64, 129, 500, 1300])) for _ in range(n)]
    suffix = [int(rng.choice([0, 1, 2, 31, 33, 64, 65, 127, 130, 260])) for _ in range(n)]
    if sum(suffix) == 0:
        suffix[0] = 7
    groups = [int(rng.choice([-1, 0, 1])) for _ in range(n)]
    b = W.make_custom_batch("rnd", geom, prefix, suffix, seed=seed, share_groups=groups)
    shape = SHAPES[int(rng.integers(0, len(SHAPES)))]
    split_kv = int(rng.choice([0, 1, 3]))
    full_parity(oracle_lib, b, seed=seed, tile_rows=shape[0], rows_per_wave=shape[1], split_kv=split_kv)


def test_page_permutation_invariance():
    geom = W.Geometry(8, 2, 128)
    b = W.make_custom_batch("perm", geom, [128, 64], [50, 90], seed=10, permute_pages=False)
    t = W.make_tensors(b, "cuda")
    ref, _ = run_hip(b, {k: v.clone() for k, v in t.items()})
    perm = np.random.default_rng(3).permutation(b.num_pages)
    inv = torch.from_numpy(np.argsort(perm)).cuda()
    b2 = W.Batch(**{**b.__dict__, "block_table": perm[b.block_table].astype(np.int32)})
    t2 = {k: v.clone() for k, v in t.items()}
    t2["k_pool"], t2["v_pool"] = t["k_pool"][inv].contiguous(), t["v_pool"][inv].contiguous()
    got, _ = run_hip(b2, t2)
    assert torch.equal(got, ref)


def test_append_entry_point_alone_is_bit_exact(oracle_lib):
    b = W.make_custom_batch("append", W.Geometry(40, 40, 128), [16, 5, 0, 48], [33, 12, 100, 1], seed=11,
                            share_groups=[0, -1, -1, 0])
    t = W.make_tensors(b, "cuda")
    host = {k: W.bf16_bits(v) for k, v in t.items()}
    sh = B.shape_of(b)
    plan = B.Plan(sh, b.prefix_len, b.suffix_len)
    bt = torch.from_numpy(b.block_table).cuda()
    plan.prism_kv_append(t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], bt)
    torch.cuda.synchronize()
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  b.block_table, b.prefix_len, b.suffix_len)
    assert np.array_equal(W.bf16_bits(t["k_pool"]), kp) and np.array_equal(W.bf16_bits(t["v_pool"]), vp)


def test_separate_entry_points_match_fused_call(oracle_lib):
    b = W.make_custom_batch("sep", W.Geometry(8, 2, 128), [64, 0], [40, 129], seed=12)
    full_parity(oracle_lib, b, entry="separate")


def test_workspace_errors():
    b = W.make_custom_batch("ws", W.Geometry(4, 4, 128), [900], [100], seed=13)
    t = W.make_tensors(b, "cuda")
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, split_kv=4)
    need = plan.prism_plan_workspace_bytes()
    assert need > 0
    bt = torch.from_numpy(b.block_table).cuda()
    out = torch.empty_like(t["q"])
    small = torch.empty(need - 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(B.PrismError) as e:
        plan.prism_prefix_attention(t["q"], t["k_pool"], t["v_pool"], bt, out, small)
    assert e.value.code == B.ERR_WORKSPACE_TOO_SMALL
    with pytest.raises(B.PrismError) as e:
        plan.prism_prefix_attention(t["q"], t["k_pool"], t["v_pool"], bt, out, None)
    assert e.value.code == B.ERR_INVALID_ARG
    plan.close()


def _sampled_parity(oracle_lib, b, n_rows, **opts):
    """Full-size check: the pools against the oracle's page-table writer over
    every byte of both pools (which also shows that nothing else was written),
    attention on sampled rows (every request's first and last rows and the rows
    next to page and tile boundaries, plus uniform picks; every row with three
    query heads, so that all heads of a wave are drawn many times over)."""
    t = W.make_tensors(b, "cuda")
    host = {k: W.bf16_bits(t[k]) for k in ("k_suffix", "v_suffix", "k_pool", "v_pool")}
    out, info = run_hip(b, t, **opts)
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  b.block_table, b.prefix_len, b.suffix_len)
    del host
    got_k, got_v = W.bf16_bits(t["k_pool"]), W.bf16_bits(t["v_pool"])
    assert np.array_equal(got_k, kp), "K pool differs from the page-table writer"
    assert np.array_equal(got_v, vp), "V pool differs from the page-table writer"
    del got_k, got_v
    base = W.sample_rows(b, n_rows, seed=1)
    rng = np.random.default_rng(2)
    Hq = b.geom.num_q_heads
    rows = np.concatenate([base] + [np.stack([base[:, 0], base[:, 1], rng.integers(0, Hq, len(base))], axis=1)
                                    for _ in range(2)]).astype(np.int32)
    ref = oracle_lib.attention_rows(W.bf16_bits(t["q"]), kp, vp, b.block_table, b.prefix_len, b.suffix_len,
                                    b.softmax_scale, rows)
    offs = b.suffix_offsets
    got = widen(W.bf16_bits(out[torch.from_numpy(offs[rows[:, 0]] + rows[:, 1]).cuda(),
                                torch.from_numpy(rows[:, 2].astype(np.int64)).cuda()]))
    check_close(got, ref, b.name)
    assert torch.isfinite(out.float()).all()
    return info


@pytest.mark.parametrize("index", [1, 2, 4])
def test_full_size_configs_sampled_rows(oracle_lib, index):
    """The benchmark configurations at full size with the default plan (the
    launch configuration the benchmark times)."""
    _sampled_parity(oracle_lib, W.make_config(index), 1500)


@pytest.mark.parametrize("shape", [(256, 32), (128, 64), (256, 64)], ids=["256x32", "128x64", "256x64"])
def test_other_kernel_shapes_at_full_size(oracle_lib, shape):
    """The 13B-class wave at full size through the kernel shapes that are not the default."""
    _sampled_parity(oracle_lib, W.make_config(2), 600, tile_rows=shape[0], rows_per_wave=shape[1])


@pytest.mark.parametrize("hit", [0.0, 0.5, 0.9])
def test_hit_rate_sweep_sampled_rows(oracle_lib, hit):
    """The hit-rate sweep at its full size: 32 requests of the 13B-class geometry."""
    b = W.make_hit_rate_batch(hit)
    assert b.batch == 32
    _sampled_parity(oracle_lib, b, 800)


def test_chunked_prefill_equals_one_shot(oracle_lib):
    """Chunked prefill (the engine the paper builds on keeps it, Sec. 4.1): the
    suffix is fed in fixed-size chunks, each chunk attending to the prefix, to
    the chunks already appended, and to itself.  Chunk boundaries fall inside
    pages, so later chunks see a partial private page as part of their prefix.
    Pools must end bit-identical and outputs within tolerance of the oracle's
    one-shot result."""
    geom = W.Geometry(8, 2, 128)
    b = W.make_custom_batch("chunked", geom, [48, 0, 200], [150, 333, 90], seed=21)
    t = W.make_tensors(b, "cuda")
    host = {k: W.bf16_bits(v) for k, v in t.items()}
    one_shot, _ = run_hip(b, {k: v.clone() for k, v in t.items()})
    chunk = 56                                   # not a multiple of the page size
    offs = b.suffix_offsets
    out = torch.full_like(t["q"], float("nan"))
    bt = torch.from_numpy(b.block_table).cuda()
    done = np.zeros(b.batch, dtype=np.int64)
    while (done < b.suffix_len).any():
        S = np.minimum(chunk, b.suffix_len - done).astype(np.int32)
        P = (b.prefix_len + done).astype(np.int32)
        rows = np.concatenate([np.arange(offs[r] + done[r], offs[r] + done[r] + S[r]) for r in range(b.batch)])
        idx = torch.from_numpy(rows).cuda()
        plan = B.Plan(B.shape_of(b), P, S, block_table=b.block_table)
        n = plan.prism_plan_workspace_bytes()
        ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
        o = torch.empty((len(rows),) + tuple(t["q"].shape[1:]), dtype=t["q"].dtype, device="cuda")
        plan.prism_prefix_prefill(t["q"][idx].contiguous(), t["k_suffix"][idx].contiguous(),
                                  t["v_suffix"][idx].contiguous(), t["k_pool"], t["v_pool"], bt, o, ws)
        torch.cuda.synchronize()
        plan.close()
        out[idx] = o
        done += S
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  b.block_table, b.prefix_len, b.suffix_len)
    assert np.array_equal(W.bf16_bits(t["k_pool"]), kp) and np.array_equal(W.bf16_bits(t["v_pool"]), vp)
    ref = oracle_lib.attention(host["q"], kp, vp, b.block_table, b.prefix_len, b.suffix_len, b.softmax_scale)
    check_close(widen(W.bf16_bits(out)), ref, "chunked")
    dmax = float((out.double() - one_shot.double()).abs().max())
    assert dmax <= 2.0 ** -7 * float(one_shot.double().abs().max())


@pytest.mark.parametrize("geom", [W.Geometry(40, 40, 128), W.Geometry(32, 8, 128)], ids=["mha", "gqa"])
def test_single_token_suffix_decode_shape(oracle_lib, geom):
    """One uncached token per request over a long cached prefix (the first
    decode step after prefill, the T_1tok term of Eq. 2)."""
    b = W.make_custom_batch("decode", geom, [1000, 37, 4096, 16], [1, 1, 1, 1], seed=22)
    full_parity(oracle_lib, b)
    full_parity(oracle_lib, b, split_kv=4)


def test_measured_peaks_are_plausible():
    """The measurement aid reports machine ceilings below the published peaks
    (2.5 PFLOP/s bf16 MFMA, 8 TB/s HBM) and well above zero."""
    scratch = torch.ones(2**28, dtype=torch.uint8, device="cuda")
    mfma, read = B.prism_measure_peaks(scratch, repeats=2)
    assert 500.0 < mfma < 2500.0 * 1.02, mfma
    assert 1000.0 < read < 8000.0 * 1.02, read
    assert bool((scratch == 1).all()), "the scratch buffer is only read"


def test_pages_beyond_the_4_gib_offset(oracle_lib):
    """Byte offsets into the pools exceed 32 bits: a 4.6 GB pool whose used
    pages sit at its far end (and its very start).  The oracle sees the same
    pages compacted into a small pool."""
    geom = W.Geometry(8, 8, 128)
    small = W.make_custom_batch("far-pages", geom, [160, 47], [40, 70], seed=3)
    used = sorted(set(int(p) for r in range(small.batch)
                      for p in small.block_table[r, :(small.prefix_len[r] + small.suffix_len[r] + 15) // 16]))
    num_pages = 140_000                                      # x 8 heads x 16 x 128 x 2 B = 4.59 GB per pool
    far = {p: (num_pages - 1 - 977 * i if i % 2 == 0 else 3 * i) for i, p in enumerate(used)}
    assert max(far.values()) * 8 * 16 * 128 * 2 > 2**32 and len(set(far.values())) == len(far)
    t = W.make_tensors(small, "cuda")
    big = {k: torch.zeros(num_pages, 8, 16, 128, dtype=torch.bfloat16, device="cuda") for k in ("k_pool", "v_pool")}
    for p, q_ in far.items():
        big["k_pool"][q_] = t["k_pool"][p]
        big["v_pool"][q_] = t["v_pool"][p]
    table = small.block_table.copy()
    for p, q_ in far.items():
        table[small.block_table == p] = q_
    shape = B.make_shape(8, 8, 128, num_pages, small.batch, small.max_blocks, small.softmax_scale)
    plan = B.Plan(shape, small.prefix_len, small.suffix_len, block_table=table)
    bt = torch.from_numpy(table).cuda()
    out = torch.full_like(t["q"], float("nan"))
    ws = torch.empty(plan.prism_plan_workspace_bytes(), dtype=torch.uint8, device="cuda")
    plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], big["k_pool"], big["v_pool"], bt, out, ws)
    torch.cuda.synchronize()
    plan.close()
    host = {k: W.bf16_bits(v) for k, v in t.items()}
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  small.block_table, small.prefix_len, small.suffix_len)
    for p, q_ in far.items():                                # the appended pages, bit for bit, where they belong
        assert np.array_equal(W.bf16_bits(big["k_pool"][q_]), kp[p])
        assert np.array_equal(W.bf16_bits(big["v_pool"][q_]), vp[p])
    untouched = torch.ones(num_pages, dtype=torch.bool, device="cuda")
    untouched[torch.tensor(sorted(far.values()), device="cuda")] = False
    assert not bool(big["k_pool"][untouched].any()) and not bool(big["v_pool"][untouched].any())
    ref = oracle_lib.attention(host["q"], kp, vp, small.block_table, small.prefix_len, small.suffix_len,
                               small.softmax_scale)
    check_close(widen(W.bf16_bits(out)), ref, "far pages")


def test_two_plans_on_two_streams(oracle_lib):
    """Calls on distinct plans are independent: two waves enqueued on two
    streams of default priority, overlapping in time, both match the oracle."""
    waves = [W.make_custom_batch("stream-a", W.Geometry(8, 2, 128), [1000, 37, 512], [90, 200, 33], seed=21),
             W.make_custom_batch("stream-b", W.Geometry(4, 4, 64), [300, 2000], [129, 64], seed=22)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    state = []
    for b, st in zip(waves, streams):
        t = W.make_tensors(b, "cuda")
        host = {k: W.bf16_bits(v) for k, v in t.items()}
        plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table, split_kv=2)
        bt = torch.from_numpy(b.block_table).cuda()
        out = torch.full_like(t["q"], float("nan"))
        ws = torch.empty(max(plan.prism_plan_workspace_bytes(), 256), dtype=torch.uint8, device="cuda")
        state.append((b, t, host, plan, bt, out, ws, st))
    torch.cuda.synchronize()
    for rep in range(3):                                     # several launches in flight on each stream
        for b, t, host, plan, bt, out, ws, st in state:
            with torch.cuda.stream(st):
                plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], bt, out, ws)
    torch.cuda.synchronize()
    for b, t, host, plan, bt, out, ws, st in state:
        plan.close()
        kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                      b.block_table, b.prefix_len, b.suffix_len)
        assert np.array_equal(W.bf16_bits(t["k_pool"]), kp) and np.array_equal(W.bf16_bits(t["v_pool"]), vp)
        ref = oracle_lib.attention(host["q"], kp, vp, b.block_table, b.prefix_len, b.suffix_len, b.softmax_scale)
        check_close(widen(W.bf16_bits(out)), ref, b.name)


def test_prefill_call_replays_from_a_hip_graph():
    """The layer call enqueues kernels only (no allocation, no memset, no
    synchronisation), so it can be captured once and replayed: every replay,
    with eager work in between, reproduces the eager result bit for bit."""
    b = W.make_custom_batch("graph", W.Geometry(8, 2, 128), [700, 64, 2300], [150, 80, 20], seed=31)
    t = W.make_tensors(b, "cuda")
    pools0 = (t["k_pool"].clone(), t["v_pool"].clone())
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table, split_kv=3)
    bt = torch.from_numpy(b.block_table).cuda()
    ws = torch.empty(max(plan.prism_plan_workspace_bytes(), 256), dtype=torch.uint8, device="cuda")
    eager = torch.full_like(t["q"], float("nan"))
    plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], bt, eager, ws)
    torch.cuda.synchronize()
    pools_eager = (t["k_pool"].clone(), t["v_pool"].clone())
    out = torch.full_like(t["q"], float("nan"))
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        t["k_pool"].copy_(pools0[0]); t["v_pool"].copy_(pools0[1])
        side.synchronize()
        graph.capture_begin()
        plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], bt, out, ws)
        graph.capture_end()
    torch.cuda.synchronize()
    for rep in range(3):
        t["k_pool"].copy_(pools0[0]); t["v_pool"].copy_(pools0[1])      # eager work between the replays
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), eager.view(torch.int16)), f"replay {rep}"
        assert torch.equal(t["k_pool"].view(torch.int16), pools_eager[0].view(torch.int16))
        assert torch.equal(t["v_pool"].view(torch.int16), pools_eager[1].view(torch.int16))
    plan.close()


def test_plan_lifetime_never_waits_for_the_device(oracle_lib):
    """Creating, using and destroying a plan waits for no other stream: a long
    run of GEMMs on a side stream is still going after a whole plan lifetime on
    the main stream (the library allocates no device memory, copies its work
    lists asynchronously on the caller's stream, and destroy waits for that
    copy only - not for the kernels it enqueued, which need nothing of the
    plan's any more)."""
    b = W.make_custom_batch("nosync", W.Geometry(8, 2, 128), [300, 64], [70, 33], seed=41)
    t = W.make_tensors(b, "cuda")
    host = {k: W.bf16_bits(v) for k, v in t.items()}
    bt = torch.from_numpy(b.block_table).cuda()
    out = torch.full_like(t["q"], float("nan"))
    # a first lifetime loads the kernels, so that the timed one below is short
    warm = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table, split_kv=2)
    ws = torch.empty(warm.prism_plan_workspace_bytes(), dtype=torch.uint8, device="cuda")
    pools = (t["k_pool"].clone(), t["v_pool"].clone())
    warm.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], pools[0], pools[1], bt, out, ws)
    torch.cuda.synchronize()
    warm.close()
    side = torch.cuda.Stream()
    done = torch.cuda.Event()
    a = torch.randn(8192, 8192, device="cuda")
    c = torch.empty_like(a)
    torch.mm(a, a, out=c)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(40):                                  # a few hundred milliseconds of fp32 GEMMs
            torch.mm(a, a, out=c)
        done.record()
    assert not done.query(), "the side work is too short for this test"
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table, split_kv=2)
    assert not done.query(), "prism_plan_create waited for the side stream"
    plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], bt, out, ws)
    assert not done.query(), "prism_prefix_prefill waited for the side stream"
    plan.close()                                             # with its kernels possibly still queued
    assert not done.query(), "prism_plan_destroy waited for the side stream"
    torch.cuda.synchronize()
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  b.block_table, b.prefix_len, b.suffix_len)
    assert np.array_equal(W.bf16_bits(t["k_pool"]), kp) and np.array_equal(W.bf16_bits(t["v_pool"]), vp)
    ref = oracle_lib.attention(host["q"], kp, vp, b.block_table, b.prefix_len, b.suffix_len, b.softmax_scale)
    check_close(widen(W.bf16_bits(out)), ref, "nosync")


def test_work_lists_follow_the_workspace():
    """The work lists live in the caller's workspace: alternating between two
    workspaces, reusing one after it was overwritten (with
    prism_plan_forget_workspace), and a workspace at an offset inside a larger
    buffer all give the same bits."""
    b = W.make_custom_batch("lists", W.Geometry(8, 2, 128), [700, 64, 130], [150, 80, 20], seed=42)
    t = W.make_tensors(b, "cuda")
    bt = torch.from_numpy(b.block_table).cuda()
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table, split_kv=3)
    n = plan.prism_plan_workspace_bytes()
    big = torch.empty(2 * n + 4096, dtype=torch.uint8, device="cuda")
    ws_a, ws_b = big[:n], big[(n + 255) // 256 * 256 + 256:][:n]
    outs = []
    for ws in (ws_a, ws_b, ws_a, ws_b):
        o = torch.full_like(t["q"], float("nan"))
        plan.prism_prefix_attention(t["q"], t["k_pool"], t["v_pool"], bt, o, ws)
        outs.append(o)
    torch.cuda.synchronize()
    ws_b.fill_(0)                                            # the caller reuses the memory ...
    plan.prism_plan_forget_workspace()                       # ... and says so
    o = torch.full_like(t["q"], float("nan"))
    plan.prism_prefix_attention(t["q"], t["k_pool"], t["v_pool"], bt, o, ws_b)
    outs.append(o)
    torch.cuda.synchronize()
    plan.close()
    for o in outs[1:]:
        assert torch.equal(o.view(torch.int16), outs[0].view(torch.int16))
    assert torch.isfinite(outs[0].float()).all()
