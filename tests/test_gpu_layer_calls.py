"""Layer calls from Python: what happens around the entry points themselves."""
import ctypes
import threading

import pytest
import torch

from paper_2605_08581_amd import binding as B
from paper_2605_08581_amd import workload as W

from gpu_util import check_close, widen

pytestmark = pytest.mark.gpu


def test_other_threads_run_during_a_layer_call():
    """The entries are replaced by libc's usleep, which takes the plan as its microseconds: every call
    then lasts 0.4 s, and another Python thread has to get its turns within it (one that
    waits for the call to end gets one)."""
    lib = B.load()
    real = [ctypes.cast(f, ctypes.c_void_p).value for f in (lib.prism_kv_append, lib.prism_prefix_attention,
                                                            lib.prism_prefix_prefill, lib.prism_prefix_prefill_static)]
    fast, usleep = B._fast, ctypes.cast(ctypes.CDLL(None).usleep, ctypes.c_void_p).value
    call = fast.make_call(400000, 0, 0, 0, 0, 0)   # no elements are needed, so None will do for every tensor
    fast.bind_api(*[usleep] * 4)
    try:
        for entry, n in ((fast.kv_append, 5), (fast.prefix_attention, 6), (fast.prefix_prefill, 8),
                         (fast.prefix_prefill_static, 7)):
            turns, over = [], threading.Event()
            other = threading.Thread(target=lambda: [turns.append(1) for _ in range(1000) if not over.wait(0.005)])
            other.start()
            status = entry(call, *[None] * n)
            got = len(turns)
            over.set()
            other.join()
            assert status == 0 and got >= 5, entry.__name__
    finally:
        fast.bind_api(*real)


def test_workspace_of_wide_elements_is_refused():
    """As many bytes as the plan needs, in floats."""
    b = W.make_custom_batch("ws", W.Geometry(4, 2, 64), [32, 5], [20, 9], seed=2)
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, split_kv=2)
    t, table = W.make_tensors(b, "cuda"), torch.from_numpy(b.block_table).cuda()
    out = torch.zeros_like(t["q"])
    ws = torch.empty(-(-plan.prism_plan_workspace_bytes() // 4), dtype=torch.float32, device="cuda")
    with pytest.raises(ValueError, match="workspace"):
        plan.prism_prefix_attention(t["q"], t["k_pool"], t["v_pool"], table, out, ws)
    with pytest.raises(ValueError, match="workspace"):
        plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"], table, out, ws)
    torch.cuda.synchronize()
    assert not out.any()
    plan.close()


@pytest.mark.parametrize("suffix", [[20, 20], [150, 40]], ids=["stream", "tile"])
def test_a_table_that_is_only_a_hint_may_differ(oracle_lib, suffix):
    """On the device the second request's cached prefix is what the first one appends in this very call;
    the table that the plan was made from does not show it."""
    b = W.make_custom_batch("hint", W.Geometry(2, 2, 128), [32, 48], suffix, seed=65)
    table = b.block_table.copy()
    table[1, :3] = table[0, :3]                    # positions 32..47 of request 0 are new tokens
    t = W.make_tensors(b, "cuda")
    host = {k: W.bf16_bits(v) for k, v in t.items()}
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table, table_is_final=False)
    ws = torch.empty(plan.prism_plan_workspace_bytes(), dtype=torch.uint8, device="cuda")
    out = torch.full_like(t["q"], float("nan"))
    plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"],
                              torch.from_numpy(table).cuda(), out, ws)
    torch.cuda.synchronize()
    plan.close()
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  table, b.prefix_len, b.suffix_len)
    ref = oracle_lib.attention(host["q"], kp, vp, table, b.prefix_len, b.suffix_len, b.softmax_scale)
    check_close(widen(W.bf16_bits(out)), ref, b.name)


@pytest.mark.parametrize("over", ["k_suffix", "v_suffix", "k_suffix, half"])
@pytest.mark.parametrize("suffix", [[3, 16], [700, 400]], ids=["stream", "tile"])
def test_out_in_the_memory_of_the_new_rows(oracle_lib, suffix, over):
    """Results are those of the append followed by attention, so out may lie where the rows to append were."""
    b = W.make_custom_batch("reuse", W.Geometry(4, 4, 64), [64, 5], suffix, seed=66)
    t = W.make_tensors(b, "cuda")
    host = {k: W.bf16_bits(v) for k, v in t.items()}
    rows, half = t[over.split(",")[0]], t["q"].numel() // 2
    buf = torch.empty(2 * rows.numel(), dtype=rows.dtype, device="cuda")
    mine = buf[:rows.numel()].view(rows.shape)
    mine.copy_(rows)
    t[over.split(",")[0]] = mine
    out = buf[half:half + rows.numel()].view(t["q"].shape) if "half" in over else mine.view(t["q"].shape)
    plan = B.Plan(B.shape_of(b), b.prefix_len, b.suffix_len, block_table=b.block_table)
    ws = torch.empty(plan.prism_plan_workspace_bytes(), dtype=torch.uint8, device="cuda")
    plan.prism_prefix_prefill(t["q"], t["k_suffix"], t["v_suffix"], t["k_pool"], t["v_pool"],
                              torch.from_numpy(b.block_table).cuda(), out, ws)
    torch.cuda.synchronize()
    plan.close()
    kp, vp = oracle_lib.kv_append(host["k_suffix"], host["v_suffix"], host["k_pool"], host["v_pool"],
                                  b.block_table, b.prefix_len, b.suffix_len)
    assert (W.bf16_bits(t["k_pool"]) == kp).all() and (W.bf16_bits(t["v_pool"]) == vp).all()
    ref = oracle_lib.attention(host["q"], kp, vp, b.block_table, b.prefix_len, b.suffix_len, b.softmax_scale)
    check_close(widen(W.bf16_bits(out)), ref, b.name)
