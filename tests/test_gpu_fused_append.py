"""GPU parity of the append done inside the prefill attention kernel: new rows
are read from the packed arrays and written to their pages by the workgroups
that own them.  The edges are where the cached prefix ends (page, tile, ring
depth) and where row tiles and key ranges meet."""
import pytest
import torch

from paper_2605_08581_amd import workload as W

from gpu_util import full_parity

pytestmark = pytest.mark.gpu

SHAPES = [(0, 0), (64, 32), (128, 32), (256, 32)]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"{t}x{w}" for t, w in SHAPES])
@pytest.mark.parametrize("geom", [W.Geometry(2, 2, 128), W.Geometry(8, 2, 64), W.Geometry(5, 1, 128)],
                         ids=["mha128", "gqa4x64", "g5x128"])
def test_end_of_the_cached_prefix(oracle_lib, geom, shape):
    """Prefixes of none, one key, around a page, around one and several key
    tiles, and far inside the steady-state loop; suffixes long enough that a
    row tile runs that loop over new keys as well."""
    prefix = [0, 1, 15, 17, 63, 64, 65, 127, 320, 333, 700]
    suffix = [700, 333, 129, 130, 66, 128, 257, 90, 520, 400, 65]
    b = W.make_custom_batch("ends", geom, prefix, suffix, seed=71)
    full_parity(oracle_lib, b, tile_rows=shape[0], rows_per_wave=shape[1])


@pytest.mark.parametrize("geom", [W.Geometry(8, 2, 128), W.Geometry(5, 1, 64)], ids=["gqa4x128", "g5x64"])
@pytest.mark.parametrize("split_kv", [2, 5])
def test_key_ranges_share_the_append(oracle_lib, split_kv, geom):
    """Split keys: every new row is appended by exactly one workgroup per head, whichever range
    holds it, and the last workgroup of each group merges up to 128 rows."""
    b = W.make_custom_batch("ranges", geom, [0, 300, 1000, 77], [300, 150, 70, 400], seed=72)
    info = full_parity(oracle_lib, b, split_kv=split_kv)
    assert info.num_reduce_groups > 0


@pytest.mark.parametrize("moved", [["q"], ["k_suffix"], ["v_suffix"], ["q", "k_suffix", "v_suffix"]], ids="-".join)
@pytest.mark.parametrize("suffix", [[3, 1, 16], [40, 130, 7]], ids=["few-rows", "tiles"])
def test_rows_off_the_16_byte_grid(oracle_lib, suffix, moved):
    """Contiguous inputs that start 8 bytes past a 16-byte boundary: views into a larger buffer."""
    def mutate(t):
        for name in moved:
            x = t[name]
            buf = torch.empty(x.numel() + 4, dtype=x.dtype, device=x.device)
            t[name] = buf[4:].view(x.shape)
            t[name].copy_(x)
            assert t[name].is_contiguous() and t[name].data_ptr() % 16 == 8
    full_parity(oracle_lib, W.make_custom_batch("views", W.Geometry(4, 2, 128), [0, 37, 500], suffix, seed=73),
                mutate=mutate)


@pytest.mark.parametrize("elements", [1, 4])
@pytest.mark.parametrize("tile_rows", [64, 128, 256])
@pytest.mark.parametrize("geom", [W.Geometry(4, 2, 128), W.Geometry(3, 1, 128), W.Geometry(2, 2, 64)], ids=["g2x128", "g3x128", "mha64"])
@pytest.mark.parametrize("copies", [1, 70], ids=["alone", "shared"])
def test_query_rows_off_the_16_byte_grid(oracle_lib, geom, tile_rows, elements, copies):
    """The row tiles' kernel takes query rows from any address: blocks of 32 that end after 1, 31, 32 and 33 rows,
    with one workgroup to a compute unit and more."""
    def mutate(t):
        buf = torch.empty(t["q"].numel() + 8, dtype=t["q"].dtype, device=t["q"].device)
        q = buf[elements:elements + t["q"].numel()].view(t["q"].shape)
        t["q"] = q.copy_(t["q"])
    b = W.make_custom_batch("q-views", geom, [0, 37, 500, 16] * copies, [11, 31, 32, 97] * copies, seed=74)
    full_parity(oracle_lib, b, mutate=mutate, tile_rows=tile_rows)
