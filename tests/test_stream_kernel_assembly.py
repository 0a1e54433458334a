"""What the compiler generated around the inline assembly of the key-splitting
kernel: M0 belongs to the direct-to-LDS copies, nothing spills, and no load into
registers is written in inline assembly (the compiler takes such registers as
written at once, while the load is still in flight)."""
import re

import pytest

from paper_2605_08581_amd import build
from test_kernel_assembly import _instructions


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    return open(build.emit_assembly("prism_stream.hip", str(tmp_path_factory.mktemp("asm")))).read().splitlines()


def test_inline_assembly_of_the_key_splitting_kernel(lines):
    copies = 0
    for kernel, inline, ins in _instructions(lines):
        assert not ins.startswith("scratch_") and not re.match(r"v_pk_(add|mul|fma)_f32\b", ins), f"{kernel}: {ins}"
        if re.search(r"\bm0\b", ins):
            assert inline and ins.startswith("s_mov_b32 m0,"), f"{kernel}: {ins}"
        if inline and re.match(r"(global|buffer|flat|scratch|ds)_(load|read)", ins):
            assert ins.startswith("buffer_load_dwordx4") and ins.endswith("lds"), f"{kernel}: {ins}"
            copies += 1
    assert copies > 0
