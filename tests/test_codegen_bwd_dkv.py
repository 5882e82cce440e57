"""Generated code of ksa_prefill_bwd_dkv.hip (no GPU needed): the kernel's registers are counted out, and a spill inside its tile
loop would wait for every tile in flight; its counted waits hold only while nothing but its own tile loads counts as vector
memory inside it; and no packed fp32 VALU instruction (see test_codegen.py)."""
import os
import re
import tempfile

import pytest

from paper_2604_24432_amd import build as B
from tests.test_codegen import _assembly, _is_plain_vector_memory, _kernels

SOURCE = "ksa_prefill_bwd_dkv.hip"


@pytest.fixture(scope="module")
def text():
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    with tempfile.TemporaryDirectory() as d:
        return _assembly(SOURCE, d)


def _dkv_kernels(text):
    kernels = {n: b for n, b in _kernels(text).items() if "ksa_bwd_dkv_direct_kernel" in n}
    assert len(kernels) == 2
    return kernels


def test_tile_loop_does_not_spill(text):
    for name, blocks in _dkv_kernels(text).items():
        ins = [i for block in blocks.values() for i in block]
        assert sum("v_mfma" in i for i in ins) >= 16 and any(i.startswith("global_load_lds_dwordx4") for i in ins), name
        assert not [i for i in ins if i.startswith("scratch_")], name
    assert not re.findall(r"\bv_pk_(?:add|mul|fma)_f32\b", text)


def test_tile_loop_holds_only_its_own_tile_loads(text):
    """Every block that the tile loop can run through, also those off the MFMA stream (the next block's rows worked out, the mask
    of a clipped tile), holds no vector memory instruction but the tile loads."""
    for name, blocks in _dkv_kernels(text).items():
        loop = _loop_blocks(blocks)
        assert sum("v_mfma" in i for label in loop for i in blocks[label]) >= 16, name
        assert any(i.startswith("global_load_lds_dwordx4") for label in loop for i in blocks[label]), name
        foreign = {label: [i for i in blocks[label] if _is_plain_vector_memory(i)] for label in loop}
        assert not any(foreign.values()), (name, {k: v for k, v in foreign.items() if v})


def _loop_blocks(blocks):
    """Labels of the blocks on a cycle of the control flow graph that an MFMA stands in."""
    labels = list(blocks)
    after = {}
    for x, label in enumerate(labels):
        nxt, falls = set(), True
        for i in blocks[label]:
            op, *rest = i.split()
            if op.startswith(("s_cbranch", "s_branch")) and rest[0] in blocks:
                nxt.add(rest[0])
            falls = op not in ("s_branch", "s_endpgm", "s_setpc_b64")
        if falls and x + 1 < len(labels):
            nxt.add(labels[x + 1])
        after[label] = nxt

    def reach(start, edges):
        seen, todo = set(), [start]
        while todo:
            for y in edges[todo.pop()]:
                if y not in seen:
                    seen.add(y), todo.append(y)
        return seen
    before = {label: {x for x in labels if label in after[x]} for label in labels}
    loop = set()
    for label in labels:
        if any("v_mfma" in i for i in blocks[label]):
            loop |= reach(label, after) & reach(label, before)
    return loop
