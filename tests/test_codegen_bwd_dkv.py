"""Generated code of ksa_prefill_bwd_dkv.hip (no GPU needed): the kernel's registers are counted out, and a spill inside its tile
loop would wait for every tile in flight; and no packed fp32 VALU instruction (see test_codegen.py)."""
import os
import re
import tempfile

import pytest

from paper_2604_24432_amd import build as B
from tests.test_codegen import _assembly, _kernels

SOURCE = "ksa_prefill_bwd_dkv.hip"


def test_tile_loop_does_not_spill():
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    with tempfile.TemporaryDirectory() as d:
        text = _assembly(SOURCE, d)
    kernels = {n: b for n, b in _kernels(text).items() if "ksa_bwd_dkv_direct_kernel" in n}
    assert len(kernels) == 2
    for name, blocks in kernels.items():
        ins = [i for block in blocks.values() for i in block]
        assert sum("v_mfma" in i for i in ins) >= 16 and any(i.startswith("global_load_lds_dwordx4") for i in ins), name
        assert not [i for i in ins if i.startswith("scratch_")], name
    assert not re.findall(r"\bv_pk_(?:add|mul|fma)_f32\b", text)
