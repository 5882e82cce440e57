"""Generated code of ksa_decode.hip (no GPU needed): where spans are dealt by the sequences' lengths, the decode kernels and the merge
kernel each work out how many a sequence takes, in floating point, and have to agree on it to the last bit."""
import os
import re
import struct
import tempfile

import pytest

from paper_2604_24432_amd import build as B
from tests.test_codegen import _assembly, _kernels


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    with tempfile.TemporaryDirectory() as d:
        return _kernels(_assembly("ksa_decode.hip", d))


def test_dealing_fuses_no_product_into_a_sum(kernels):
    """The bounds of the search are products with 1.0001 and 1.0002, halved sums of which follow: plain multiplications in every kernel."""
    literals = [hex(struct.unpack("I", struct.pack("f", x))[0]) for x in (1.0001, 1.0002)]
    dealing = {}
    for name, blocks in kernels.items():
        uses = [i for ins in blocks.values() for i in ins if any(x in i for x in literals)]
        if uses:
            dealing[name] = uses
    # two head sizes: four kernels by query heads per KV head, two merge kernels
    assert len(dealing) == 12 and sum("merge" in n for n in dealing) == 4, list(dealing)
    for name, uses in dealing.items():
        fused = [i for i in uses if not re.match(r"v_mul_f32", i)]
        assert not fused and len(uses) == 2, (name, uses)
