"""The HBM traffic summary finds the kernels that the benchmark workload runs today, and bench.py names them."""
import os
import re
import tempfile

import pytest

from paper_2604_24432_amd import build as B
from paper_2604_24432_amd import traffic_summary as T
from tests.test_codegen import _assembly, _kernels

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _mangled(name):
    """ksa_x<128, 4, true> -> the part of its symbol that says the same."""
    base, _, args = name.replace(" ", "").rstrip(">").partition("<")
    return base + "I" + "".join(f"Lb{int(a == 'true')}E" if a in ("true", "false") else f"Li{a}E" for a in args.split(",")) + "E"


@pytest.mark.parametrize("key", ["prefill", "decode"])
def test_the_workloads_kernels_exist_under_the_names_given(key):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    name = dict(T.KERNELS)[key]
    with tempfile.TemporaryDirectory() as d:
        symbols = _kernels(_assembly({"prefill": "ksa_prefill.hip", "decode": "ksa_decode.hip"}[key], d))
    assert [s for s in symbols if _mangled(name) in s], name
    bench = open(os.path.join(ROOT, "bench.py")).read()
    assert name.replace(" ", "") in bench.replace(" ", "")


def test_summary_from_counter_files(tmp_path, monkeypatch):
    names = {"copy": "__amd_rocclr_copyBuffer", **{k: f"void (anonymous namespace)::{n}((anonymous namespace)::Args)" for k, n in T.KERNELS}}
    for counter, values in (("FETCH_SIZE", (524288, 2000, 3000)), ("WRITE_SIZE", (1048576, 100, 200))):
        os.makedirs(tmp_path / counter)
        with open(tmp_path / counter / "x_counter_collection.csv", "w") as f:
            f.write("Kernel_Name,Counter_Name,Counter_Value\n")
            f.writelines(f'"{n}",{counter},{v}\n' for n, v in zip(names.values(), values))
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(T, "ROOT", str(tmp_path))
    monkeypatch.setattr("sys.argv", ["x", str(tmp_path / "FETCH_SIZE"), str(tmp_path / "WRITE_SIZE"), "abc"])
    monkeypatch.syspath_prepend(ROOT)
    T.main()
    text = (tmp_path / "profiles" / "hbm_traffic.txt").read_text()
    got = {k: float(v) for k, v in re.findall(r"(\w+)_traffic_bytes: (\S+)", text)}
    assert got == {"prefill": pytest.approx((4000 + 100) * 1024, rel=1e-3), "decode": pytest.approx((6000 + 200) * 1024, rel=1e-3)}
