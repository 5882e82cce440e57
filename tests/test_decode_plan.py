"""How many spans a decode call takes that leaves their number to the library (plan_decode in ksa_api.cpp; no GPU needed)."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_24432_amd", "csrc")
TEXT, SUMMARY, STATIC = 0, 1, 2
STATIC_BYTES = 8 << 20


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """Of a list of (entry, least workspace or not, batch, heads, KV heads, d, tokens, c, m, C)."""
    exe = str(tmp_path_factory.mktemp("plan") / "decode_plan")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "tests", "sanitize", "hip_stub"), "-I", os.path.join(ROOT, "include"),
                    "-I", CSRC, os.path.join(ROOT, "tests", "plan", "decode_plan.cpp"), os.path.join(CSRC, "ksa_api.cpp"),
                    os.path.join(CSRC, "ksa_layout.cpp"), "-o", exe], check=True)

    def run(calls):
        out = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in calls), capture_output=True, text=True, check=True)
        return [dict(zip(("status", "n_splits", "n_spans", "wide", "bytes"), map(int, line.split()))) for line in out.stdout.splitlines()]
    return run


def call(batch, heads, kv_heads, d, rows, entry=TEXT, least=0):
    """With a cache of about so many rows (chunks of 64 with 8 summaries, a window of two chunks)."""
    return (entry, least, batch, heads, kv_heads, d, max(2, (rows - 128) // 8) * 64, 64, 8, 1)


def rows_of(c):
    return c[6] // c[7] * c[8] + (c[9] + 1) * c[7]


def random_calls(count, seed):
    rng = random.Random(seed)
    for _ in range(count):
        kv_heads = rng.choice([1, 1, 2, 3, 4, 8, 8, 16, 32, 64])
        batch = rng.choice([1, 2, 3, 5, 8, 13, 16, 24, 31, 33, 48, 63, 64, 65, 70, 100, 200])
        rows = int(10 ** rng.uniform(2.3, 6))
        if batch * kv_heads * rows < 1e8:
            yield call(batch, kv_heads * rng.choice([1, 2, 4, 8]), kv_heads, rng.choice([64, 128]), rows, rng.choice([TEXT, TEXT, TEXT, STATIC]), rng.choice([0, 0, 1]))


def test_dealt_spans_are_several_per_sequence(plans):
    """Spans are dealt by length only where every sequence can have two and more on average: with fewer there is nothing to balance, and
    records and merge are for nothing."""
    calls = [c for c in random_calls(20000, 1)]
    dealt = 0
    for c, got in zip(calls, plans(calls)):
        batch, heads, kv_heads, d = c[2:6]
        if got["status"]:
            assert c[0] == STATIC     # (records of the least number beyond the static array)
            continue
        assert got["n_spans"] * heads * (d + 2) * 4 <= (STATIC_BYTES if c[0] == STATIC else got["bytes"])
        if got["n_splits"]:
            assert got["n_spans"] == batch * got["n_splits"]
            continue
        dealt += 1
        assert 1 < batch <= 64 and got["n_spans"] >= 2 * batch, (c, got)
    assert dealt > 200


# batch, heads, KV heads, rows -> spans per sequence (0: dealt) that were the fastest or level with them; see the comment at plan_decode
@pytest.mark.parametrize("shape,n_splits,n_spans", [((64, 32, 32, 1600), 1, 64), ((64, 64, 32, 2096), 1, 64), ((33, 64, 32, 4000), 2, 66), ((44, 128, 32, 3500), 2, 88),
                                                    ((64, 16, 16, 1600), 2, 128), ((33, 32, 16, 9000), 0, 99), ((60, 32, 16, 1600), 0, 180),
                                                    ((64, 16, 8, 6400), 0, 160), ((33, 8, 2, 11496), 0, 256), ((8, 32, 8, 9352), 0, 64),
                                                    ((16, 16, 8, 6640), 0, 96), ((96, 16, 4, 7808), 4, 384), ((4, 32, 8, 21872), 16, 64),
                                                    ((28, 128, 32, 3500), 0, 56), ((64, 32, 8, 16504), 0, 192), ((8, 32, 8, 17000), 0, 64)],
                         ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else None)
def test_many_sequences_and_heads(plans, shape, n_splits, n_spans):
    batch, heads, kv_heads, rows = shape
    got, = plans([call(batch, heads, kv_heads, 128, rows)])
    assert (got["status"], got["n_splits"], got["n_spans"]) == (0, n_splits, n_spans)


def test_a_workspace_of_the_asked_size_changes_nothing(plans):
    calls = [c for c in random_calls(5000, 2) if c[0] == TEXT and c[1] == 0]
    for c, own, static in zip(calls, plans(calls), plans([(STATIC, *c[1:]) for c in calls])):
        if static["status"] == 0:
            assert all(own[x] == static[x] for x in ("n_splits", "n_spans", "wide")), c


def test_spans_are_not_too_short(plans):
    """More than 64 spans of a sequence have 768 rows each, or 512 within one round of workgroups; and none has less than 16."""
    calls = list(random_calls(20000, 3))
    for c, got in zip(calls, plans(calls)):
        n, groups, rows = got["n_splits"], c[2] * c[4], rows_of(c)
        if n > 1:
            assert n <= max(64, rows // 768, min(rows // 512, 256 // groups)) and n * 16 <= rows, (c, got)


@pytest.mark.parametrize("shape,workgroups", [((3, 2, 1, 50000), 255), ((3, 1, 1, 93328), 255), ((3, 2, 1, 76664), 255),
                                              ((1, 64, 8, 118744), 512), ((1, 32, 8, 118744), 512), ((3, 1, 1, 316664), 768), ((1, 8, 8, 35000), 512)])
def test_the_last_round_is_full_with_few_long_sequences(plans, shape, workgroups):
    batch, heads, kv_heads, rows = shape
    got, = plans([call(batch, heads, kv_heads, 128, rows)])
    assert got["n_spans"] * kv_heads == workgroups
