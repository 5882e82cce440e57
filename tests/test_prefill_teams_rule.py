"""Which launches of the forward and dQ kernels for short key runs share a query tile's keys between two teams of waves
(ksa_two_teams in ksa_internal.h; no GPU needed)."""
import os
import subprocess

import numpy as np
import pytest

from oracle import ksa_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_24432_amd", "csrc")


@pytest.fixture(scope="module")
def teams(tmp_path_factory):
    """Of (head_dim, workgroups, heads per workgroup, rows per query tile, tokens, c, m, C): longest list, forward, dQ."""
    exe = str(tmp_path_factory.mktemp("plan") / "teams")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "plan", "teams.cpp"),
                    "-o", exe], check=True)

    def run(*line):
        return tuple(int(x) for x in subprocess.run([exe], input=" ".join(map(str, line)), capture_output=True, text=True, check=True).stdout.split())
    return run


def lists(n, c, m, C, q_rows):
    """Keys that some row of a query tile sees, per tile of the two index spaces."""
    mask = np.array(O.mask(n, c, m, C), dtype=bool)
    text = np.array([i // c * (c + m) + i % c for i in range(n)])
    sums = np.array([u // m * (c + m) + c + u % m for u in range(n // c * m)], dtype=int)
    return [int(mask[rows[t:t + q_rows]].any(0).sum()) for rows in (text, sums) for t in range(0, len(rows), q_rows)]


@pytest.mark.parametrize("q_rows", [32, 128])
@pytest.mark.parametrize("layout", [(48, 6, 2), (20, 5, 2), (64, 8, 1), (8, 1, 8), (8, 0, 7), (16, 0, 1), (48, 0, 0), (64, 0, 0), (1, 0, 63), (7, 3, 1)],
                         ids=lambda x: "x".join(map(str, x)))
def test_lists_of_one_tile_take_one_team(teams, layout, q_rows):
    for n in (1, 20, 48, 64, 65, 81, 130, 300):
        most = max(lists(n, *layout, q_rows))
        longest, fwd, dq = teams(64, 8, 1, q_rows, n, *layout)
        assert most <= longest <= most + 48, (n, most, longest)
        if longest <= 64:
            assert (fwd, dq) == (0, 0)
        assert dq == (longest > 64) and fwd == (longest > 72)


# one head, a text of so many tokens at 64: the launches that were measured on both sides
@pytest.mark.parametrize("layout,n,fwd,dq", [((48, 6, 2), 33, 0, 0), ((20, 5, 2), 33, 0, 0), ((8, 0, 128), 64, 0, 0), ((8, 0, 128), 70, 0, 1),
                                             ((48, 0, 0), 2500, 0, 0), ((32, 0, 1), 2500, 0, 0), ((16, 0, 1), 700, 0, 0), ((8, 0, 7), 700, 1, 1),
                                             ((1, 0, 63), 1500, 1, 1), ((64, 8, 1), 512, 1, 1), ((48, 6, 2), 300, 1, 1)])
def test_measured(teams, layout, n, fwd, dq):
    assert teams(64, 40, 1, 32, n, *layout)[1:] == (fwd, dq)
    assert teams(64, 257, 1, 32, n, *layout)[1:] == (0, 0)


def test_head_dim_128(teams):
    assert teams(128, 64, 1, 128, 1024, 8, 1, 128)[1:] == (1, 1)       # more than eight tiles
    assert teams(128, 64, 1, 32, 512, 64, 8, 1)[1:] == (0, 0)
    assert teams(128, 64, 4, 32, 1024, 8, 1, 128)[1:] == (0, 0)        # four heads per workgroup read the same keys
