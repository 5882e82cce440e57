"""The plan of the backward pass's dK / dV work (build_dkv in ksa_layout.cpp; no GPU needed): which kernel a launch takes, and that
the pieces of every key tile are the steps that kernel counts for it, each once."""
import os
import subprocess

import numpy as np
import pytest

from oracle import ksa_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_24432_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "dkv_plan")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "plan", "dkv_plan.cpp"), os.path.join(CSRC, "ksa_layout.cpp"), "-o", exe], check=True)

    def run(*shape, flags=0):
        out = subprocess.run([exe], input=" ".join(map(str, shape)) + f" {flags}", capture_output=True, text=True, check=True)
        v = [int(x) for x in out.stdout.split()]
        return dict(direct=v[0], unsplit_direct=v[1], pieces=v[2], splits=v[3], slots=v[4], steps=v[5:])
    return run


# batch, heads, KV heads, d, tokens, c, m, C -> kernel with 32-row query tiles where tiles are split (or none has to be), and where dq
# cannot hold partial sums.  Both kernels were timed on these (see the comment at build_dkv).
MEASURED = [((1, 16, 4, 64, 2048, 1, 0, 1023), 0, 0), ((1, 8, 1, 128, 2048, 1, 0, 1023), 0, 0), ((1, 16, 4, 128, 2048, 8, 1, 128), 0, 0),
            ((1, 16, 4, 128, 4096, 64, 0, 4096), 0, 0), ((1, 16, 16, 64, 2048, 1, 0, 1023), 0, 0), ((1, 8, 1, 64, 4096, 64, 8, 1), 0, 0),
            ((1, 32, 8, 128, 8192, 64, 8, 1), 1, 0), ((1, 32, 8, 64, 8192, 64, 8, 1), 1, 0), ((2, 32, 8, 128, 4096, 64, 8, 1), 1, 0),
            ((1, 16, 16, 128, 4096, 64, 8, 1), 1, 0), ((2, 1, 1, 128, 6551, 20, 5, 2), 0, 0), ((4, 16, 4, 64, 1106, 96, 32, 1), 1, 1), ((1, 16, 16, 128, 20003, 8, 1, 128), 1, 1), ((1, 16, 16, 128, 4096, 1, 0, 1023), 1, 1),
            ((1, 32, 8, 128, 20003, 1, 0, 1023), 1, 1), ((1, 16, 16, 128, 8192, 64, 0, 4096), 1, 1), ((1, 16, 16, 128, 4096, 64, 0, 4096), 0, 0)]


@pytest.mark.parametrize("shape,direct,unsplit_direct", MEASURED, ids=["x".join(map(str, s[0])) for s in MEASURED])
def test_the_faster_kernel_is_taken(plan, shape, direct, unsplit_direct):
    got = plan(*shape)
    assert (got["direct"], got["unsplit_direct"]) == (direct, unsplit_direct)


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("shape", [(1, 8, 1, 128, 2048, 1, 0, 1023), (1, 4, 1, 64, 613, 16, 2, 100), (2, 8, 1, 128, 682, 20, 5, 100),
                                   (1, 8, 1, 64, 1100, 64, 8, 1), (2, 3, 1, 64, 585, 8, 1, 60), (1, 2, 2, 128, 31, 8, 2, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_pieces_are_the_steps_of_the_kernel(plan, shape, flags):
    B, Hq, Hkv, d, n, c, m, C = shape
    got = plan(*shape, flags=flags)
    mask = np.array(O.mask(n, c, m, C, flags=flags), dtype=bool)
    rows = [np.array([u // m * (c + m) + c + u % m for u in range(n // c * m)], dtype=int), np.array([i // c * (c + m) + i % c for i in range(n)])]
    block, want = 32 if got["direct"] else 64, []
    for keys in rows:                    # summary-space tiles come first
        for t in range(0, len(keys), 128):
            blocks = 0
            for q in rows:
                sees = mask[np.ix_(q, keys[t:t + 128])].any(1).nonzero()[0]
                if not got["direct"] and q is rows[0] and keys is rows[0]:   # all later summary rows of the last key's chunk
                    sees = np.arange(t, (min(t + 128, len(keys)) - 1) // m * m + m)
                blocks += sees[-1] // block - sees[0] // block + 1 if len(sees) else 0
            want.append(blocks * (Hq // Hkv))
    assert got["steps"] == want
    assert got["slots"] <= B * mask.shape[0] * Hq // 512 // (B * Hkv)   # one partial sum (128 KiB per 128 x d) per 512 rows of dq


@pytest.mark.parametrize("shape", [(1, 8, 1, 128, 131072, 64, 8, 1), (1, 8, 1, 64, 131072, 8, 1, 128)], ids=lambda s: "x".join(map(str, s)))
def test_building_a_layout_stays_cheap(shape):
    """Every caller pays for the plan, also one that only runs the forward pass.  A layout of one KV head has the most pieces to weigh
    up; it takes 1.1 times as long as one of the same text with 32/8 heads, whose schedule is longer and whose plan is short
    (playing every candidate launch through piece by piece: 3.5 - 4.2 times)."""
    import time

    import paper_2604_24432_amd as K
    B, _, _, d, n, c, m, C = shape
    best = {}
    for _ in range(25):
        for heads in ((8, 1), (32, 8)):
            p = K.make_params(B, n, c, m, C, *heads, d)
            t = time.perf_counter()
            lay = K.ksa_build_layout(p)
            best[heads] = min(best.get(heads, 1.0), time.perf_counter() - t)
            del lay
    print({k: f"{v * 1e6:.0f} us" for k, v in best.items()})
    assert best[8, 1] < 2.5 * best[32, 8]
