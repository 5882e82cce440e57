"""GPU parity of the dK / dV kernel with 32-row query tiles (ksa_prefill_bwd_dkv.hip) and of the line to the one with 64-row
blocks (which layout takes which: test_layout_dkv.py): chunks that divide a query tile, are divided by one, or neither; incomplete
last tiles of either space; one to eight query heads per KV head; rows that are no numbers, or whose log-sum-exp is none."""
import math

import numpy as np
import pytest
import torch

import paper_2604_24432_amd as K
from paper_2604_24432_amd import synth
from oracle import ksa_oracle as O

pytestmark = pytest.mark.gpu


def run(shape, flags=0, seed=0):
    B, Hq, Hkv, d, n, c, m, C = shape
    cfg = synth.KsaConfig("dkv", B, Hq, Hkv, d, n, c, m, C, seed=n + c + seed)
    q, k, v = (x.cuda() for x in synth.make_prefill_inputs(cfg))
    g = synth.make_upstream_gradient(cfg).cuda()
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, Hq, Hkv, d, flags=flags))
    return cfg, lay, q, k, v, g


# batch, heads, KV heads, d, n, c, m, C
SHAPES = [(1, 4, 2, 128, 31, 8, 1, 2), (1, 2, 1, 128, 33, 16, 2, 1), (2, 3, 1, 64, 129, 32, 4, 0), (1, 8, 1, 128, 353, 64, 8, 1),
          (1, 2, 2, 64, 641, 96, 32, 1), (1, 4, 1, 128, 500, 128, 64, 1), (1, 2, 1, 128, 479, 48, 6, 2), (1, 2, 2, 64, 383, 1, 0, 70),
          (1, 4, 4, 128, 417, 2, 1, 100), (1, 4, 4, 128, 900, 128, 64, 1), (1, 2, 2, 128, 510, 64, 0, 9), (1, 2, 2, 64, 300, 100, 0, 9), (1, 2, 1, 128, 385, 64, 0, 9)]


@pytest.mark.parametrize("self_only", [0, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_against_oracle(shape, self_only):
    if self_only and shape[6] < 2:
        pytest.skip("one summary per chunk")
    cfg, lay, q, k, v, g = run(shape, K.KSA_FLAG_SUMMARY_SELF_ONLY if self_only else 0)
    o, lse = K.ksa_prefill_fwd(lay, q, k, v)
    got = K.ksa_prefill_bwd(lay, q, k, v, o, lse, g)
    ref = O.prefill_bwd(*(x.float().cpu().numpy() for x in (q, k, v, g)), cfg.n_text, cfg.chunk_len, cfg.n_summary,
                        cfg.window_chunks, flags=self_only)
    for name, x, r in zip(("dq", "dk", "dv"), got, ref):
        # bf16 weights (2^-9 each, in quadrature), the forward's bf16 output in delta, one bf16 rounding of the result: see
        # test_gpu_prefill_bwd_split.py; few keys per row are at the upper end
        rel = np.linalg.norm(x.float().cpu().numpy() - r) / np.linalg.norm(r)
        print(f"{shape} {name}: relative error {rel:.2e}", flush=True)
        assert rel <= 5e-3, name


# launches that the kernel with 64-row blocks takes, with split tiles
WIDE = [(1, 8, 1, 64, 700, 1, 0, 400), (1, 3, 1, 128, 1060, 100, 4, 4), (1, 8, 1, 64, 536, 48, 6, 1), (2, 3, 1, 64, 585, 8, 1, 60),
        (2, 3, 1, 128, 1146, 64, 8, 4), (2, 8, 1, 64, 640, 1, 0, 500)]


@pytest.mark.parametrize("packed", [False, True], ids=["dense", "packed"])
@pytest.mark.parametrize("self_only", [0, 1])
@pytest.mark.parametrize("shape", WIDE + [(1, 8, 2, 128, 1300, 64, 8, 1)], ids=lambda s: "x".join(map(str, s)))
def test_split_tiles_of_64_row_blocks_and_packed_gradients(shape, self_only, packed):
    """packed: gradients in one tensor, whose dq cannot hold partial sums, so that no tile is split."""
    if self_only and shape[6] < 2:
        pytest.skip("one summary per chunk")
    cfg, lay, q, k, v, g = run(shape, K.KSA_FLAG_SUMMARY_SELF_ONLY if self_only else 0)
    o, lse = K.ksa_prefill_fwd(lay, q, k, v)
    Hq, Hkv = shape[1], shape[2]
    out = {}
    if packed:
        both = torch.empty((shape[0], q.shape[1], Hq + 2 * Hkv, shape[3]), dtype=torch.bfloat16, device="cuda")
        out = dict(dq=both[:, :, :Hq], dk=both[:, :, Hq:Hq + Hkv], dv=both[:, :, Hq + Hkv:])
    got = K.ksa_prefill_bwd(lay, q, k, v, o, lse, g, **out)
    ref = O.prefill_bwd(*(x.float().cpu().numpy() for x in (q, k, v, g)), cfg.n_text, cfg.chunk_len, cfg.n_summary,
                        cfg.window_chunks, flags=self_only)
    for name, x, r in zip(("dq", "dk", "dv"), got, ref):
        rel = np.linalg.norm(x.float().cpu().numpy() - r) / np.linalg.norm(r)   # bound: see test_against_oracle
        print(f"{shape} {name}: relative error {rel:.2e}", flush=True)
        assert rel <= 5e-3, name


@pytest.mark.parametrize("value", [math.nan, -math.inf, math.inf])
@pytest.mark.parametrize("shape", [(1, 2, 1, 128, 353, 64, 8, 1), (1, 2, 2, 64, 383, 1, 0, 70), (1, 2, 2, 64, 900, 128, 64, 1)],
                         ids=["chunks", "window", "64-row blocks"])
def test_log_sum_exp_that_is_no_number(shape, value):
    """A weight of a row without a log-sum-exp is none (infinite: zero) for the keys that the row sees and zero for the others, in
    both gradients."""
    cfg, lay, q, k, v, g = run(shape)
    o, lse = K.ksa_prefill_fwd(lay, q, k, v)
    row = 200
    lse[0, :, row] = value
    _, dk, dv = K.ksa_prefill_bwd(lay, q, k, v, o, lse, g)
    g0 = g.clone()
    g0[0, row] = 0                       # without the row's contribution
    lse[0, :, row] = math.inf
    _, want_dk, want_dv = K.ksa_prefill_bwd(lay, q, k, v, o, lse, g0)
    sees = torch.from_numpy(np.array(O.mask(cfg.n_text, cfg.chunk_len, cfg.n_summary, cfg.window_chunks)[row], dtype=bool)).cuda()
    for x, want in ((dk, want_dk), (dv, want_dv)):
        assert torch.equal(x[0, ~sees], want[0, ~sees])
        if value == math.inf:
            assert torch.equal(x, want)
        else:
            assert not bool(torch.isfinite(x[0, sees]).any())


@pytest.mark.parametrize("shape,space,at", [((1, 8, 2, 128, 1024, 64, 8, 1), 1, 16), ((1, 8, 2, 128, 960, 48, 6, 1), 1, 20),
                                            ((1, 4, 4, 128, 2048, 8, 1, 128), 1, 17), ((1, 4, 2, 64, 1024, 128, 16, 1), 1, 16),
                                            ((1, 4, 4, 128, 1024, 1, 0, 199), 0, 330), ((1, 4, 4, 64, 1024, 1, 0, 199), 0, 330)],
                         ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else str(x))
def test_row_behind_those_that_see_a_key_tile(shape, space, at):
    """A NaN or infinity in a row behind the last one that sees any of a tile's 128 keys changes nothing in the tile's gradients,
    also where the row shares a query tile with that last one.  (dO itself enters every row's delta, which dK of a query tile's
    keys takes whole: there only dV is asked.)"""
    cfg, lay, q, k, v, g = run(shape)
    n, c, m = cfg.n_text, cfg.chunk_len, cfg.n_summary
    o, lse = K.ksa_prefill_fwd(lay, q, k, v)
    _, dk, dv = K.ksa_prefill_bwd(lay, q, k, v, o, lse, g)
    rows = [np.array([i // c * (c + m) + i % c for i in range(n)]),
            np.array([u // m * (c + m) + c + u % m for u in range(n // c * m)], dtype=int)]
    mask = np.array(O.mask(n, c, m, cfg.window_chunks), dtype=bool)
    behind = []                          # keys of the tiles whose rows of this space all lie in front of row `at`
    for keys in rows:
        for t in range(0, len(keys), 128):
            sees = mask[np.ix_(rows[space], keys[t:t + 128])].any(1).nonzero()[0]
            if len(sees) == 0 or sees[-1] < at:
                behind.append(keys[t:t + 128])
    behind = torch.from_numpy(np.concatenate(behind)).cuda()
    for name, x, value in (("dO", g, math.nan), ("dO", g, math.inf), ("q", q, math.nan), ("q", q, math.inf)):
        keep = x.clone()
        x[0, int(rows[space][at])] = value
        _, dk1, dv1 = K.ksa_prefill_bwd(lay, q, k, v, o, lse, g)
        x.copy_(keep)
        assert torch.equal(dv1[0, behind], dv[0, behind]), (name, value)
        assert name == "dO" or torch.equal(dk1[0, behind], dk[0, behind]), (name, value)
        assert not bool(torch.isfinite(dk1).all()), (name, value)   # it reached those that see it
