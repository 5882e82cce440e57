"""GPU parity of the forward and dQ kernels for short key runs in launches with no more workgroups than compute units, where eight
waves share a query tile's keys: lists of one tile (a launch of its own, or nothing for the second four), of an even and an odd number, both softmax
references, waves without rows, and rows that are no numbers."""
import numpy as np
import pytest
import torch

import paper_2604_24432_amd as K
from paper_2604_24432_amd import synth
from oracle import ksa_oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, Hq, Hkv, d, n, c, m, C
    *[(1, 2, 1, 64, n, 16, 2, 1) for n in (1, 16, 40, 500)],       # one and two tiles
    *[(1, 1, 1, 64, n, 64, 8, 1) for n in (190, 321, 1500)],       # up to six, most of them the same for all rows
    (2, 3, 1, 64, 700, 48, 6, 2),                                  # running maxima, one head per workgroup
    (1, 8, 1, 64, 1100, 20, 5, 2),                                 # four heads per workgroup
    (1, 2, 2, 128, 900, 8, 1, 128),                                # head_dim 128: lists of more than eight tiles
    (1, 3, 1, 128, 1000, 512, 0, 3),
    (1, 3, 1, 128, 1100, 24, 3, 40),
    (3, 1, 1, 128, 1201, 1, 0, 600),
]


@pytest.mark.parametrize("outliers", [0.0, 0.03])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_against_oracle(shape, outliers):
    B, Hq, Hkv, d, n, c, m, C = shape
    cfg = synth.KsaConfig("teams", B, Hq, Hkv, d, n, c, m, C, seed=n + c, key_outlier_frac=outliers)
    q, k, v = synth.make_prefill_inputs(cfg)
    g = synth.make_upstream_gradient(cfg)
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, Hq, Hkv, d))
    dev = [x.cuda() for x in (q, k, v)]
    o, lse = K.ksa_prefill_fwd(lay, *dev)
    host = [x.float().numpy() for x in (q, k, v)]
    o_ref, lse_ref = O.prefill(*host, n, c, m, C)
    err, lerr = np.abs(o.float().cpu().numpy() - o_ref), np.abs(lse.cpu().numpy() - lse_ref)
    print(f"{shape}: max-abs {err.max():.3e} mean-abs {err.mean():.3e} lse {lerr.max():.3e}", flush=True)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3 and lerr.max() <= 4e-3     # the bars of test_gpu_prefill_direct.py
    dq = K.ksa_prefill_bwd(lay, *dev, o, lse, g.cuda())[0]
    ref = O.prefill_bwd(*host, g.float().numpy(), n, c, m, C)[0]
    rel = np.linalg.norm(dq.float().cpu().numpy() - ref) / max(np.linalg.norm(ref), 1e-3)
    print(f"  dq: relative error {rel:.2e}", flush=True)
    # test_gpu_prefill_bwd_split.py; with outliers rows are nearly one-hot and the forward's rounded output (2^-9) enters delta
    assert rel <= (5e-3 if outliers == 0 else 2.4e-2)


@pytest.mark.parametrize("shape", [(1, 1, 1, 64, 640, 64, 8, 1), (1, 1, 1, 64, 640, 48, 6, 1), (1, 2, 2, 128, 900, 8, 1, 128)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_no_number_stays_in_its_row(shape, value):
    B, Hq, Hkv, d, n, c, m, C = shape
    cfg = synth.KsaConfig("teams", B, Hq, Hkv, d, n, c, m, C, seed=n)
    q, k, v = (x.cuda() for x in synth.make_prefill_inputs(cfg))
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, Hq, Hkv, d))
    want, _ = K.ksa_prefill_fwd(lay, q, k, v)
    rows = [0, cfg.aug_len // 2 + 3, cfg.aug_len - 1]
    q[:, rows, :, 5] = value
    got, lse = K.ksa_prefill_fwd(lay, q, k, v)
    others = [x for x in range(cfg.aug_len) if x not in rows]
    assert bool(torch.isfinite(got[:, others].float()).all()) and bool(torch.isfinite(lse[:, :, others]).all())
    assert bool(torch.isnan(got[:, rows].float()).all())
    # (rows beside one that is no number keep running maxima instead of a fixed reference: another rounding of the weights)
    assert (got[:, others].float() - want[:, others].float()).norm() <= 9e-3 * want[:, others].float().norm()


@pytest.mark.parametrize("d,n", [(64, 1), (64, 8), (64, 70), (64, 1420), (64, 1600), (128, 1), (128, 33), (128, 380), (128, 410), (128, 900)])
def test_largest_key_norm(d, n):
    """Short texts, whose workgroups take the K norms themselves, and those just beyond: the workspace ends with the largest squared
    norm of each KV head (exact for whole-numbered keys), whichever row it is in."""
    B, H, c, m = 2, 2, 8, 1
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, 1, H, H, d))
    ws = torch.empty(K.prefill_workspace_bytes(lay), dtype=torch.uint8, device="cuda")
    q, v = (f(B, lay.aug_len, H, d, dtype=torch.bfloat16, device="cuda") for f in (torch.zeros, torch.ones))
    for row in {0, lay.aug_len // 2, lay.aug_len - 1}:
        k = torch.ones_like(v)
        k[1, row, 0, d - 1] = 16
        o, _ = K.ksa_prefill_fwd(lay, q, k, v, workspace=ws)
        assert ws[-4 * B * H:].view(torch.float32).tolist() == [d, d, d - 1 + 256, d], row
        assert bool((o == 1).all())
