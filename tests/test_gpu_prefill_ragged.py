"""GPU parity of the pipelined forward kernel (long key runs) where a run's last key tile reaches past the end of its index
space: texts that end on, before and behind a multiple of 64 and of 16, summary runs that end inside a tile.  Sampled rows
against the oracle, with the last rows of the text and of the summaries among them; every row's count of visible keys through
Q = 0 (tolerances and method of test_gpu_prefill.py)."""
import numpy as np
import pytest
import torch

import paper_2604_24432_amd as K
from paper_2604_24432_amd import synth
from oracle import ksa_oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, Hq, Hkv, d, n, c, m, C: enough key tiles per query tile for this kernel
    *[(1, 4, 1, 128, n, 64, 0, 4096) for n in (4097, 4159, 4177)],
    (2, 4, 1, 128, 4099, 4, 0, 4096),           # runs that start off the chunk grid
    (1, 4, 1, 128, 36893, 64, 8, 1),
    (1, 4, 1, 128, 40009, 8, 1, 128),
    (1, 4, 1, 64, 32801, 64, 0, 4096),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_ends_of_runs(shape):
    B, Hq, Hkv, d, n, c, m, C = shape
    cfg = synth.KsaConfig("ragged", B, Hq, Hkv, d, n, c, m, C, seed=n, key_outlier_frac=0.01 if n % 2 else 0.0)
    q, k, v = synth.make_prefill_inputs(cfg)
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, Hq, Hkv, d))
    kd, vd = k.cuda(), v.cuda()
    o, lse = K.ksa_prefill_fwd(lay, q.cuda(), kd, vd)
    rows = np.unique(np.concatenate([synth.sample_rows(cfg, 24).numpy()[-64:], np.arange(cfg.aug_len - 40, cfg.aug_len),
                                     np.random.default_rng(n).integers(0, cfg.aug_len, 24)]))
    o_ref, lse_ref = O.prefill(q.float().numpy(), k.float().numpy(), v.float().numpy(), n, c, m, C, rows=rows)
    err = np.abs(o.float().cpu().numpy()[:, rows] - o_ref)
    lerr = np.abs(lse.cpu().numpy()[:, :, rows] - lse_ref)
    print(f"{shape}: max-abs {err.max():.3e} mean-abs {err.mean():.3e} lse {lerr.max():.3e}", flush=True)
    assert bool(torch.isfinite(o.float()).all()) and err.max() <= 2e-2 and err.mean() <= 2e-3 and lerr.max() <= 4e-3
    _, lse = K.ksa_prefill_fwd(lay, torch.zeros_like(q).cuda(), kd, vd)
    a = np.arange(cfg.aug_len, dtype=np.int64)
    j, r = a // (c + m), a % (c + m)
    want = np.where(r < c, np.minimum(j, C) * c + r + 1 + np.maximum(j - C, 0) * m, c + (r - c) + 1)
    assert np.array_equal(np.rint(np.exp(lse.cpu().numpy().astype(np.float64))), np.broadcast_to(want, lse.shape))
