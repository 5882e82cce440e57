"""GPU parity of the decode kernels where a span, a wave or a lane group has no row or one: a single span per sequence
(the workgroup stores the result itself), more spans than rows, the large workgroups of launches with few spans, and
invalid positions in both forms."""
import numpy as np
import pytest
import torch

import paper_2604_24432_amd as K
from oracle import ksa_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_splits", [0, 1, 2, 9])
@pytest.mark.parametrize("shape", [(1, 4, 1, 128), (3, 8, 1, 64), (2, 2, 2, 64), (2, 4, 2, 128), (40, 8, 8, 128)],
                         ids=lambda s: "x".join(map(str, s)))
def test_rows_and_spans(shape, n_splits):
    B, Hq, Hkv, d = shape
    c, m, C, n = 16, 2, 1, 16 * 130
    p = K.make_params(B, n, c, m, C, Hq, Hkv, d)
    gen = torch.Generator().manual_seed(B + n_splits)
    q, ks, vs, kt, vt = (torch.randn(s, generator=gen).to(torch.bfloat16) for s in
                         ((B, Hq, d), (B, Hkv, n // c * m, d), (B, Hkv, n // c * m, d), (B, Hkv, n, d), (B, Hkv, n, d)))
    pos = [(0, 15, 16, 700, n - 1, 33)[b % 6] for b in range(B)]
    base = [max(0, x // c - C) * c for x in pos]
    s_cap, rows = K.cache_geometry(p)
    kc, vc = (torch.zeros((B, Hkv, rows, d), dtype=torch.bfloat16) for _ in "kv")
    kc[:, :, :s_cap], vc[:, :, :s_cap] = ks, vs
    for b, x in enumerate(pos):
        for i in range(base[b], x + 1):
            kc[b, :, K.cache_text_row(p, i)], vc[b, :, K.cache_text_row(p, i)] = kt[b, :, i], vt[b, :, i]
    W = (C + 1) * c
    win = lambda t: torch.stack([torch.nn.functional.pad(t[b, :, base[b]:base[b] + W], (0, 0, 0, W))[:, :W] for b in range(B)])
    o, lse = K.ksa_decode_fwd(p, q.cuda(), kc.cuda(), vc.cuda(), torch.tensor(pos, dtype=torch.int32).cuda(), n_splits=n_splits)
    ref, ref_lse = O.decode(*(x.float().numpy() for x in (q, ks, vs, win(kt), win(vt))), base, pos, c, m, C)
    err, lerr = np.abs(o.float().cpu().numpy() - ref), np.abs(lse.cpu().numpy() - ref_lse)
    print(f"{shape} splits {n_splits}: max-abs {err.max():.3e} lse {lerr.max():.3e}", flush=True)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3 and lerr.max() <= 1e-4


@pytest.mark.parametrize("n_splits", [1, 3])
def test_invalid_positions_give_nan_rows(n_splits):
    p = K.make_params(3, 256, 16, 2, 1, 4, 2, 64)
    _, rows = K.cache_geometry(p)
    q, kc, vc = (torch.randn(s).to(torch.bfloat16).cuda() for s in ((3, 4, 64), (3, 2, rows, 64), (3, 2, rows, 64)))
    o, lse = K.ksa_decode_fwd(p, q, kc, vc, torch.tensor([-1, 100, 256], dtype=torch.int32).cuda(), n_splits=n_splits)
    assert bool(torch.isnan(o[[0, 2]]).all()) and bool(torch.isnan(lse[[0, 2]]).all())
    assert bool(torch.isfinite(o[1]).all()) and bool(torch.isfinite(lse[1]).all())
