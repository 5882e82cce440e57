"""GPU parity of the decode kernels' two ways to the scores (matrix unit with four and eight query heads per KV head, vector
unit with one and two) where a wave's block of 16 or 32 rows crosses from the summaries into the ring, over the ring's seam or
past the last row, and with cache rows that are not dense.  Every row that the token does not see is a NaN, so a weight of zero
would not hide it.  The reference is the softmax over the visible rows in 64 bits; the outputs are bf16 of values below 4
(2^-7 at most for the last rounding), the log-sum-exp comes from fp32 scores (1e-4, as in test_gpu_decode.py)."""
import numpy as np
import pytest
import torch

import paper_2604_24432_amd as K

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_splits", [1, 3])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (8, 2), (8, 1), (12, 3)], ids=lambda h: "x".join(map(str, h)))
@pytest.mark.parametrize("form", [(5, 1, 9), (64, 8, 1), (24, 3, 2), (1, 0, 76)], ids=lambda f: "x".join(map(str, f)))
def test_blocks_across_the_pieces_of_the_cache(form, heads, d, n_splits):
    (c, m, C), (Hq, Hkv) = form, heads
    n = 40 * max(c, 5)
    pos = [0, 1, c * (C + 1) - 1, c * (C + 1), c * (C + 2) + c // 2, n // 2 + 3, n - 1, 17]
    B, G = len(pos), Hq // Hkv
    p = K.make_params(B, n, c, m, C, Hq, Hkv, d)
    _, rows = K.cache_geometry(p)
    gen = torch.Generator().manual_seed(c * 100 + d + Hq)
    q = torch.randn((B, Hq, d), generator=gen).to(torch.bfloat16)
    kv = torch.full((2, B, rows, Hkv, d), float("nan"), dtype=torch.bfloat16)     # heads between the rows: not dense
    want, want_lse = np.zeros((B, Hq, d)), np.zeros((B, Hq))
    for b, x in enumerate(pos):
        r = K.ksa_decode_ranges(p, x)
        seen = np.concatenate([np.arange(r[i], r[i] + r[i + 1]) for i in (0, 2, 4)])
        kv[:, b, seen] = torch.randn((2, len(seen), Hkv, d), generator=gen).to(torch.bfloat16)
        for h in range(Hq):
            ks, vs = (kv[i, b, seen, h // G].double().numpy() for i in (0, 1))
            s = ks @ q[b, h].double().numpy() / np.sqrt(d)
            w = np.exp(s - s.max())
            want[b, h], want_lse[b, h] = w @ vs / w.sum(), s.max() + np.log(w.sum())
    k, v = (t.permute(0, 2, 1, 3) for t in kv.cuda())
    o, lse = K.ksa_decode_fwd(p, q.cuda(), k, v, torch.tensor(pos, dtype=torch.int32).cuda(), n_splits=n_splits)
    err, lerr = np.abs(o.double().cpu().numpy() - want), np.abs(lse.cpu().numpy() - want_lse)
    print(f"{form} {heads} d{d} splits {n_splits}: max-abs {err.max():.3e} lse {lerr.max():.3e}", flush=True)
    assert np.isfinite(err).all() and (err <= 1e-4 + 2.0 ** -8 * np.abs(want)).all() and lerr.max() <= 1e-4


@pytest.mark.parametrize("cancel", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (8, 2), (8, 1)], ids=lambda h: "x".join(map(str, h)))
def test_scores_whose_unscaled_products_exceed_fp32(heads, d, cancel):
    """q . k of one row is beyond fp32, or a partial sum of it far below, while the scaled score is not: the row has all the weight."""
    (c, m, C), (Hq, Hkv), n = (64, 8, 1), heads, 1500
    p = K.make_params(1, n, c, m, C, Hq, Hkv, d)
    _, rows = K.cache_geometry(p)
    gen = torch.Generator().manual_seed(d + Hq)
    k, v = (torch.randn((1, Hkv, rows, d), generator=gen).to(torch.bfloat16) for _ in range(2))
    q = torch.full((1, Hq, d), 0.25, dtype=torch.bfloat16)
    r = K.ksa_decode_ranges(p, n - 1)
    row = r[2] + r[3] // 2
    k[0, :, row] = 2.0 ** 126 if cancel and d == 64 else 2.0 ** 125
    if cancel:
        k[0, :, row, :32] = -2.0 ** 125           # -2^128 so far
    for n_splits in (1, 3):
        o, lse = K.ksa_decode_fwd(p, q.cuda(), k.cuda(), v.cuda(), torch.tensor([n - 1], dtype=torch.int32).cuda(), n_splits=n_splits)
        assert torch.equal(o[0].cpu(), v[0, :, row].repeat_interleave(Hq // Hkv, 0))
        want = 0.25 * float(k[0, 0, row].double().sum()) / np.sqrt(d)
        assert np.abs(lse.cpu().double().numpy() / want - 1).max() <= 1e-6      # fp32: the scale, its product, the logarithm's base
