"""GPU parity of the decode step where the library chooses the number of spans: each of its choices (one span per sequence in a
large workgroup, many short spans, spans dealt by the sequences' lengths), with sequences of one row, invalid positions, and a
workspace of the least accepted size, which holds fewer spans than the library would take."""
import numpy as np
import pytest
import torch

import paper_2604_24432_amd as K
from oracle import ksa_oracle as O

pytestmark = pytest.mark.gpu


def inputs(B, Hq, Hkv, d, n, c, m, C, pos, seed):
    """Caches in which every row is the one of its text index or summary ordinal, and the oracle's logical rows."""
    p = K.make_params(B, n, c, m, C, Hq, Hkv, d)
    s_cap, rows = K.cache_geometry(p)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q, kc, vc = (torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
                 for s in ((B, Hq, d), (B, Hkv, rows, d), (B, Hkv, rows, d)))
    base = [max(0, x // c - C) * c for x in pos]
    W = (C + 1) * c
    at = torch.tensor([[K.cache_text_row(p, min(t, n - 1)) for t in range(b, b + W)] for b in base], device="cuda")
    win = lambda t: t[torch.arange(B, device="cuda")[:, None], :, at].transpose(1, 2)
    ref, ref_lse = O.decode(*(x.float().cpu().numpy() for x in (q, kc[:, :, :s_cap], vc[:, :, :s_cap], win(kc), win(vc))),
                            base, pos, c, m, C)
    return p, q, kc, vc, torch.tensor(pos, dtype=torch.int32, device="cuda"), ref, ref_lse


def compare(name, o, lse, ref, ref_lse):
    err, lerr = np.abs(o.float().cpu().numpy() - ref), np.abs(lse.cpu().numpy() - ref_lse)
    print(f"{name}: max-abs {err.max():.3e} mean-abs {err.mean():.3e} lse {lerr.max():.3e}", flush=True)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3 and lerr.max() <= 1e-4   # the bars of the other decode tests


def least_workspace(p):
    """What a call with n_splits = 0 accepts: about 1536 workgroups, spans of at least 768 rows."""
    groups, rows = p.batch * p.n_kv_heads, K.cache_geometry(p)[1]
    splits = max(1, min(-(-1536 // groups), max(1, rows // 768), 64))
    return torch.empty(p.batch * p.n_q_heads * splits * (p.head_dim + 2) * 4, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("case", [
    # B, Hq, Hkv, d, n, c, m, C: rows of a full cache
    (1, 4, 1, 128, 16 * 130, 16, 2, 1),        # 292: a few spans
    (1, 8, 1, 64, 16 * 2000, 16, 2, 1),        # 4032: 64 spans of one sequence
    (3, 8, 8, 128, 20 * 300, 20, 5, 2),        # 1560: a workgroup per compute unit
    (13, 16, 4, 128, 64 * 60, 64, 8, 1),       # 608: a number of pairs that fills no round
    (24, 8, 8, 128, 64 * 50, 64, 8, 1),        # 528 in 192 pairs: one span each in large workgroups
    (16, 32, 16, 64, 1500, 1, 0, 1023),        # 1024 in 256 pairs: the same with two heads per KV head
    (70, 8, 8, 64, 64 * 200, 64, 8, 1),        # 1728 in 560 pairs: more than 64 sequences
], ids=lambda c: "x".join(map(str, c)))
def test_default_spans(case):
    B, n = case[0], case[4]
    pos = [(n - 1, 0, n // 2, 15, 16, n - 17)[b % 6] for b in range(B)]
    p, q, kc, vc, pos_t, ref, ref_lse = inputs(*case, pos, seed=B)
    assert K.decode_workspace_bytes(p) >= least_workspace(p).numel()
    compare(f"{case}", *K.ksa_decode_fwd(p, q, kc, vc, pos_t), ref, ref_lse)
    compare("  least workspace", *K.ksa_decode_fwd(p, q, kc, vc, pos_t, workspace=least_workspace(p)), ref, ref_lse)


@pytest.mark.parametrize("shape", [(8, 8, 8, 64), (64, 4, 1, 64), (5, 16, 8, 64), (3, 16, 2, 64)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("alike", [False, True])
def test_dealt_spans(shape, alike):
    """A million rows in all: full caches, one long sequence among short ones, one that reads a single row."""
    B, Hq, Hkv, d = shape
    c, m, C = 64, 8, 1
    n = -(-1_000_000 // (B * Hkv) // m) * c
    pos = [n - 1] * B if alike else [(n - 1, 0, n // 3, 64, n - 70, 200)[b % 6] for b in range(B)]
    p, q, kc, vc, pos_t, ref, ref_lse = inputs(B, Hq, Hkv, d, n, c, m, C, pos, seed=B)
    o, lse = K.ksa_decode_fwd(p, q, kc, vc, pos_t)
    compare(f"{shape} rows {K.cache_geometry(p)[1]}", o, lse, ref, ref_lse)
    compare("  least workspace", *K.ksa_decode_fwd(p, q, kc, vc, pos_t, workspace=least_workspace(p)), ref, ref_lse)
    so, slse = torch.full_like(q, 7.0), torch.full((B, Hq), 7.0, device="cuda")
    K.ksa_decode_fwd_static(p, q, kc, vc, pos_t, so, slse)
    assert torch.equal(so, o) and torch.equal(slse, lse)
    bad = pos_t.clone()
    bad[1:B - 1] = -1        # sequences that read nothing among those that do
    o2, lse2 = K.ksa_decode_fwd(p, q, kc, vc, bad)
    assert bool(torch.isnan(o2[1:B - 1]).all()) and bool(torch.isnan(lse2[1:B - 1]).all())
    for b in (0, B - 1):
        compare(f"  sequence {b} beside invalid ones", o2[b], lse2[b], ref[b], ref_lse[b])


@pytest.mark.parametrize("shape", [
    # B, Hq, Hkv, d, rows: spans that the library deals
    (9, 8, 2, 128, 31000),      # four query heads per KV head: 256 for 9 sequences
    (6, 4, 4, 128, 35000),      # one
    (7, 16, 2, 128, 40000),     # eight
    (33, 32, 16, 64, 1600),     # 99 for 33
    (50, 16, 16, 64, 1600),     # 150 for 50
    (64, 16, 8, 64, 1600),      # 160 for 64
], ids=lambda s: "x".join(map(str, s)))
def test_dealt_spans_of_ragged_batches(shape):
    """Lengths from one row to a full cache, with the workspace of the asked size and of the least one, and sequences that read nothing."""
    B, Hq, Hkv, d, rows = shape
    c, m, C = 64, 8, 1
    n = (rows - 128) // m * c
    pos = [min(n - 1, (n - 1) * (b + 1) // B + 17 * (b % 3)) for b in range(B)]
    pos[1], pos[B // 2] = 0, 70
    p, q, kc, vc, pos_t, ref, ref_lse = inputs(B, Hq, Hkv, d, n, c, m, C, pos, seed=B)
    compare(f"{shape}", *K.ksa_decode_fwd(p, q, kc, vc, pos_t), ref, ref_lse)
    compare("  least workspace", *K.ksa_decode_fwd(p, q, kc, vc, pos_t, workspace=least_workspace(p)), ref, ref_lse)
    pos_t[2:4] = -1
    o, lse = K.ksa_decode_fwd(p, q, kc, vc, pos_t)
    assert bool(torch.isnan(o[2:4]).all()) and bool(torch.isnan(lse[2:4]).all())
    rest = [b for b in range(B) if b not in (2, 3)]
    compare("  beside invalid ones", o[rest], lse[rest], ref[rest], ref_lse[rest])
