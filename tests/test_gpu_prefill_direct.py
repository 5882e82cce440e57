"""GPU parity of the forward kernel for short key runs and for chunk shapes that are no powers of two
(csrc/ksa_prefill_direct.hip) at the sizes where it can go wrong: query tiles of 1 to 129 rows, key lists that end on and
beside a multiple of 64, tiles that hold the last summaries and the first text rows, chunks of 64 and more rows, every head
stack, and rows so far apart that such mixed tiles are not formed.  Tolerances as in test_gpu_prefill.py."""
import numpy as np
import pytest
import torch

import paper_2604_24432_amd as K
from paper_2604_24432_amd import synth
from oracle import ksa_oracle as O

pytestmark = pytest.mark.gpu

MAX_ABS, MEAN_ABS, LSE_ABS = 2e-2, 2e-3, 4e-3

SHAPES = [
    # B, Hq, Hkv, d, n, c, m, C
    *[(1, 4, 1, 128, n, 12, 3, 1) for n in (1, 11, 12, 31, 33, 64, 129)],
    *[(1, 2, 1, 64, n, 8, 1, 2) for n in (63, 65, 127, 257)],
    (2, 3, 1, 128, 300, 20, 5, 2),          # three heads per group: one head per workgroup
    (1, 8, 1, 128, 700, 48, 6, 2),          # two slices of four heads
    (1, 2, 2, 64, 650, 96, 12, 1),          # chunks longer than a key tile
    (1, 2, 2, 128, 1100, 192, 64, 0),       # ... with summaries that fill one
    (1, 2, 1, 128, 700, 100, 0, 3),         # no summaries
    (1, 4, 2, 128, 1024, 128, 16, 1),       # powers of two: fixed reference
    (3, 2, 1, 128, 515, 1, 0, 70),          # token window
]


def compare(got, ref, what):
    o, lse = (x.float().cpu().numpy().astype(np.float64) for x in got)
    err, lerr = np.abs(o - ref[0]), np.abs(lse - ref[1])
    print(f"{what}: max-abs {err.max():.3e} mean-abs {err.mean():.3e} lse {lerr.max():.3e}", flush=True)
    assert np.isfinite(o).all() and err.max() <= MAX_ABS and err.mean() <= MEAN_ABS and lerr.max() <= LSE_ABS, what


@pytest.mark.parametrize("outliers", [0.0, 0.03])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_edges(shape, outliers):
    B, Hq, Hkv, d, n, c, m, C = shape
    cfg = synth.KsaConfig("direct", B, Hq, Hkv, d, n, c, m, C, seed=n + c, key_outlier_frac=outliers)
    q, k, v = synth.make_prefill_inputs(cfg)
    flags = K.KSA_FLAG_SUMMARY_SELF_ONLY if m > 1 and n % 2 else 0
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, Hq, Hkv, d, flags=flags))
    got = K.ksa_prefill_fwd(lay, q.cuda(), k.cuda(), v.cuda())
    ref = O.prefill(q.float().numpy(), k.float().numpy(), v.float().numpy(), n, c, m, C, flags=flags)
    compare(got, ref, str(shape))


def test_rows_far_apart():
    """K / V rows 8 MiB apart: the rows of a tile across the border of summaries and text are beyond 32-bit offsets."""
    n, c, m, C = 95, 20, 5, 1
    cfg = synth.KsaConfig("far", 1, 2, 1, 64, n, c, m, C, seed=9)
    q, k, v = synth.make_prefill_inputs(cfg)
    stride = 1 << 22
    far = [torch.empty(cfg.aug_len * stride, dtype=torch.bfloat16, device="cuda").as_strided(k.shape, (0, stride, 64, 1)) for _ in "kv"]
    for x, y in zip(far, (k, v)):
        x.copy_(y)
    lay = K.ksa_build_layout(K.make_params(1, n, c, m, C, 2, 1, 64))
    got = K.ksa_prefill_fwd(lay, q.cuda(), *far)
    ref = O.prefill(q.float().numpy(), k.float().numpy(), v.float().numpy(), n, c, m, C)
    compare(got, ref, "rows 8 MiB apart")


@pytest.mark.parametrize("n,c,m,C,d", [(2048, 64, 8, 1, 128), (512, 64, 8, 1, 64), (4096, 8, 1, 32, 128), (1000, 64, 0, 3, 64), (37, 16, 2, 1, 128)])
def test_output_in_the_memory_of_an_input(n, c, m, C, d):
    """o = q and, with chunk shapes that are powers of two, o = v on layouts whose key runs are short."""
    B, H = 2, 4
    cfg = synth.KsaConfig("inplace", B, H, H, d, n, c, m, C, seed=n)
    q, k, v = (x.cuda() for x in synth.make_prefill_inputs(cfg))
    ref = O.prefill(*(x.float().cpu().numpy() for x in (q, k, v)), n, c, m, C)
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, H, H, d))
    x = q.clone()
    compare(K.ksa_prefill_fwd(lay, x, k, v, o=x), ref, "o = q")
    x = v.clone()
    compare(K.ksa_prefill_fwd(lay, q, k, x, o=x), ref, "o = v")


@pytest.mark.parametrize("what,value", [("q", np.nan), ("k", np.nan), ("k", np.inf)])
@pytest.mark.parametrize("shape", [(1, 4, 2, 64, 700, 48, 6, 2), (1, 4, 1, 128, 700, 20, 5, 2), (1, 4, 1, 128, 700, 64, 8, 1), (1, 3, 1, 64, 640, 8, 1, 16)],
                         ids=lambda s: "x".join(map(str, s)))
def test_no_number_reaches_the_rows_that_see_it_alone(shape, what, value):
    """A NaN or an infinity in a query row or a key row: rows that do not see it keep their results."""
    B, Hq, Hkv, d, n, c, m, C = shape
    cfg = synth.KsaConfig("nan", B, Hq, Hkv, d, n, c, m, C, seed=n)
    t = dict(zip("qkv", (x.cuda() for x in synth.make_prefill_inputs(cfg))))
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, Hq, Hkv, d))
    clean, clean_lse = K.ksa_prefill_fwd(lay, t["q"], t["k"], t["v"])
    rows = [20, 45, cfg.aug_len // 2 + 3, cfg.aug_len - 30]
    t[what][:, rows, :, 5] = value
    o, lse = K.ksa_prefill_fwd(lay, t["q"], t["k"], t["v"])
    sees = torch.zeros(cfg.aug_len, dtype=torch.bool)
    if what == "q":
        sees[rows] = True
    else:
        sees = torch.from_numpy(np.stack([lay.mask_row(a)[rows].any() for a in range(cfg.aug_len)]))
    sees = sees.cuda()
    if value != value:
        assert bool(torch.isnan(o[:, sees]).all()) and bool(torch.isnan(lse[:, :, sees]).all())
    assert bool(sees.any()) and not bool(sees.all())
    # against other references a weight is rounded differently: 2^-9 of an output of about 1, twice
    assert (o[:, ~sees].float() - clean[:, ~sees].float()).abs().max() <= MAX_ABS
    assert (lse[:, :, ~sees] - clean_lse[:, :, ~sees]).abs().max() <= LSE_ABS


@pytest.mark.parametrize("shape,bar", [((8, 32, 8, 128, 37, 64, 8, 1), 1.85e-3), ((4, 16, 16, 128, 500, 8, 1, 32), 2.06e-3), ((4, 12, 4, 64, 200, 64, 8, 1), 2.03e-3)],
                         ids=["37", "500", "200"])
def test_short_texts_keep_running_maxima(shape, bar):
    """Rows of few keys: a largest weight of exactly 1 is not rounded, which shows in the error of the whole output.  The bars
    lie halfway between what running maxima and fixed references measured over inputs like these (1.76e-3 / 1.93e-3, 2.00e-3 /
    2.12e-3, 1.94e-3 / 2.11e-3; another seed moves them by less than 0.01e-3)."""
    B, Hq, Hkv, d, n, c, m, C = shape
    cfg = synth.KsaConfig("short", B, Hq, Hkv, d, n, c, m, C, seed=n)
    gen = torch.Generator().manual_seed(n)
    q, k, v = (torch.randn((B, cfg.aug_len, h, d), generator=gen).to(torch.bfloat16) for h in (Hq, Hkv, Hkv))
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, Hq, Hkv, d))
    o, lse = K.ksa_prefill_fwd(lay, q.cuda(), k.cuda(), v.cuda())
    ref, lse_ref = O.prefill(*(x.float().numpy() for x in (q, k, v)), n, c, m, C)
    rel = np.linalg.norm(o.float().cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"{shape}: relative error {rel:.3e}", flush=True)
    assert rel <= bar
    assert np.abs(lse.cpu().numpy() - lse_ref).max() <= 1e-5     # sums of unrounded fp32 weights, values of a few units


def test_summary_rows_whose_chunks_lie_far_apart():
    """One summary per chunk, a query tile of 128 summaries, K / V rows 512 KiB apart: the text of the tile's first chunk and
    its last summary are more than 4 GiB apart (forward and dQ), while the rows of either kind stay within it."""
    B, H, d, n, c, m, C = 1, 4, 128, 8128, 64, 1, 0
    cfg = synth.KsaConfig("far", B, H, H, d, n, c, m, C, seed=3)
    q, k, v = synth.make_prefill_inputs(cfg)
    g = synth.make_upstream_gradient(cfg)
    stride = 1 << 18
    both = torch.empty(cfg.aug_len * stride, dtype=torch.bfloat16, device="cuda")
    kf, vf = (both[at:].as_strided(k.shape, (0, stride, d, 1)) for at in (0, H * d))
    kf.copy_(k), vf.copy_(v)
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, H, H, d))
    o, lse = K.ksa_prefill_fwd(lay, q.cuda(), kf, vf)
    dq, dk, dv = (torch.empty_like(x, device="cuda") for x in (q, k, v))
    K.ksa_prefill_bwd(lay, q.cuda(), kf, vf, o, lse, g.cuda(), dq=dq, dk=dk, dv=dv)
    near = K.ksa_prefill_fwd(lay, q.cuda(), k.cuda(), v.cuda())
    grads = K.ksa_prefill_bwd(lay, q.cuda(), k.cuda(), v.cuda(), *near, g.cuda())
    rows = np.concatenate([np.arange(64, 8255, 65), np.arange(100, 140)])      # every summary, some text
    ref = O.prefill(*(x.float().numpy() for x in (q, k, v)), n, c, m, C, rows=rows)
    compare((o[:, rows], lse[:, :, rows]), ref, "summaries 4 GiB behind their tile's text")
    # contiguous tensors: the same up to the order of the keys in a list (weights against another reference, one bf16
    # rounding of the result: 2^-9 each)
    for x, y in ((o, near[0]), (dq, grads[0]), (dk, grads[1]), (dv, grads[2])):
        assert (x.float() - y.float()).norm() <= 5e-3 * y.float().norm()


@pytest.mark.parametrize("n,c,m,C", [(64, 1, 0, 63), (64 * 254, 1, 0, 63), (64 * 254 + 1, 1, 0, 63), (64 * 255, 1, 0, 63), (128 * 254 - 127, 1, 0, 63),
                                     (14464, 64, 8, 1), (14464 + 64, 64, 8, 1), (32768, 128, 1, 1), (50048, 64, 1, 2)])
def test_norm_parts(n, c, m, C):
    """The largest K row norm of a head is found wherever that row is: first and last rows of both spaces and of the parts
    that the norms are kept in, below and above one key tile per part.  Whole-numbered keys: the norm is exact."""
    d, n_chunks = 64, n // c
    lay = K.ksa_build_layout(K.make_params(1, n, c, m, C, 1, 1, d))
    L = lay.aug_len
    nt, ns = -(-n // 64), -(-n_chunks * m // 64)
    run = max(1, -(-(nt + ns) // 254))
    text = {0, n - 1, min(64 * run, n) - 1, min(64 * run, n - 1), (nt - 1) // run * run * 64}
    rows = [t + t // c * m for t in text] + [u + (u // m + 1) * c for u in ({0, n_chunks * m - 1, (ns - 1) // run * run * 64} if m else ())]
    ws = torch.empty(K.prefill_workspace_bytes(lay), dtype=torch.uint8, device="cuda")
    at = 2 * d * 64 * (nt + ns) + 4 * (nt + ns)     # behind the key-major V and the norms of the parts
    q, v = torch.zeros(1, L, 1, d, dtype=torch.bfloat16, device="cuda"), torch.ones(1, L, 1, d, dtype=torch.bfloat16, device="cuda")
    for row in rows:
        k = torch.ones_like(v)
        k[0, row, 0, 1] = 16
        o, _ = K.ksa_prefill_fwd(lay, q, k, v, workspace=ws)
        assert ws[at:at + 4].view(torch.float32).item() == d - 1 + 256, row
        assert bool((o == 1).all())
