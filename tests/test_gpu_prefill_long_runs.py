"""GPU parity of the kernels for long key runs: ksa_prefill_kernel (forward) and ksa_bwd_dq_kernel (dense causal dQ), on layouts
that are past the lines of takes_direct() and dq_takes_direct() (csrc/ksa_layout.cpp): every head stack, both summary rules,
strided tensors, waves with a fixed and with a running softmax reference side by side, values of extreme magnitude, chunk
lengths that are no powers of two (backward).  Sampled rows against the oracle; bars of test_gpu_prefill.py and
test_gpu_prefill_bwd_split.py."""
import numpy as np
import pytest
import torch

import paper_2604_24432_amd as K
from paper_2604_24432_amd import synth
from oracle import ksa_oracle as O

pytestmark = pytest.mark.gpu

MAX_ABS, MEAN_ABS, LSE_ABS = 2e-2, 2e-3, 4e-3
SELF = K.KSA_FLAG_SUMMARY_SELF_ONLY

FORWARD = [
    # B, Hq, Hkv, d, n, c, m, C, flags
    (1, 2, 2, 128, 8192, 64, 0, 4096, 0),        # one head per workgroup
    (1, 2, 2, 128, 12032, 64, 8, 128, 0),
    (1, 2, 2, 128, 12032, 64, 8, 128, SELF),
    (1, 2, 1, 128, 12032, 64, 8, 128, SELF),     # two
    (2, 4, 1, 128, 12032, 64, 8, 128, SELF),     # four
    (1, 4, 1, 64, 12032, 64, 8, 128, 0),
    (1, 1, 1, 128, 12011, 8, 1, 1024, 0),        # the last run of either space ends inside a key tile
]


def wide(x, extra):
    """x as the middle heads of a tensor with `extra` more heads on either side."""
    B, L, H, d = x.shape
    t = torch.zeros((B, L, H + 2 * extra, d), dtype=x.dtype, device="cuda")
    t[:, :, extra:extra + H] = x
    return t[:, :, extra:extra + H]


def mean_tiles(lay):
    """Key tiles per query tile of the launch order."""
    pairs = lay.tile_pairs()
    return len(pairs["kind"]) / len(set(zip(pairs["q_space"].tolist(), pairs["q_begin"].tolist())))


@pytest.mark.parametrize("inputs", ["plain", "strided", "mixed references", "V x 2^70", "V x 2^-30"])
@pytest.mark.parametrize("shape", FORWARD, ids=lambda s: "x".join(map(str, s)))
def test_forward(shape, inputs):
    B, Hq, Hkv, d, n, c, m, C, flags = shape
    cfg = synth.KsaConfig("long", B, Hq, Hkv, d, n, c, m, C, seed=n + Hq)
    q, k, v = synth.make_prefill_inputs(cfg)
    f = 2.0 ** int(inputs.split("^")[1]) if "^" in inputs else 1.0
    if inputs == "mixed references":     # a bound of about 80 in the exponent domain, above the limit of 60
        q[:, :, 1::2] *= 4
        q[:, cfg.aug_len // 2:, ::2] *= 4
    lay = K.ksa_build_layout(K.make_params(B, n, c, m, C, Hq, Hkv, d, flags=flags))
    ws = torch.full((K.prefill_workspace_bytes(lay),), 255, dtype=torch.uint8, device="cuda")
    dev = [x.cuda() for x in (q, k, v * f)]
    o = torch.empty_like(dev[0])
    if inputs == "strided":
        both = torch.zeros((B, cfg.aug_len, 2 * Hkv + 1, d), dtype=torch.bfloat16, device="cuda")
        both[:, :, :Hkv], both[:, :, Hkv + 1:] = dev[1], dev[2]
        dev, o = [wide(dev[0], 1), both[:, :, :Hkv], both[:, :, Hkv + 1:]], wide(o, 2)
    o, lse = K.ksa_prefill_fwd(lay, *dev, o=o, workspace=ws)
    # this kernel alone writes the key-major copy of V, which comes first in the workspace
    assert bool((ws[:2 * d * 64] != 255).any())
    again, lse_again = K.ksa_prefill_fwd(lay, *dev, workspace=ws)
    assert torch.equal(o, again) and torch.equal(lse, lse_again)
    rows = np.unique(np.concatenate([np.arange(40), np.arange(cfg.aug_len - 40, cfg.aug_len),
                                     np.random.default_rng(n).integers(0, cfg.aug_len, 60)]))
    ref, lse_ref = O.prefill(q.float().numpy(), k.float().numpy(), v.float().numpy(), n, c, m, C, flags=flags, rows=rows)
    got = o[:, rows].float().cpu().numpy().astype(np.float64) / f
    err, lerr = np.abs(got - ref), np.abs(lse.cpu().numpy()[:, :, rows] - lse_ref)
    print(f"{shape} {inputs}: max-abs {err.max():.3e} mean-abs {err.mean():.3e} lse {lerr.max():.3e}", flush=True)
    assert np.isfinite(got).all() and err.max() <= MAX_ABS and err.mean() <= MEAN_ABS and lerr.max() <= LSE_ABS


@pytest.mark.parametrize("what,value", [("q", np.nan), ("k", np.nan), ("k", np.inf)])
@pytest.mark.parametrize("shape", [(4, 1, 128, 5003, 64, 0, 4096), (2, 2, 128, 12032, 64, 8, 128), (4, 1, 64, 8192, 64, 0, 4096)],
                         ids=lambda s: "x".join(map(str, s)))
def test_no_number_reaches_the_rows_that_see_it_alone(shape, what, value):
    """A NaN or an infinity in a query row or a key row: rows that do not see it keep their results."""
    Hq, Hkv, d, n, c, m, C = shape
    cfg = synth.KsaConfig("nan", 1, Hq, Hkv, d, n, c, m, C, seed=n)
    t = dict(zip("qkv", (x.cuda() for x in synth.make_prefill_inputs(cfg))))
    lay = K.ksa_build_layout(K.make_params(1, n, c, m, C, Hq, Hkv, d))
    ws = torch.full((K.prefill_workspace_bytes(lay),), 255, dtype=torch.uint8, device="cuda")
    clean, clean_lse = K.ksa_prefill_fwd(lay, t["q"], t["k"], t["v"], workspace=ws)
    assert bool((ws[:2 * d * 64] != 255).any())
    rows = [1500, cfg.aug_len // 2 + 3, cfg.aug_len - 30] + ([cfg.aug_len - 5] if what == "q" else [])
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


BACKWARD = [
    # B, Hq, Hkv, n, c, C: head_dim 128, no summaries, more than 48 key tiles per query tile
    (1, 4, 1, 6500, 64, 4096),
    (1, 2, 1, 6500, 100, 100),
    (1, 1, 1, 6655, 6655, 0),
    (2, 3, 1, 6401, 48, 200),
    (1, 4, 2, 10001, 1, 4000),       # both ends of a row's keys move
]


@pytest.mark.parametrize("strided", [False, True], ids=["dense", "strided"])
@pytest.mark.parametrize("shape", BACKWARD, ids=lambda s: "x".join(map(str, s)))
def test_backward(shape, strided):
    B, Hq, Hkv, n, c, C = shape
    cfg = synth.KsaConfig("causal", B, Hq, Hkv, 128, n, c, 0, C, seed=n)
    host = [*synth.make_prefill_inputs(cfg), synth.make_upstream_gradient(cfg)]
    q, k, v, g = (x.cuda() for x in host)
    lay = K.ksa_build_layout(K.make_params(B, n, c, 0, C, Hq, Hkv, 128))
    assert mean_tiles(lay) > 48
    dq = torch.empty_like(q)
    if strided:
        both = torch.cat([k, k[:, :, :1], v], 2)
        q, k, v, dq = wide(q, 1), both[:, :, :Hkv], both[:, :, Hkv + 1:], wide(dq, 2)
    o, lse = K.ksa_prefill_fwd(lay, q, k, v, o=torch.empty_like(g))
    got = K.ksa_prefill_bwd(lay, q, k, v, o, lse, g, dq=dq)
    rows = np.unique(np.concatenate([np.arange(0, n, 131), np.arange(n - 70, n)]))
    ref = O.prefill_bwd(*(x.float().numpy() for x in host), n, c, 0, C, q_rows=rows, k_rows=rows)
    for name, x, r in zip(("dq", "dk", "dv"), got, ref):
        rel = np.linalg.norm(x[:, rows].float().cpu().numpy() - r) / np.linalg.norm(r)
        print(f"{shape} {name}: relative error {rel:.2e}", flush=True)
        assert rel <= 5e-3, name
