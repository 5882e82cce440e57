"""The calls of the decode loop look at their arguments in few steps and only then one by one: what was refused stays refused, with
the same kind of error, and what is unusual but allowed (views with strides of their own, a batch of one) still runs."""
import pytest
import torch

import paper_2604_24432_amd as K

pytestmark = pytest.mark.gpu

B, HQ, HKV, D, N, C, M, W = 2, 4, 2, 64, 256, 16, 2, 1


def call(kind, **change):
    p = change.pop("params", None) or K.make_params(B, N, C, M, W, HQ, HKV, D)
    rows = N // C * M + (W + 1) * C
    gen = torch.Generator(device="cuda").manual_seed(3)
    t = {n: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16) for n, s in
         (("q", (B, HQ, D)), ("k_cache", (B, HKV, rows, D)), ("v_cache", (B, HKV, rows, D)), ("k_new", (B, HKV, D)), ("v_new", (B, HKV, D)))}
    t["pos"] = torch.tensor([N - 1, 40] if kind != "summary" else [3, 7], dtype=torch.int32, device="cuda")
    for name, f in change.items():
        t[name] = f(t[name])
    if kind == "append":
        K.ksa_cache_append(p, K.KSA_ROW_TEXT, t["k_new"], t["v_new"], t["pos"], t["k_cache"], t["v_cache"])
        return t["k_cache"].clone(), t["v_cache"].clone()
    return (K.ksa_decode_fwd if kind == "text" else K.ksa_decode_summary_fwd)(p, t["q"], t["k_cache"], t["v_cache"], t["pos"])


WRONG = [dict(k_cache=lambda t: t.cpu()), dict(k_cache=lambda t: t.float()), dict(v_cache=lambda t: t[:, :, :-1]), dict(pos=lambda t: t.long()),
         dict(pos=lambda t: t[:1]), dict(pos=lambda t: t.repeat_interleave(2)[::2]), dict(k_cache=lambda t: t.transpose(2, 3)),
         dict(v_cache=lambda t: t.transpose(0, 1).contiguous().transpose(0, 1)), dict(k_cache=lambda t: t.float().cpu().numpy()),
         dict(k_cache=lambda t: t.view(B, HKV, -1))]


@pytest.mark.parametrize("kind", ["text", "summary", "append"])
@pytest.mark.parametrize("change", WRONG, ids=lambda c: next(iter(c)))
def test_wrong_arguments_are_refused(kind, change):
    with pytest.raises(ValueError):
        call(kind, **change)


@pytest.mark.parametrize("change", [dict(q=lambda t: t[:, :2]), dict(q=lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)), dict(q=lambda t: t.half())],
                         ids=["heads", "strides", "dtype"])
def test_wrong_queries_are_refused(change):
    with pytest.raises(ValueError):
        call("text", **change)


@pytest.mark.parametrize("change", [dict(k_new=lambda t: t[:1]), dict(v_new=lambda t: t.transpose(0, 1).contiguous().transpose(0, 1))], ids=["batch", "strides"])
def test_wrong_rows_are_refused(change):
    with pytest.raises(ValueError):
        call("append", **change)


@pytest.mark.parametrize("kind", ["text", "summary", "append"])
@pytest.mark.parametrize("fields", [dict(chunk_len=0), dict(chunk_len=-16), dict(n_q_heads=3), dict(batch=0)], ids=lambda f: next(iter(f)))
def test_parameters_that_make_no_sense_are_reported(kind, fields):
    p = K.make_params(B, N, C, M, W, HQ, HKV, D)
    for name, value in fields.items():
        setattr(p, name, value)
    with pytest.raises(K.KsaError, match="ksa_cache_geometry"):
        call(kind, params=p)


@pytest.mark.parametrize("kind", ["text", "summary", "append"])
def test_views_with_strides_of_their_own(kind):
    """Caches that are every other row of a larger tensor: same results as from dense ones."""
    wide = lambda t: torch.stack([t, t + 1], 3).flatten(2, 3)[:, :, ::2]
    for a, b in zip(call(kind), call(kind, k_cache=wide, v_cache=wide)):
        assert torch.equal(a, b)
