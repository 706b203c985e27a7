"""Infinities and NaN reach only what depends on them.  A query sees no key behind its mask, so what a masked key, or a
query that a key does not answer to, holds must not show, neither in the output nor in a gradient.  (Matrix cores multiply
masked entries by a probability of zero, and zero times infinity is NaN.)  fp32 of any size, bf16 of any but whole
tiles (head size 64 or 128, sequence lengths multiples of 128).

The clean part of a result is compared with that of the same call without the bad values; the ordinary bars apply, as the
rows in question may be computed in another order then."""
import numpy as np
import pytest
import torch

from paper_2408_10013_amd import binding as sb
from paper_2408_10013_amd import runner

import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

GPT = dict(arch="gpt_preln", act="gelu", norm="layernorm", mask="causal", has_bias=True, eps=1e-5)
BERT = dict(GPT, arch="bert_postln", mask="keypad")
T5 = dict(arch="t5_dec", act="gelu", norm="rmsnorm", mask="causal", has_bias=False, eps=1e-6)
CAUSAL = {
    "f32_d32": dict(GPT, dtype="f32", B=2, S=70, H=64, A=2, F=64),
    "f32_d64": dict(GPT, dtype="f32", B=2, S=128, H=128, A=2, F=64),
    "f32_d96": dict(GPT, dtype="f32", B=2, S=150, H=96, A=1, F=64),
    "f32_d128": dict(GPT, dtype="f32", B=2, S=200, H=128, A=1, F=64),
    "f32_rows": dict(GPT, dtype="f32", B=2, S=30, H=64, A=1, F=64),
    "bf16_d32": dict(GPT, dtype="bf16", B=2, S=70, H=64, A=2, F=64),
    "bf16_d64": dict(GPT, dtype="bf16", B=2, S=200, H=128, A=2, F=64),
    "bf16_d96": dict(GPT, dtype="bf16", B=2, S=128, H=96, A=1, F=64),
    "bf16_d128": dict(GPT, dtype="bf16", B=2, S=161, H=256, A=2, F=64),
    "bf16_relu": dict(GPT, dtype="bf16", act="relu", B=2, S=100, H=128, A=2, F=64),
    "bf16_d36": dict(GPT, dtype="bf16", B=2, S=40, H=72, A=2, F=64),
}
KEYPAD = {
    "f32_d64": dict(BERT, dtype="f32", B=2, S=150, H=128, A=2, F=64),
    "f32_d128": dict(BERT, dtype="f32", B=2, S=150, H=128, A=1, F=64),
    "bf16_d64": dict(BERT, dtype="bf16", B=2, S=150, H=128, A=2, F=64),
    "bf16_d96": dict(BERT, dtype="bf16", B=2, S=150, H=96, A=1, F=64),
    "bf16_d128": dict(BERT, dtype="bf16", B=2, S=150, H=128, A=1, F=64),
}


def run(l, case, x=None, dy=None):
    """y, lse, dx and the gradients of q, k, v of one layer, as fp32 arrays [B, S, ...]."""
    st = runner.Stack([l], 3 * runner.saved_bytes_per_layer(l) + (1 << 20), 0, DEV, budget_bytes=0)
    hp.load_weights(l, case["w"], st.dev)
    st.register_weights()
    x = runner.to_device(case["x"] if x is None else x, l.dtype, st.dev)
    dy = runner.to_device(case["dy"] if dy is None else dy, l.dtype, st.dev)
    kv = torch.from_numpy(case["kv_len"]).to(st.dev) if "kv_len" in case else None
    kvp = kv.data_ptr() if kv is not None else 0
    sb.ssdt_step_begin(st.ctx, 1)
    y, saved = sb.ssdt_layer_fwd(st.ctx, l.desc, l.wstruct, 0, x.data_ptr(), 0, kvp, st.ws_ptr, st.ws_bytes, st.stream)
    dx = torch.empty_like(dy)
    sb.ssdt_layer_bwd(st.ctx, l.desc, l.wstruct, saved, kvp, dy.data_ptr(), dx.data_ptr(), 0, l.gstruct, st.ws_ptr,
                      st.ws_bytes, st.stream)
    torch.cuda.synchronize()
    off = st.ws_ptr - st.ws.data_ptr() + sb.ssdt_layer_bwd_temporaries(l.desc)["d_qkv"]
    d_qkv = st.ws[off:off + 3 * dx.numel() * dx.element_size()].view(dx.dtype)
    lse = saved.e[sb.SV_NAMES.index("lse")].ptr
    out = dict(y=runner.to_host(st.view(y, (l.B, l.S, l.H))), dx=runner.to_host(dx).reshape(l.B, l.S, l.H),
               lse=runner.to_host(st.view(lse, (l.B, l.A, l.S), torch.float32)),
               d_qkv=runner.to_host(d_qkv).reshape(l.B, l.S, 3 * l.H))
    st.close()
    return out


def close(got, ref, dtype):
    bad = int((~np.isfinite(ref)).sum()), int((~np.isfinite(got)).sum())
    assert bad == (0, 0), "values that are not finite: %d of the clean run, %d of %d" % (*bad, got.size)
    assert hp.rel_err(got, ref) <= hp.TOL[dtype]


def layer_of(v):
    l = runner.Layer(**v)
    case = hp.make_layer_case(l, 9100 + l.H + l.S, bias_std=0.05, kv_len_range=(40, 75) if v["mask"] == "keypad" else None)
    return l, case


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", list(CAUSAL))
def test_a_bad_token_does_not_reach_earlier_ones(name, bad):
    l, case = layer_of(CAUSAL[name])
    clean = run(l, case)
    for k in sorted({l.S - 1, l.S // 2 + 3, 5}):
        x = case["x"].copy()
        x[k] = bad          # token k of the first sequence
        got = run(l, case, x=x)
        close(got["y"][0, :k], clean["y"][0, :k], l.dtype)
        close(got["y"][1], clean["y"][1], l.dtype)
        close(got["lse"][0, :, :k], clean["lse"][0, :, :k], l.dtype)
        assert bool(np.isnan(got["y"][0, k:]).all())
        # the queries' gradients before it (those of keys and values do depend on the bad queries behind them)
        close(got["d_qkv"][0, :k, :l.H], clean["d_qkv"][0, :k, :l.H], l.dtype)
        close(got["dx"][1], clean["dx"][1], l.dtype)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", list(CAUSAL))
def test_a_bad_output_gradient_does_not_reach_later_tokens(name, bad):
    l, case = layer_of(CAUSAL[name])
    clean = run(l, case)
    for k in sorted({0, l.S // 2 + 3, l.S - 2}):
        dy = case["dy"].copy()
        dy[k] = bad
        got = run(l, case, dy=dy)
        close(got["d_qkv"][0, k + 1:], clean["d_qkv"][0, k + 1:], l.dtype)
        close(got["dx"][0, k + 1:], clean["dx"][0, k + 1:], l.dtype)
        close(got["dx"][1], clean["dx"][1], l.dtype)
        assert bool(np.isnan(got["dx"][0, k]).all())


@pytest.mark.parametrize("name", list(KEYPAD))
def test_padded_keys_have_no_gradient_even_from_bad_queries(name):
    l, case = layer_of(KEYPAD[name])
    clean = run(l, case)
    n = int(case["kv_len"][0])
    x = case["x"].copy()
    x[3] = float("nan")
    got = run(l, case, x=x)
    assert int(np.count_nonzero(got["d_qkv"][0, n:, l.H:])) == 0     # exact zeros for keys and values
    close(got["y"][1], clean["y"][1], l.dtype)
    close(got["dx"][1], clean["dx"][1], l.dtype)


@pytest.mark.parametrize("name", ["f32_d64", "bf16_d64", "bf16_d128"])
def test_an_infinite_value_reaches_its_own_queries_as_itself(name):
    """One element of V is +inf.  The outputs that see it are +inf in its column (no probability is zero); earlier queries
    and all other columns stay finite."""
    l, case = layer_of(dict(CAUSAL[name], B=1))
    st = runner.Stack([l], 3 * runner.saved_bytes_per_layer(l) + (1 << 20), 0, DEV, budget_bytes=0)
    hp.load_weights(l, case["w"], st.dev)
    # column 7 of the first head's V is input feature 3, scaled so that only token k, where this feature stands out, overflows
    col, k = 2 * l.H + 7, l.S // 2
    l.w["w_qkv"][:, col] = 0
    l.w["w_qkv"][3, col] = 8e37
    l.w["b_qkv"][col] = l.w["ln1_b"][3] = 0
    l.w["ln1_g"][3] = 1
    x = runner.to_device(case["x"], l.dtype, st.dev)
    x[:, 3] = x.float().mean(1).to(x.dtype)      # next to zero after the norm
    x[k] = 0
    x[k, 3] = 100                                # sqrt(H - 1) after the norm, 11 and more
    sb.ssdt_step_begin(st.ctx, 1)
    _, saved = sb.ssdt_layer_fwd(st.ctx, l.desc, l.wstruct, 0, x.data_ptr(), 0, 0, st.ws_ptr, st.ws_bytes, st.stream)
    torch.cuda.synchronize()
    o = st.view(saved.e[sb.SV_NAMES.index("o")].ptr, (l.S, l.H)).float()
    v = st.view(saved.e[sb.SV_NAMES.index("qkv")].ptr, (l.S, 3 * l.H)).float()[:, col]
    assert torch.isposinf(v[k]) and torch.isfinite(v).sum() == l.S - 1
    assert torch.isposinf(o[k:, 7]).all()
    o[k:, 7] = 0
    assert torch.isfinite(o).all()
    st.close()


@pytest.mark.parametrize("B,S,H,F", [(1, 40, 64, 64), (3, 100, 64, 128), (2, 197, 256, 1024)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_an_infinite_output_gradient_makes_its_bias_gradient_infinite(dtype, B, S, H, F):
    """The bias gradient of the last product is the column sum of dy: infinite, and not NaN, in the one column that holds an
    infinity, whatever row it is in."""
    l = runner.Layer(dtype=dtype, **GPT, B=B, S=S, H=H, A=H // 64, F=F)
    case = hp.make_layer_case(l, 9300 + H, bias_std=0.05)
    for row in (0, 17, B * S - 1):
        dy = case["dy"].copy()
        dy[row, 5] = float("-inf")
        run(l, case, dy=dy)
        db = runner.to_host(l.g["b_2"])
        assert bool(np.isneginf(db[5])), db[5]
        ref = case["dy"].astype(np.float64).sum(0)
        assert hp.rel_err(np.delete(db, 5), np.delete(ref, 5)) <= hp.TOL[dtype]
