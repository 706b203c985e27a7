"""Layers whose backward just fits the 64 MiB of ssdt_layer_bwd_static stay servable: what the kernels take for speed only
(partial products of split contractions, finer chunks of column sums) must not push them over the edge, nor make a workspace
too small that holds everything else."""
import pytest
import torch

from paper_2408_10013_amd import binding as sb
from paper_2408_10013_amd import runner

import helpers as hp
from test_gpu_layer import check_against_oracle

GPT = dict(arch="gpt_preln", act="gelu", norm="layernorm", mask="causal", has_bias=True, eps=1e-5)
BERT = dict(arch="bert_postln", act="gelu", norm="layernorm", mask="keypad", has_bias=True, eps=1e-5)
T5_ENC = dict(arch="t5_enc", act="relu", norm="rmsnorm", mask="none", has_bias=False, eps=1e-6)
T5_DEC = dict(arch="t5_dec", act="relu", norm="rmsnorm", mask="causal", has_bias=False, eps=1e-6)
EDGE = [
    dict(T5_ENC, dtype="f32", B=14, S=128, H=920, A=23, F=3680),
    dict(T5_ENC, dtype="f32", B=4, S=1141, H=360, A=9, F=1440),
    dict(T5_DEC, dtype="f32", B=12, S=37, S_kv=187, H=1544, A=193, F=3856),
    dict(T5_DEC, dtype="bf16", B=2, S=1408, S_kv=40, H=768, A=6, F=3072),
    dict(BERT, dtype="bf16", B=3, S=446, H=1960, A=49, F=4896),
    dict(GPT, dtype="bf16", B=16, S=128, H=1056, A=66, F=4224),
]


@pytest.mark.parametrize("case", EDGE, ids=lambda c: "%s_%s_%d" % (c["arch"], c["dtype"], c["H"]))
def test_backward_workspace_stays_within_the_static_one(case):
    _, bwd = sb.ssdt_layer_workspace(runner.Layer(**case).desc)
    assert bwd <= 64 << 20


def test_no_room_is_reported_for_splits_that_do_not_happen():
    """2 x 128 tokens, H 256: no product is split (buffers, column sums and, for operands that are not aligned, a transposed copy)."""
    l = runner.Layer(**dict(GPT, dtype="bf16", B=2, S=128, H=256, A=2, F=1024))
    assert sb.ssdt_layer_workspace(l.desc)[1] == 1986816


# Layers whose backward is split further if the workspace has room for it, and the bytes that it takes without
SMALL = [
    (dict(GPT, dtype="bf16", B=32, S=128, H=256, A=2, F=1024), 31784960),
    (dict(T5_DEC, act="gelu", dtype="bf16", B=32, S=128, S_kv=100, H=256, A=4, F=1024), 36765696),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case,nbytes", SMALL, ids=lambda c: c["arch"] if isinstance(c, dict) else "")
def test_backward_takes_a_workspace_without_room_for_partial_products(case, nbytes):
    l = runner.Layer(**case)
    assert sb.ssdt_layer_workspace(l.desc)[1] > nbytes
    c = hp.make_layer_case(l, 8800 + l.H, bias_std=0.05)
    st = runner.Stack([l], 3 * runner.saved_bytes_per_layer(l) + (1 << 20), 0, "cuda:0", budget_bytes=0)
    hp.load_weights(l, c["w"], st.dev)
    x, dy = (runner.to_device(c[k], l.dtype, st.dev) for k in ("x", "dy"))
    enc = runner.to_device(c["enc"], l.dtype, st.dev) if "enc" in c else None
    d_enc = torch.zeros_like(enc) if enc is not None else None
    ptr = lambda t: t.data_ptr() if t is not None else 0
    guard = torch.full((nbytes + 4096,), 0xA5, dtype=torch.uint8, device=st.dev)
    assert guard.data_ptr() % 256 == 0
    dx = torch.empty_like(dy)
    sb.ssdt_step_begin(st.ctx, 1)
    y, saved = sb.ssdt_layer_fwd(st.ctx, l.desc, l.wstruct, 0, x.data_ptr(), ptr(enc), 0, st.ws_ptr, st.ws_bytes, st.stream)
    sb.ssdt_layer_bwd(st.ctx, l.desc, l.wstruct, saved, 0, dy.data_ptr(), dx.data_ptr(), ptr(d_enc), l.gstruct, st.ws_ptr, st.ws_bytes,
                      st.stream)
    with_room = {k: v.clone() for k, v in l.g.items()}
    if d_enc is not None:
        d_enc.zero_()
    sb.ssdt_layer_bwd(st.ctx, l.desc, l.wstruct, saved, 0, dy.data_ptr(), dx.data_ptr(), ptr(d_enc), l.gstruct, guard.data_ptr(),
                      nbytes, st.stream)
    torch.cuda.synchronize()
    assert bool((guard[nbytes:] == 0xA5).all())
    assert any(not torch.equal(with_room[k], v) for k, v in l.g.items())     # (the other order of additions)
    res = dict(y=runner.to_host(st.view(y, (l.T, l.H))), dx=dx, d_enc=d_enc, grads=l.g)
    st.close()
    check_against_oracle(l, c, res, hp.TOL[l.dtype])
