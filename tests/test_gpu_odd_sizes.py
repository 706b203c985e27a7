"""The kernels that take any size, at the edges of their tiles: forward and backward of small layers against the CPU
checker.  bf16 widths that are multiples of 8 go through the matrix-core GEMM with 64- and 128-wide tiles, 64-deep
stages and a split contraction."""
import pytest
import torch

from paper_2408_10013_amd import binding as sb
from paper_2408_10013_amd import runner, synth

import helpers as hp
from test_gpu_layer import check_against_oracle, run_single_layer

pytestmark = pytest.mark.gpu

GPT = dict(arch="gpt_preln", act="gelu", norm="layernorm", mask="causal", has_bias=True, eps=1e-5)

SIZES = {
    "one_token": dict(B=1, S=1, H=64, A=1, F=64),                # a single row; contraction over one token
    "tile_less_one": dict(B=1, S=127, H=64, A=1, F=136),         # last row / column of a tile missing
    "tile_plus_one": dict(B=1, S=129, H=64, A=1, F=264),         # a tile with one row
    "stage_tail": dict(B=3, S=43, H=72, A=3, F=200),             # K = 72, 200, 129: tails of 8, 8 and 1 behind whole stages
    "narrow": dict(B=2, S=65, H=8, A=1, F=8),                    # one 16-byte chunk per row
    "split_k": dict(B=1, S=40, H=64, A=1, F=2048),               # 32 stages on one tile: contraction split
    "split_tokens": dict(B=5, S=333, H=64, A=1, F=128),          # 27 stages over tokens (the last one short), split, bias sums
}

BERT = dict(GPT, arch="bert_postln", mask="keypad")
T5 = dict(arch="t5_dec", act="gelu", norm="rmsnorm", mask="causal", has_bias=False, eps=1e-6)
# attention: sequence lengths around its tiles of 64 and 128, every padded head size, all three masks
HEADS = {
    "causal_d8": dict(GPT, B=2, S=129, H=24, A=3, F=32),
    "causal_d32": dict(GPT, B=1, S=191, H=64, A=2, F=64),
    "causal_d64": dict(GPT, B=2, S=65, H=128, A=2, F=64),
    "causal_d72": dict(GPT, B=1, S=257, H=144, A=2, F=64),
    "causal_d96_whole": dict(GPT, B=1, S=128, H=96, A=1, F=64),
    "causal_d128": dict(GPT, B=1, S=385, H=128, A=1, F=64),
    "keypad_d64": dict(BERT, B=3, S=200, H=64, A=1, F=64),
    "keypad_d128": dict(BERT, B=2, S=127, H=256, A=2, F=64),
    "cross_d40": dict(T5, B=2, S=3, S_kv=131, H=80, A=2, F=64),
    "cross_d128": dict(T5, B=1, S=130, S_kv=63, H=128, A=1, F=64),
    "causal_d104": dict(GPT, B=1, S=33, H=104, A=1, F=64),
    "keypad_d120": dict(BERT, B=3, S=161, H=240, A=2, F=64),
    "cross_d112": dict(T5, B=2, S=31, S_kv=129, H=112, A=1, F=64),
    "cross_d12": dict(T5, B=2, S=37, S_kv=21, H=36, A=3, F=52),   # bf16, ReLU: K-contiguous rows element by element
    "cross_d18": dict(T5, B=1, S=40, S_kv=70, H=54, A=3, F=64),   # a head size that is no multiple of 4
    # bf16: where the row kernels take over, on either side of the lines
    "causal_5_tokens": dict(GPT, B=64, S=5, H=64, A=8, F=32),
    "causal_6_tokens": dict(GPT, B=64, S=6, H=64, A=8, F=32),
    "cross_1_of_32": dict(T5, B=64, S=1, S_kv=32, H=128, A=16, F=32),
    "cross_1_of_33": dict(T5, B=64, S=1, S_kv=33, H=128, A=16, F=32),
    "cross_4_of_16": dict(T5, B=64, S=4, S_kv=16, H=128, A=16, F=32),
    "cross_5_of_16": dict(T5, B=64, S=5, S_kv=16, H=128, A=16, F=32),
    "cross_d64_heads8": dict(T5, B=2, S=150, S_kv=300, H=256, A=4, F=64),
}


@pytest.mark.parametrize("name", list(HEADS))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_of_any_length_and_head_size(name, dtype):
    v = HEADS[name]
    l = runner.Layer(dtype=dtype, **v)
    case = hp.make_layer_case(l, 8000 + len(name), bias_std=0.05, kv_len_range=(1, v["S"]) if v["mask"] == "keypad" else None)
    if v["mask"] == "keypad":
        case["kv_len"][-1] = 0     # a sequence without keys
    on = run_single_layer(l, case, offload=True, fetch=False)
    check_against_oracle(l, case, on, hp.TOL[dtype])


@pytest.mark.parametrize("name", list(SIZES))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_edges_of_tiles(name, dtype):
    l = runner.Layer(dtype=dtype, **GPT, **SIZES[name])
    case = hp.make_layer_case(l, 7000 + len(name), bias_std=0.05)
    # Saved tensors are not compared one by one: with a single row the mean of that row is one number, which the bf16
    # rounding of the row moves by up to 2^-9 times the largest value however close to zero it is, so it has no relative
    # bar of its own.  The output and every gradient depend on all of them.
    on = run_single_layer(l, case, offload=True, fetch=False)
    check_against_oracle(l, case, on, hp.TOL[dtype])


PRECISE = {
    "d32": dict(GPT, B=2, S=333, H=128, A=4, F=64),
    "d64": dict(BERT, B=2, S=333, H=128, A=2, F=64),
    "d96": dict(GPT, B=2, S=200, H=192, A=2, F=64),
    "d128": dict(GPT, B=2, S=300, H=256, A=2, F=64),
    "d64_cross_lengths": dict(GPT, mask="none", B=3, S=150, H=128, A=2, F=64),
}


@pytest.mark.parametrize("name", list(PRECISE))
def test_probabilities_enter_the_products_in_fp32(name):
    """bf16 attention of any size: outputs and value gradients against 64 bits, from the very q, k, v and dO that the kernels
    read.  Inputs exact, probabilities and sums in fp32: an output can only miss the correctly rounded bf16 where the exact
    value lies within its fp32 error of a rounding boundary.  Exponents of up to 16 are rounded to 2^-20, boundaries are 2^-8
    of a value apart: 2 x 2^-20 / 2^-8 = 0.05 % of the outputs (0.02 to 0.06 % measured).  Twice that is the bar;
    probabilities rounded to 16 bits give 0.2 %, to bf16 30 %."""
    l = runner.Layer(dtype="bf16", **PRECISE[name])
    case = hp.make_layer_case(l, 8500 + l.H, bias_std=0.05, kv_len_range=(l.S // 2, l.S) if l.mask == "keypad" else None)
    case["w"]["w_qkv"] = synth.bf16_round(case["w"]["w_qkv"] * 4)
    st = runner.Stack([l], 3 * runner.saved_bytes_per_layer(l) + (1 << 20), 0, "cuda:0", budget_bytes=0)
    hp.load_weights(l, case["w"], st.dev)
    x, dy = (runner.to_device(case[k], "bf16", st.dev) for k in ("x", "dy"))
    kv = torch.from_numpy(case["kv_len"]).to(st.dev) if "kv_len" in case else None
    kvp = kv.data_ptr() if kv is not None else 0
    dx = torch.empty_like(dy)
    sb.ssdt_step_begin(st.ctx, 1)
    _, saved = sb.ssdt_layer_fwd(st.ctx, l.desc, l.wstruct, 0, x.data_ptr(), 0, kvp, st.ws_ptr, st.ws_bytes, st.stream)
    sb.ssdt_layer_bwd(st.ctx, l.desc, l.wstruct, saved, kvp, dy.data_ptr(), dx.data_ptr(), 0, l.gstruct, st.ws_ptr, st.ws_bytes,
                      st.stream)
    torch.cuda.synchronize()
    tmp, base = sb.ssdt_layer_bwd_temporaries(l.desc), st.ws_ptr - st.ws.data_ptr()

    def heads(t, cols, at):      # [B, A, S, d] of the columns from `at` on
        t = t.double().cpu().reshape(l.B, l.S, cols)[:, :, at:at + l.H]
        return t.reshape(l.B, l.S, l.A, -1).transpose(1, 2)
    qkv = st.view(saved.e[sb.SV_NAMES.index("qkv")].ptr, (l.T, 3 * l.H))
    q, k, v = (heads(qkv, 3 * l.H, i * l.H) for i in range(3))
    o = heads(st.view(saved.e[sb.SV_NAMES.index("o")].ptr, (l.T, l.H)), l.H, 0)
    n = l.T * l.H * 2
    do = heads(st.ws[base + tmp["t0"]:base + tmp["t0"] + n].view(torch.bfloat16), l.H, 0)   # gradient of o, still there
    dv = heads(st.ws[base + tmp["d_qkv"]:base + tmp["d_qkv"] + 3 * n].view(torch.bfloat16), 3 * l.H, 2 * l.H)
    s = q @ k.transpose(2, 3) / (l.H // l.A) ** 0.5
    if l.mask == "causal":
        s.masked_fill_(torch.ones(l.S, l.S, dtype=torch.bool).triu(1), float("-inf"))
    if l.mask == "keypad":
        for b in range(l.B):
            s[b, :, :, int(case["kv_len"][b]):] = float("-inf")
    p = torch.softmax(s, -1)
    st.close()
    for what, got, ref in (("o", o, p @ v), ("dv", dv, p.transpose(2, 3) @ do)):
        missed = float((got != ref.to(torch.bfloat16).double()).double().mean())
        print(name, what, "%.4f %%" % (100 * missed))
        assert missed <= 1e-3, (what, missed)
