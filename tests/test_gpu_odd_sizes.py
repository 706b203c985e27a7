"""The kernels that take any size, at the edges of their tiles: forward and backward of small layers against the CPU
checker.  bf16 widths that are multiples of 8 go through the matrix-core GEMM; sizes as small as these choose its tiles of 32 x 32 to
64 x 64 with the wavefronts side by side along k (fp32: 32 x 32) and split nothing by themselves: the larger tiles and the splits are
pinned."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import layer_oracle as lo
from paper_2408_10013_amd import binding as sb
from paper_2408_10013_amd import runner, synth

import helpers as hp
import test_gpu_stack as ts
from test_gpu_layer import check_against_oracle, run_single_layer

pytestmark = pytest.mark.gpu

GPT = dict(arch="gpt_preln", act="gelu", norm="layernorm", mask="causal", has_bias=True, eps=1e-5)

SIZES = {
    "one_token": dict(B=1, S=1, H=64, A=1, F=64),                # a single row; contraction over one token
    "tile_less_one": dict(B=1, S=127, H=64, A=1, F=136),         # last row / column of a tile missing
    "tile_plus_one": dict(B=1, S=129, H=64, A=1, F=264),         # a tile with one row
    "stage_tail": dict(B=3, S=43, H=72, A=3, F=200),             # K = 72, 200, 129: tails of 8, 8 and 1 behind whole stages
    "narrow": dict(B=2, S=65, H=8, A=1, F=8),                    # one 16-byte chunk per row
    "split_k": dict(B=1, S=40, H=64, A=1, F=2048),               # 32 stages of 64 on one tile
    "split_tokens": dict(B=5, S=333, H=64, A=1, F=128),          # 27 stages of 64 over tokens (the last one short), bias sums
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
    "cross_d12": dict(T5, B=2, S=37, S_kv=21, H=36, A=3, F=52),   # widths that are no multiple of 8
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


# ReLU: at lengths or widths that are not whole tiles the forward keeps the order of additions of the FMA kernels, in bf16 too, but
# for the MLP's two products, which have the one order of the bf16 tiles with 64 k a stage
RELU = {
    "d12": dict(T5, act="relu", B=2, S=37, S_kv=45, H=36, A=3, F=52),           # K-contiguous rows element by element; heads
    "d20_enc": dict(T5, arch="t5_enc", mask="none", act="relu", B=2, S=70, H=60, A=3, F=72),  # that end inside a 16-byte load
    "d64": dict(T5, act="relu", B=2, S=65, S_kv=130, H=128, A=2, F=200),
    "d96": dict(T5, act="relu", B=1, S=100, S_kv=33, H=96, A=1, F=136),
    "d128": dict(T5, act="relu", B=1, S=67, S_kv=64, H=256, A=2, F=72),
    "d18": dict(T5, act="relu", B=1, S=40, S_kv=70, H=54, A=3, F=64),
}


@pytest.mark.parametrize("name", list(RELU))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_relu_layers_of_any_size(name, dtype):
    """Forward and saved tensors against the checker; the backward against the checker's with ReLU's decisions taken from the
    stored activations, as the library takes them."""
    l = runner.Layer(dtype=dtype, **RELU[name])
    case = hp.make_layer_case(l, 8200 + l.H)
    on = run_single_layer(l, case, offload=True)
    check_against_oracle(l, case, on, hp.TOL[dtype], check_bwd=False)
    d = hp.oracle_desc(l)
    _, sv = lo.layer_fwd(d, case["w"], case["x"], case.get("enc"), None)
    dx, denc, gr = hp.layer_bwd_same_relu_decisions(d, case["w"], sv, case["dy"], None, on["saved"]["g"])
    errs = {"dx": hp.rel_err(runner.to_host(on["dx"]), dx)}
    if denc is not None:
        errs["d_enc"] = hp.rel_err(runner.to_host(on["d_enc"]), denc)
    assert set(on["grads"]) == set(gr)
    for k in gr:
        errs["grad." + k] = hp.rel_err(runner.to_host(on["grads"][k]), gr[k])
    bad = {k: e for k, e in errs.items() if not e <= hp.TOL[dtype]}
    assert not bad, bad


@pytest.mark.parametrize("H,A", [(36, 3), (128, 2)])
def test_relu_forward_products_add_in_the_order_of_k(H, A):
    """bf16, ReLU, ragged: every element of the projection is a chain of fused multiply-adds, k ascending, bit for bit.  (In
    64 bits a product of two bf16 is exact, and so is its sum with an fp32 number but where that outweighs it beyond 2^29.)"""
    l = runner.Layer("t5_enc", "bf16", B=2, S=37, H=H, A=A, F=64, act="relu", norm="rmsnorm", mask="none", has_bias=False, eps=1e-6)
    case = hp.make_layer_case(l, 8300 + H)
    saved = run_single_layer(l, case, offload=False)["saved"]
    a, w = saved["a"].astype(np.float64), case["w"]["w_qkv"].astype(np.float64)
    acc = np.zeros((l.T, 3 * H), dtype=np.float32)
    for k in range(H):
        acc = (a[:, k:k + 1] * w[k] + acc).astype(np.float32)
    assert np.array_equal(saved["qkv"], synth.bf16_round(acc))


def hook(name):
    return ctypes.c_int.in_dll(sb.lib(), "_ZN4ssdt1k%d%sE" % (len(name), name))


def split_products(l, tile, splits, passes=1):
    """How many of a bf16 layer's products are split where a tile and a number of splits are pinned: those with a stage for a second
    part; in the forward, if the workspace that was reported holds the parts."""
    ws, stage, n = max(sb.ssdt_layer_workspace(l.desc)), 128 if tile in (6, 7, 8) else 64, 0
    parts = lambda k: -(-(s := -(-k // stage)) // -(-s // splits))
    for rows, i, o in ((l.T, l.H, 3 * l.H), (l.T, l.H, l.H), (l.T, l.H, l.F), (l.T, l.F, l.H)):
        n += parts(i) > 1 and splits * (rows + 1) * o * 4 <= ws
        n += passes * ((parts(rows) > 1) + (parts(o) > 1))
    return n if tile != 9 else 0


@pytest.fixture
def pin():
    """Sets a kernel's test hook for the time of a test."""
    was = []

    def set_(name, value):
        v = hook(name)
        was.append((v, v.value))
        v.value = value
    yield set_
    for v, old in reversed(was):
        v.value = old


# rows 333 (2 tiles of 128 and 77 rows), widths 200 (1 and 72), 264 (2 and 8), 600; contractions with tails of 8 and 13 of 64
RAGGED = dict(GPT, B=3, S=111, H=200, A=5, F=264)


@pytest.mark.parametrize("splits", [1, 2, 3])
@pytest.mark.parametrize("tile", [0, 1, 2])
def test_every_bf16_tile_at_ragged_sizes(pin, tile, splits):
    """128 x 128, 64 x 128 and 64 x 64 tiles, the contraction whole and in parts, both products of a backward together."""
    pin("g_tile_cfg", tile)
    pin("g_tile_splits", splits)
    l = runner.Layer(dtype="bf16", **RAGGED)
    case = hp.make_layer_case(l, 8400 + tile, bias_std=0.05)
    before = hook("g_tile_reduces").value
    check_against_oracle(l, case, run_single_layer(l, case, offload=False, fetch=False), hp.TOL["bf16"])
    assert hook("g_tile_reduces").value - before == split_products(l, tile, splits) == (12 if splits > 1 else 0)


# contractions of 1 and 2 stages of 64 (H 40, F 72, 111 tokens), of 4, 5, 6 and 10 (RAGGED), of 3, 9 and 25 (H 520, F 136)
@pytest.mark.parametrize("size", [dict(B=3, S=37, H=40, A=1, F=72), RAGGED, dict(B=2, S=70, H=520, A=5, F=136)], ids=["1", "4", "9"])
@pytest.mark.parametrize("tile", [3, 4, 5, 6, 7, 8, 9])
def test_every_ring_of_stages(pin, tile, size):
    """Tiles whose stages stand in a ring of three or four, from 6 on with the wavefronts side by side along k (6 to 8: stages of 128;
    9: 256 x 128): fewer stages than the ring holds, as many, and more; whole and split."""
    l = runner.Layer(dtype="bf16", **dict(GPT, **{k: size[k] for k in "BSHAF"}))
    case = hp.make_layer_case(l, 8420 + tile, bias_std=0.05)
    pin("g_tile_cfg", tile)
    for splits in (1, 2) if tile != 9 else (1,):
        pin("g_tile_splits", splits)
        before = hook("g_tile_reduces").value
        check_against_oracle(l, case, run_single_layer(l, case, offload=False, fetch=False), hp.TOL["bf16"])
        done = hook("g_tile_reduces").value - before
        assert done == split_products(l, tile, splits) and (done > 0) == (splits > 1 and (l.H > 40 or tile < 6))


@pytest.mark.parametrize("kind", ["t5_enc", "t5_dec"])
@pytest.mark.parametrize("size", [dict(B=2, S=128, H=256, A=2, F=512), dict(B=8, S=128, H=1024, A=16, F=2560), dict(B=8, S=256, H=2048, A=32, F=4096)],
                         ids=["256", "1024", "2048"])
def test_relu_layers_of_whole_tiles_add_in_one_order(pin, kind, size):
    """The output of a layer with ReLU, which the next layer's ReLU decides on, has the same bits whatever tile the products take by
    themselves: those of 128 x 128 tiles (two decoder layers moved by 5 % with the MLP's products in another order)."""
    l = runner.Layer(dtype="bf16", **dict(T5, arch=kind, act="relu", mask="none" if kind == "t5_enc" else "causal", S_kv=0 if kind == "t5_enc" else 128, **size))
    case = hp.make_layer_case(l, 8460, bias_std=0.05)
    own = run_single_layer(l, case, offload=False, fetch=False)["y"]
    pin("g_tile_cfg", 0)
    assert np.array_equal(own, run_single_layer(l, case, offload=False, fetch=False)["y"])


# by themselves these products take the wavefronts along k (the first three) and 256 x 128 tiles (the last)
RAGGED_RELU = {
    "45x256": dict(T5, arch="t5_enc", mask="none", act="relu", B=3, S=15, H=256, A=4, F=1024),
    "200x512": dict(T5, act="relu", B=2, S=100, S_kv=77, H=512, A=8, F=1280),
    "655x1024": dict(T5, act="relu", B=5, S=131, S_kv=60, H=1024, A=16, F=2560),
    "3000x2048": dict(T5, arch="t5_enc", mask="none", act="relu", B=3, S=1000, H=2048, A=16, F=8192),
}


@pytest.mark.parametrize("name", list(RAGGED_RELU))
def test_relu_layers_of_ragged_sizes_add_in_one_order(pin, name):
    """As above, and the layer behind decides as much as at whole tiles."""
    l = runner.Layer(dtype="bf16", **RAGGED_RELU[name])
    case = hp.make_layer_case(l, 8465, bias_std=0.05)
    own = run_single_layer(l, case, offload=False, fetch=False)["y"]
    for tile in (0, 4):
        pin("g_tile_cfg", tile)
        assert np.array_equal(own, run_single_layer(l, case, offload=False, fetch=False)["y"])


def test_ragged_relu_stack(pin):
    """Two encoder and two decoder layers: every layer's output has the bits of 128 x 128 tiles; outputs and gradients against the
    checker, ReLU's decisions taken from the stored activations."""
    kw = dict(T5, act="relu", dtype="bf16", B=3, H=256, A=4, F=512)
    mk = lambda: [runner.Layer(**dict(kw, arch="t5_enc", mask="none", S=111)) for _ in range(2)] + [runner.Layer(**kw, S=67, S_kv=111) for _ in range(2)]
    layers = mk()
    cases = [hp.make_layer_case(l, 8470 + i, bias_std=0.05) for i, l in enumerate(layers)]
    x, dy, enc_x = (runner.to_device(a, "bf16", "cuda:0") for a in (cases[2]["x"], cases[2]["dy"], cases[0]["x"]))
    per = max(runner.saved_bytes_per_layer(l) for l in layers)
    caps = []
    for tile in (-1, 0):
        pin("g_tile_cfg", tile)
        ls = mk()
        st = ts.build(ls, cases, 8 * per, 6 * per, keep_last=1, min_offload_elems=0, budget_bytes=0)
        y, dx, dxe, grads = ts.run_gpu(st, ls, x, dy, enc_x=enc_x, capture=True)[:4]
        caps.append(st.capture)
        if tile < 0:
            relu_g = {i: runner.to_host(t) for i, t in st.capture["g"].items()}
            got = dict(y=y, dx=dx, dx_enc=dxe, **{"l%d.%s" % (i, k): v for i, g in enumerate(grads) for k, v in g.items()})
            got = {k: runner.to_host(v) for k, v in got.items()}
        st.close()
    for i in range(4):
        assert torch.equal(caps[0]["y"][i], caps[1]["y"][i]), i
    y_ref, dx_ref, dxe_ref, g_ref = ts.oracle_stack(layers, cases, cases[2]["x"], cases[2]["dy"], enc_x=cases[0]["x"], relu_g=relu_g)
    ref = dict(y=y_ref, dx=dx_ref, dx_enc=dxe_ref, **{"l%d.%s" % (i, k): v for i, g in enumerate(g_ref) for k, v in g.items()})
    bad = {k: e for k, e in ((k, hp.rel_err(got[k], ref[k])) for k in ref) if not e <= hp.TOL["bf16"]}
    assert not bad, bad


# stages of 64 k (tile 32) or 32 (tile 64): 1 and 2 of either, as many as the ring holds, and more; widths that end inside a tile
# and inside a stage; the middle size ends a row of k inside a 64-byte unit
@pytest.mark.parametrize("size", [dict(B=3, S=9, H=24, A=1, F=52), dict(B=3, S=37, H=132, A=2, F=100), dict(B=2, S=185, H=260, A=5, F=516)],
                         ids=["1", "3", "9"])
@pytest.mark.parametrize("tile,ring", [(32, 2), (32, 3), (64, 3)])
def test_every_ring_of_stages_f32(pin, tile, ring, size):
    """Direct loads, and the same with operands that start at 4 bytes, which go through registers: the same bits."""
    l = runner.Layer(dtype="f32", **dict(GPT, **size))
    case = hp.make_layer_case(l, 8470 + tile + ring, bias_std=0.05)
    pin("g_f32_tile", tile)
    pin("g_f32_ring", ring)
    res = run_backward(l, case)
    check_against_oracle(l, case, res, hp.TOL["f32"])
    kept = {k: v.clone() for k, v in res["grads"].items()}
    l.w = {k: shifted(v, 1) if k.startswith("w_") else v for k, v in l.w.items()}
    l.wstruct = sb.make_weights({k: v.data_ptr() for k, v in l.w.items()})
    other = run_backward(l, case)
    assert np.array_equal(res["y"], other["y"]) and torch.equal(res["dx"], other["dx"])
    assert all(torch.equal(kept[k], other["grads"][k]) for k in kept)


@pytest.mark.parametrize("name", ["d12", "d64"])
def test_relu_products_with_the_larger_tile(pin, name):
    pin("g_f32_tile", 64)
    l = runner.Layer(dtype="bf16", **RELU[name])
    case = hp.make_layer_case(l, 8200 + l.H)
    check_against_oracle(l, case, run_single_layer(l, case, offload=False), hp.TOL["bf16"], check_bwd=False)


@pytest.mark.parametrize("size", ["ragged", "odd_k"])
@pytest.mark.parametrize("tile", [64, 32])
def test_every_f32_tile_at_ragged_sizes(pin, tile, size):
    pin("g_f32_tile", tile)
    v = RAGGED if size == "ragged" else dict(RAGGED, H=90, A=3, F=131)
    l = runner.Layer(dtype="f32", **v)
    case = hp.make_layer_case(l, 8450 + tile, bias_std=0.05)
    check_against_oracle(l, case, run_single_layer(l, case, offload=False, fetch=False), hp.TOL["f32"])


def run_backward(l, case, x=None, dx=None, passes=1):
    """Output, dx and gradients of one layer, bypassing the cache; with several passes the gradients add up."""
    st = runner.Stack([l], 4 * runner.saved_bytes_per_layer(l) + (1 << 20), 0, "cuda:0", budget_bytes=0)
    if not l.w:
        hp.load_weights(l, case["w"], st.dev)
    x = runner.to_device(case["x"], l.dtype, st.dev) if x is None else x
    dy = runner.to_device(case["dy"], l.dtype, st.dev)
    dx = torch.empty_like(dy) if dx is None else dx
    kv = torch.from_numpy(case["kv_len"]).to(st.dev) if "kv_len" in case else None
    kvp = kv.data_ptr() if kv is not None else 0
    sb.ssdt_step_begin(st.ctx, 1)
    y, saved = sb.ssdt_layer_fwd(st.ctx, l.desc, l.wstruct, 0, x.data_ptr(), 0, kvp, st.ws_ptr, st.ws_bytes, st.stream)
    for i in range(passes):
        sb.ssdt_layer_bwd(st.ctx, l.desc_acc if i else l.desc, l.wstruct, saved, kvp, dy.data_ptr(), dx.data_ptr(), 0, l.gstruct,
                          st.ws_ptr, st.ws_bytes, st.stream)
    torch.cuda.synchronize()
    res = dict(y=runner.to_host(st.view(y, (l.T, l.H))), dx=dx.clone(), d_enc=None, grads=l.g)
    st.close()
    return res


@pytest.mark.parametrize("dtype,tile,splits", [("f32", -1, 0), ("bf16", -1, 0)] + [("bf16", t, 1) for t in range(10)] +
                         [("bf16", t, 4) for t in range(9)])
def test_split_products_add_to_what_the_gradients_hold(pin, dtype, tile, splits):
    """1665 tokens, 64 x 128 weights: a second backward adds to the gradients, bias sums included, in the product's own epilogue
    or, where the contraction over tokens is split, in the reduction's."""
    pin("g_tile_cfg", tile)
    pin("g_tile_splits", splits)
    l = runner.Layer(dtype=dtype, **GPT, **SIZES["split_tokens"])
    case = hp.make_layer_case(l, 8600, bias_std=0.05)
    before = hook("g_tile_reduces").value
    res = run_backward(l, case, passes=2)
    if tile >= 0:
        done = hook("g_tile_reduces").value - before
        assert done == split_products(l, tile, splits, passes=2) and (done >= 8) == (splits > 1)
    res["grads"] = {k: v.float() / 2 for k, v in res["grads"].items()}   # (exact)
    check_against_oracle(l, case, res, hp.TOL[dtype])


@pytest.mark.parametrize("tile", [-1, 0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_dx_may_overwrite_the_input(pin, dtype, tile):
    """A post-norm layer whose dx takes the place of x: the weight gradient must have read x by then."""
    if tile >= 0:
        pin("g_tile_cfg", tile)
        pin("g_f32_tile", 64)
    l = runner.Layer(dtype=dtype, **BERT, B=2, S=70, H=128, A=2, F=200)
    case = hp.make_layer_case(l, 8650, bias_std=0.05, kv_len_range=(40, 70))
    x = runner.to_device(case["x"], dtype, torch.device("cuda:0"))
    check_against_oracle(l, case, run_backward(l, case, x=x, dx=x), hp.TOL[dtype])


def shifted(t, n):
    """A copy of t that starts n elements behind an aligned address."""
    buf = torch.empty(t.numel() + 256, dtype=t.dtype, device=t.device)
    assert buf.data_ptr() % 256 == 0
    return buf[n:n + t.numel()].view(t.shape).copy_(t)


@pytest.mark.parametrize("what", ["weights", "input", "gradients"])
@pytest.mark.parametrize("n", [1, 4])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_operands_that_are_not_16_byte_aligned(dtype, n, what):
    """Whole tiles of 128.  bf16: products with such operands go through transposed copies and the 128 x 128 kernel (weights in
    the forward, x in the weight gradient), or through the FMA kernel."""
    l = runner.Layer(dtype=dtype, **BERT, B=2, S=128, H=128, A=1, F=256)
    case = hp.make_layer_case(l, 8700, bias_std=0.05, kv_len_range=(64, 128))
    dev = torch.device("cuda:0")
    hp.load_weights(l, case["w"], dev)
    x = runner.to_device(case["x"], dtype, dev)
    if what == "weights":
        l.w = {k: shifted(v, n) if k.startswith("w_") else v for k, v in l.w.items()}
        l.wstruct = sb.make_weights({k: v.data_ptr() for k, v in l.w.items()})
    elif what == "gradients":
        l.g = {k: shifted(v, n) for k, v in l.g.items()}
        l.gstruct = sb.make_weights({k: v.data_ptr() for k, v in l.g.items()})
    else:
        x = shifted(x, n)
    check_against_oracle(l, case, run_backward(l, case, x=x), hp.TOL[dtype])


@pytest.mark.parametrize("n", [0, 1, 4])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_encoder_gradient_is_added_to_what_there_is(dtype, n):
    """A decoder layer's gradient of the encoder output, by the product's epilogue (aligned) and by a pass of its own: added to a sum
    of its own size, rounded to the type once or, in that pass, twice."""
    l = runner.Layer(dtype=dtype, **dict(T5, B=3, S=37, S_kv=45, H=64, A=2, F=72))
    case = hp.make_layer_case(l, 8750)
    d = hp.oracle_desc(l)
    _, sv = lo.layer_fwd(d, case["w"], case["x"], case["enc"], None)
    _, ref, _ = lo.layer_bwd(d, case["w"], sv, case["dy"], None)
    st = runner.Stack([l], 4 * runner.saved_bytes_per_layer(l) + (1 << 20), 0, "cuda:0", budget_bytes=0)
    hp.load_weights(l, case["w"], st.dev)
    x, dy, enc = (runner.to_device(case[k], dtype, st.dev) for k in ("x", "dy", "enc"))
    start = torch.randn(enc.shape, generator=torch.Generator().manual_seed(87)).to(enc.dtype).to(st.dev) * float(np.abs(ref).max())
    guard, dx = shifted(torch.cat([start, torch.full_like(start, 7)]), n), torch.empty_like(dy)
    sb.ssdt_step_begin(st.ctx, 1)
    _, saved = sb.ssdt_layer_fwd(st.ctx, l.desc, l.wstruct, 0, x.data_ptr(), enc.data_ptr(), 0, st.ws_ptr, st.ws_bytes, st.stream)
    sb.ssdt_layer_bwd(st.ctx, l.desc, l.wstruct, saved, 0, dy.data_ptr(), dx.data_ptr(), guard.data_ptr(), l.gstruct, st.ws_ptr,
                      st.ws_bytes, st.stream)
    torch.cuda.synchronize()
    got, behind = runner.to_host(guard[:len(start)]), runner.to_host(guard[len(start):])
    st.close()
    assert hp.rel_err(got, runner.to_host(start) + ref) <= hp.TOL[dtype] and (behind == 7).all()


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


# fp32 rows of 2, 4, 8 and 16 chunks of 256 floats, and one beyond what the vector kernels hold
@pytest.mark.parametrize("H,A", [(260, 5), (516, 6), (1028, 257), (2052, 18), (4100, 50)])
@pytest.mark.parametrize("kind", ["gpt_preln", "bert_postln", "t5_enc"])
def test_f32_norms_of_any_width(kind, H, A):
    """Forward and backward, with and without a residual gradient and shift; 70 rows: two chunks of the gains' sums, one ragged."""
    v = dict(gpt_preln=GPT, bert_postln=dict(BERT, mask="none"), t5_enc=dict(T5, arch="t5_enc", mask="none"))[kind]
    l = runner.Layer(dtype="f32", **dict(v, B=2, S=35, H=H, A=A, F=64))
    case = hp.make_layer_case(l, 8900 + H, bias_std=0.05)
    check_against_oracle(l, case, run_single_layer(l, case, offload=False, fetch=False), hp.TOL["f32"])


# 32 chunks and 33, where the second stage changes its loop, a last round of it that is not full, and all of its 128
@pytest.mark.parametrize("rows", [32 * 32, 33 * 32, 72 * 32 + 27, 128 * 32, 6001])
@pytest.mark.parametrize("accumulate", [False, True])
def test_gain_and_shift_gradients_of_many_chunks(rows, accumulate):
    H, dev = 40, "cuda:0"
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=dev)
    dy, x, mean, rstd, gamma, old = rnd(rows, H), rnd(rows, H), rnd(rows), rnd(rows).abs() + 0.5, rnd(H), rnd(2, H)
    dx, grads, partial = torch.empty_like(x), old.clone(), torch.full((2 * 128 * H,), float("nan"), device=dev)
    f = sb.lib()._ZN4ssdt1k8norm_bwdEPKvS2_PKfS4_S2_S2_PvS5_S5_PfmiiiibP12ihipStream_t
    f.argtypes = [ctypes.c_void_p] * 10 + [ctypes.c_size_t] + [ctypes.c_int] * 4 + [ctypes.c_bool, ctypes.c_void_p]
    layernorm = 0
    assert f(dy.data_ptr(), x.data_ptr(), mean.data_ptr(), rstd.data_ptr(), gamma.data_ptr(), None, dx.data_ptr(), grads[0].data_ptr(),
             grads[1].data_ptr(), partial.data_ptr(), partial.numel(), rows, H, layernorm, sb.F32, accumulate,
             torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    m, r = mean.double()[:, None], rstd.double()[:, None]
    base = old.double() if accumulate else torch.zeros(2, H, dtype=torch.float64, device=dev)
    # one addition per row of a chunk, eight chunks, sixteen threads and the old value, and three roundings of each term
    eps = (-(-rows // min(rows // 32, 128)) + 8 + 16 + 1 + 3) * 2.0 ** -24
    for got, term, size, b in ((grads[0], dy.double() * (x.double() - m) * r, dy.double().abs() * (x.double().abs() + m.abs()) * r, base[0]),
                               (grads[1], dy.double(), dy.double().abs(), base[1])):
        assert bool(((got.double() - b - term.sum(0)).abs() <= eps * (size.sum(0) + b.abs())).all())


# One axis of a grid holds fewer than 2^24 workgroups of 256.  Attention by tiles: forward 65535 x 257 workgroups, backward
# 2 x 65535 x 129.  Norm backward: one workgroup for four rows, and up to 128 for the first stage of the gain gradient.
@pytest.mark.parametrize("dtype,B,S,A", [("bf16", 65535, 6, 257), ("bf16", 65535, 9, 129), ("bf16", 262143, 256, 1), ("f32", 262143, 256, 1)])
def test_more_workgroups_than_one_axis_of_a_grid_holds(dtype, B, S, A):
    """First, middle and last sequences against the checker."""
    v = dict(T5, arch="t5_enc", mask="none", S=S, H=8 * A, A=A, F=8, dtype=dtype)
    l, some = runner.Layer(B=B, **v), [0, 1, B // 2, B - 1]
    ref = runner.Layer(B=len(some), **v)
    case = hp.make_layer_case(ref, 8900 + A)
    e = 2 if dtype == "bf16" else 4
    st = runner.Stack([l], runner.saved_bytes_per_layer(l) + 2 * l.T * l.H * e + (64 << 20), 0, "cuda:0", budget_bytes=0)
    hp.load_weights(l, case["w"], st.dev)
    rows = torch.cat([torch.arange(b * S, (b + 1) * S) for b in some]).to(st.dev)
    data = {}
    for k in ("x", "dy"):
        part = runner.to_device(case[k], dtype, st.dev)
        data[k] = torch.ones(l.T, l.H, dtype=part.dtype, device=st.dev)
        data[k][rows] = part
    dx = torch.zeros_like(data["dy"])
    sb.ssdt_step_begin(st.ctx, 1)
    y, saved = sb.ssdt_layer_fwd(st.ctx, l.desc, l.wstruct, 0, data["x"].data_ptr(), 0, 0, st.ws_ptr, st.ws_bytes, st.stream)
    sb.ssdt_layer_bwd(st.ctx, l.desc, l.wstruct, saved, 0, data["dy"].data_ptr(), dx.data_ptr(), 0, l.gstruct, st.ws_ptr,
                      st.ws_bytes, st.stream)
    torch.cuda.synchronize()
    d = hp.oracle_desc(ref)
    y_ref, sv = lo.layer_fwd(d, case["w"], case["x"])
    dx_ref, _, _ = lo.layer_bwd(d, case["w"], sv, case["dy"])
    errs = {"y": hp.rel_err(runner.to_host(st.view(y, (l.T, l.H))[rows]), y_ref), "dx": hp.rel_err(runner.to_host(dx[rows]), dx_ref)}
    o = st.view(saved.e[sb.SV_NAMES.index("o")].ptr, (l.T, l.H))[rows]
    errs["o"] = hp.rel_err(runner.to_host(o), sv["o"])
    st.close()
    assert max(errs.values()) <= hp.TOL[dtype], errs


def test_operands_of_more_than_2_to_the_34_elements():
    """524288 tokens, F 32776: the MLP's activations and their gradients as K-contiguous and as k-major operands, the tiles at their
    far end included, by the matrix-core kernels.  First, middle and last sequences against the checker; all others have no
    gradient."""
    B, S, F = 8192, 64, 32776
    some, v = [0, 1, B // 2, B - 1], dict(GPT, act="relu", dtype="bf16", S=S, H=8, A=1, F=F)
    l, ref = runner.Layer(B=B, **v), runner.Layer(B=4, **v)
    assert l.T * F >= 1 << 34
    case = hp.make_layer_case(ref, 8950, bias_std=0.05)
    st = runner.Stack([l], 2 * l.T * F + 64 * l.T * l.H + (64 << 20), 0, "cuda:0", budget_bytes=0)
    hp.load_weights(l, case["w"], st.dev)
    rows = torch.cat([torch.arange(b * S, (b + 1) * S) for b in some]).to(st.dev)
    data = {k: torch.full((l.T, l.H), fill, dtype=torch.bfloat16, device=st.dev) for k, fill in (("x", 1), ("dy", 0))}
    for k in data:
        data[k][rows] = runner.to_device(case[k], "bf16", st.dev)
    dx = torch.zeros_like(data["dy"])
    sb.ssdt_profile(st.ctx, True)
    sb.ssdt_step_begin(st.ctx, 1)
    y, saved = sb.ssdt_layer_fwd(st.ctx, l.desc, l.wstruct, 0, data["x"].data_ptr(), 0, 0, st.ws_ptr, st.ws_bytes, st.stream)
    sb.ssdt_layer_bwd(st.ctx, l.desc, l.wstruct, saved, 0, data["dy"].data_ptr(), dx.data_ptr(), 0, l.gstruct, st.ws_ptr, st.ws_bytes,
                      st.stream)
    torch.cuda.synchronize()
    ran = {p["name"] for p in sb.ssdt_profile_read(st.ctx)}
    sb.ssdt_profile(st.ctx, False)
    res = {"y": runner.to_host(st.view(y, (l.T, l.H))[rows]), "dx": runner.to_host(dx[rows])}
    g = runner.to_host(st.view(saved.e[sb.SV_NAMES.index("g")].ptr, (l.T, F))[rows])
    res.update({k: runner.to_host(t) for k, t in l.g.items()})
    st.close()
    assert "gemm_tile_k" in ran and not ran & {"gemm_generic_k", "gemm_nt128_k", "transpose_k"}, ran
    d = hp.oracle_desc(ref)
    y_ref, sv = lo.layer_fwd(d, case["w"], case["x"])
    dx_ref, _, gr = hp.layer_bwd_same_relu_decisions(d, case["w"], sv, case["dy"], None, g)
    bad = {k: e for k, e in ((k, hp.rel_err(res[k], r)) for k, r in dict(gr, y=y_ref, dx=dx_ref).items()) if not e <= hp.TOL["bf16"]}
    assert not bad, bad


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
