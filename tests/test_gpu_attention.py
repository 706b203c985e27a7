"""bf16 attention of whole tiles by itself, forward and backward, against 64 bits: one block of 128 queries, more blocks than run at a
time (a workgroup then does several), numbers of heads that the eight XCDs do and do not share evenly, sequences of few keys or none."""
import ctypes
import math

import pytest
import torch

from paper_2408_10013_amd import binding as sb

pytestmark = pytest.mark.gpu

NONE, CAUSAL, KEYPAD = 0, 1, 2


class Attn(ctypes.Structure):
    """struct Attn of csrc/kernels.h."""
    _fields_ = [(n, t) for t, names in [
        (ctypes.c_int, "B A Sq Sk d"), (ctypes.c_float, "scale"), (ctypes.c_int, "mask"), (ctypes.c_void_p, "kv_len"), (ctypes.c_int, "dtype"),
        (ctypes.c_void_p, "q k v"), (ctypes.c_long, "ldq ldk ldv"), (ctypes.c_void_p, "o"), (ctypes.c_long, "ldo"), (ctypes.c_void_p, "lse"),
        (ctypes.c_bool, "ordered"), (ctypes.c_void_p, "dout"), (ctypes.c_long, "lddo"), (ctypes.c_void_p, "dq dk dv"),
        (ctypes.c_long, "lddq lddk lddv"), (ctypes.c_void_p, "delta")] for n in names.split()]


def call(name, a):
    f = getattr(sb.lib(), "_ZN4ssdt1k8%sERKNS0_4AttnEP12ihipStream_t" % name)
    f.argtypes, f.restype = [ctypes.POINTER(Attn), ctypes.c_void_p], ctypes.c_int
    assert f(ctypes.byref(a), torch.cuda.current_stream().cuda_stream) == 0


def few_keys(B, A, Sq, Sk, d, mask, items):
    f = sb.lib()._ZN4ssdt1k13attn_few_keysERKNS0_4AttnEl
    f.argtypes, f.restype = [ctypes.POINTER(Attn), ctypes.c_long], ctypes.c_bool
    return f(ctypes.byref(Attn(B, A, Sq, Sk, d, 1 / math.sqrt(d), mask)), items)


# B, A, Sq, Sk, d, mask; the kernel: "few" keys, one block of 128 queries to a workgroup, or "deal", where workgroups take several in
# turn; whether there are more blocks than workgroups that run at a time (768 at head size 64, 512 at 128)
CASES = {
    "one_block": (1, 1, 128, 128, 128, CAUSAL, "few", False),
    "one_block_d64": (1, 3, 128, 128, 64, CAUSAL, "few", False),
    "few_keys": (5, 16, 512, 512, 64, KEYPAD, "few", False),
    "few_keys_many_blocks": (27, 43, 384, 384, 64, KEYPAD, "few", True),   # 3483
    "cross": (2, 8, 128, 384, 64, NONE, "few", False),
    "cross_many_blocks": (35, 16, 128, 512, 128, NONE, "few", True),
    "causal_512": (4, 5, 512, 512, 128, CAUSAL, "few", False),
    "one_round": (3, 43, 640, 640, 64, CAUSAL, "deal", False),             # 645 blocks of 768 workgroups, a last row that is not full
    "two_rounds": (4, 16, 1152, 1152, 128, CAUSAL, "deal", True),          # 576 blocks of nine to a head
    "two_rounds_odd_heads": (3, 21, 1152, 1152, 128, CAUSAL, "deal", True),  # 567, numbers of heads that are no multiple of eight
    "two_rounds_odd_heads_d64": (3, 43, 896, 896, 64, CAUSAL, "deal", True),  # 903
    "padded_odd_heads": (7, 13, 1024, 1024, 128, KEYPAD, "deal", True),    # 728
    "padded_odd_heads_d64": (9, 19, 640, 640, 64, KEYPAD, "deal", True),   # 855
    "many_rounds": (1, 264, 768, 768, 128, CAUSAL, "deal", True),          # 1584
    "padded_many_rounds": (13, 8, 1024, 1024, 64, KEYPAD, "deal", True),
    "padded_d128": (19, 8, 512, 512, 128, KEYPAD, "deal", True),
    "cross_longer_queries": (9, 8, 1280, 128, 128, NONE, "deal", True),
}
LENGTHS = (0, 1, 63, 64, 65, 128, 200, 0, 0, 500)


@pytest.mark.parametrize("name", list(CASES))
def test_attention_of_whole_tiles(name):
    B, A, Sq, Sk, d, mask, kernel, rounds = CASES[name]
    items = B * A * Sq // 128
    assert few_keys(B, A, Sq, Sk, d, mask, items) == (kernel == "few") and (items > (768 if d == 64 else 512)) == rounds
    H, dev = A * d, "cuda:0"
    gen = torch.Generator(device=dev)
    gen.manual_seed(len(name))
    rnd = lambda *s: torch.randn(*s, generator=gen, device=dev).bfloat16()
    q, k, v, do = rnd(B * Sq, H), rnd(B * Sk, H), rnd(B * Sk, H), rnd(B * Sq, H)
    lens = [min(Sk, LENGTHS[b % len(LENGTHS)]) if mask == KEYPAD else Sk for b in range(B)]
    ref = [t.double() for t in (q, k, v, do)]
    for b, n in enumerate(lens):    # what lies behind the tile that holds the last key is never looked at
        behind = slice(b * Sk + -(-n // 64) * 64, (b + 1) * Sk)
        k[behind], v[behind] = math.nan, math.nan
    kv_len = torch.tensor(lens, dtype=torch.int32, device=dev)
    o, dq, dk, dv = (torch.full_like(t, math.nan) for t in (q, q, k, v))
    lse, delta = torch.empty(B, A, Sq, device=dev), torch.empty(2, B, A, Sq, device=dev)
    P = lambda t: t.data_ptr()
    a = Attn(B, A, Sq, Sk, d, 1 / math.sqrt(d), mask, P(kv_len) if mask == KEYPAD else 0, sb.BF16, P(q), P(k), P(v), H, H, H,
             P(o), H, P(lse), False, P(do), H, P(dq), P(dk), P(dv), H, H, H, P(delta))
    call("attn_fwd", a)
    for b, n in enumerate(lens):    # (the backward's tiles of padded keys may be read: zeros times zero probability)
        k[b * Sk + n:(b + 1) * Sk], v[b * Sk + n:(b + 1) * Sk] = 0, 0
    call("attn_bwd", a)
    torch.cuda.synchronize()

    def close(got, want, bound):
        # `bound`: what one rounding to bf16 (8 bits: 2^-8 of the value) of each probability or dS can make of the sum; the result is
        # rounded once more.  The fp32 sums and exponentials stay below 2^-16 of the sum of absolute values.
        bound = 2 ** -8 * want.abs() + (1 + 2 ** -7) * bound + 1e-30
        err = (got.double() - want).abs()
        assert bool((err <= bound).all()), (err / bound).max().item()

    heads = lambda t, b, n: t[b * n:(b + 1) * n].reshape(n, A, d).transpose(0, 1).contiguous()
    flat = lambda t: t.transpose(0, 1).reshape(t.shape[1], H)
    for b, n in enumerate(lens):
        Q, K, V, DO = heads(ref[0], b, Sq), heads(ref[1], b, Sk), heads(ref[2], b, Sk), heads(ref[3], b, Sq)
        s = torch.matmul(Q, K.transpose(1, 2).contiguous()) / math.sqrt(d)
        if mask == CAUSAL:
            s.masked_fill_(torch.ones(Sq, Sk, dtype=torch.bool, device=dev).triu(1), -math.inf)
        s[:, :, n:] = -math.inf
        p = torch.softmax(s, -1) if n else torch.zeros_like(s)
        at, kat = slice(b * Sq, (b + 1) * Sq), slice(b * Sk, (b + 1) * Sk)
        x, e = torch.matmul(p, V), 2 ** -8
        close(o[at], flat(x), flat(torch.matmul(p * e, V.abs())))
        want = torch.logsumexp(s, -1)
        assert torch.equal(torch.isinf(lse[b].double()), torch.isinf(want))
        assert n == 0 or bool(((lse[b].double() - want).abs() <= 1e-5 * (1 + want.abs())).all())
        ds = torch.matmul(DO, V.transpose(1, 2).contiguous())
        ds = p * (ds - (p * ds).sum(-1, keepdim=True)) / math.sqrt(d)
        # delta is summed from the output as it is stored: rounded, and made of rounded probabilities
        off = (DO.abs() * (x.abs() * e + torch.matmul(p * e, V.abs()))).sum(-1, keepdim=True)
        off = ds.abs() * e + p * off / math.sqrt(d) * (1 + e)
        close(dq[at], flat(torch.matmul(ds, K)), flat(torch.matmul(off, K.abs())))
        close(dk[kat], flat(torch.matmul(ds.transpose(1, 2).contiguous(), Q)), flat(torch.matmul(off.transpose(1, 2).contiguous(), Q.abs())))
        close(dv[kat], flat(torch.matmul(p.transpose(1, 2).contiguous(), DO)), flat(torch.matmul(p.transpose(1, 2).contiguous() * e, DO.abs())))


@pytest.mark.parametrize("B,S,A,d,f32", [(1, 1, 1, 64, False), (3, 37, 16, 128, False), (5, 197, 43, 64, False), (9, 1000, 8, 64, False), (2, 131, 12, 64, True),
                                         (7, 333, 3, 128, False), (64, 5, 96, 16, False)])
def test_row_sums_of_the_backward(B, S, A, d, f32):
    """delta = sum over a head's columns of o dO, one KiB of a token's row and more, tokens that do not fill the workgroups' sixteen."""
    dev = "cuda:0"
    gen = torch.Generator(device=dev)
    gen.manual_seed(S)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=dev).to(torch.float32 if f32 else torch.bfloat16)
    o, do, lse = rnd(B * S, A * d), rnd(B * S, A * d), torch.randn(B, A, S, generator=gen, device=dev)
    lse[0, 0, 0] = -math.inf
    out = torch.full((2, B, A, S), math.nan, device=dev)
    f = sb.lib()._ZN4ssdt1k14attn_delta_vecEPKvlS2_lPfPKfS3_iiiiiP12ihipStream_t
    f.argtypes = [ctypes.c_void_p, ctypes.c_long] * 2 + [ctypes.c_void_p] * 3 + [ctypes.c_int] * 5 + [ctypes.c_void_p]
    assert f(o.data_ptr(), A * d, do.data_ptr(), A * d, out[0].data_ptr(), lse.data_ptr(), out[1].data_ptr(), B, S, A, d,
             sb.F32 if f32 else sb.BF16, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    prod = (o.double() * do.double()).reshape(B, S, A, d).permute(0, 2, 1, 3)
    # d fused multiply-adds and additions in fp32, 2^-24 of the sum of absolute values each
    assert bool(((out[0].double() - prod.sum(-1)).abs() <= d * 2.0 ** -24 * prod.abs().sum(-1)).all())
    want = lse * 1.4426950408889634
    want[0, 0, 0] = math.inf
    assert torch.allclose(out[1], want, rtol=1e-6, atol=0)
