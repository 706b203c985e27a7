"""bf16 products by themselves: kernels of one tile that differ in the order in which they load and read, not in that of their sums."""
import ctypes

import pytest
import torch

from paper_2408_10013_amd import binding as sb

pytestmark = pytest.mark.gpu
P, I, L, B = ctypes.c_void_p, ctypes.c_int, ctypes.c_long, ctypes.c_bool


class Gemm(ctypes.Structure):
    """struct Gemm of csrc/kernels.h."""
    _fields_ = [("M", I), ("N", I), ("K", I), ("A", P), ("lda", L), ("transA", B), ("B", P), ("ldb", L), ("transB", B), ("C", P), ("ldc", L),
                ("epi", I), ("bias", P), ("resid", P), ("ldr", L), ("C2", P), ("aux", P), ("act", I), ("dtype", I), ("colsum", P),
                ("colsum_accumulate", B), ("scratch", P), ("scratch_bytes", ctypes.c_size_t), ("split", B), ("one_order", B), ("ordered", B)]


@pytest.fixture
def tile():
    hook = ctypes.c_int.in_dll(sb.lib(), "_ZN4ssdt1k10g_tile_cfgE")

    def pin(cfg):
        hook.value = cfg
    yield pin
    hook.value = -1


def rnd(*shape):
    return torch.randn(*shape, device="cuda:0").bfloat16()


def close(got, a, b):
    """To the last bit but for the fp32 sums: a result rounded to bf16, 2^-9 of it, and K additions of 2^-24 of the absolute sum."""
    a, b = a.double(), b.double()
    want, size = a @ b, a.abs() @ b.abs()
    assert bool(((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + a.shape[1] * 2.0 ** -24 * size).all())


# 128 x 128 in a ring of two, 64 x 128 in one of three, 128 x 128 in one of four; contractions with tails, of 1 stage, 9, 10 and 16, and sizes that end inside a
# tile, more tiles than run at a time
@pytest.mark.parametrize("cfg", [0, 3, 5])
@pytest.mark.parametrize("M,N,K", [(130, 136, 40), (2300, 1920, 584), (2100, 1928, 1000), (4090, 2040, 520), (1660, 25144, 528)])
def test_every_order_of_loads_and_reads(tile, M, N, K, cfg):
    torch.manual_seed(M)
    a, b, out = rnd(M, K), rnd(K, N), []
    f = sb.lib()._ZN4ssdt1k4gemmERKNS0_4GemmEP12ihipStream_t
    f.argtypes, f.restype = [ctypes.POINTER(Gemm), ctypes.c_void_p], ctypes.c_int
    for which in (cfg, 1):  # 1: 64 x 128 in a ring of two
        tile(which)
        c = torch.full((M, N), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        g = Gemm(M=M, N=N, K=K, A=a.data_ptr(), lda=K, B=b.data_ptr(), ldb=N, C=c.data_ptr(), ldc=N, dtype=sb.BF16)
        assert f(ctypes.byref(g), torch.cuda.current_stream().cuda_stream) == 0
        out.append(c)
    torch.cuda.synchronize()
    assert torch.equal(*out)
    close(out[0], a, b)


@pytest.mark.parametrize("rows,width,out,four", [(512, 2880, 2880, True), (440, 2696, 2696, True), (384, 2520, 2520, False), (300, 1600, 1928, False)])
def test_both_products_of_a_linears_backward(tile, rows, width, out, four):
    """64 x 128 tiles in a ring of three, by four wavefronts from 960 workgroups on, by eight below; bias sums with the weight gradient."""
    up = lambda n, by: -(-n // by)
    assert four == (up(width, 64) * up(out, 128) + up(rows, 64) * up(width, 128) >= 960)
    torch.manual_seed(rows)
    x, w, dy, res = rnd(rows, width), rnd(width, out), rnd(rows, out), []
    f = sb.lib()._ZN4ssdt1k14gemm_pair_bf16ERKNS0_4GemmES3_PKNS0_8PairPlanEP12ihipStream_t
    f.argtypes, f.restype = [ctypes.POINTER(Gemm), ctypes.POINTER(Gemm), ctypes.c_void_p, ctypes.c_void_p], ctypes.c_int
    for cfg in (3, 1):
        tile(cfg)
        dw, dx, db = (torch.full(s, float("nan"), device="cuda:0", dtype=torch.bfloat16) for s in ((width, out), (rows, width), (out,)))
        gw = Gemm(M=width, N=out, K=rows, A=x.data_ptr(), lda=width, transA=True, B=dy.data_ptr(), ldb=out, C=dw.data_ptr(), ldc=out,
                  dtype=sb.BF16, colsum=db.data_ptr())
        gd = Gemm(M=rows, N=width, K=out, A=dy.data_ptr(), lda=out, B=w.data_ptr(), ldb=out, transB=True, C=dx.data_ptr(), ldc=width, dtype=sb.BF16)
        assert f(ctypes.byref(gw), ctypes.byref(gd), None, torch.cuda.current_stream().cuda_stream) == 0
        res.append((dw, dx, db))
    torch.cuda.synchronize()
    assert all(torch.equal(*p) for p in zip(*res))
    close(res[0][0], x.t().contiguous(), dy)
    close(res[0][1], dy, w.t().contiguous())
    close(res[0][2], torch.ones(1, rows, device="cuda:0"), dy)
