"""What the build refuses, and what the machine code of libssdt.so must hold."""
import os
import re
import subprocess

import pytest

import machine_code as mc
from paper_2408_10013_amd import build

BUFFER = """#include <hip/hip_runtime.h>
__global__ void fill_k(uint4 *out) {
  __shared__ __attribute__((%s)) char lds[4096];
  *(uint4 *)(lds + threadIdx.x * 16) = out[threadIdx.x];
  __syncthreads();
  out[threadIdx.x] = *(uint4 *)(lds + (255 - threadIdx.x) * 16);
}
"""


def test_a_misspelt_attribute_does_not_build(tmp_path):
    """An attribute that the compiler does not know is dropped with a warning, and with it the alignment that 16-byte LDS
    accesses need."""
    for attribute, ok in (("aligned(16)", True), ("aligned16", False)):
        src = tmp_path / "fill.hip"
        src.write_text(BUFFER % attribute)
        r = subprocess.run([build.HIPCC] + build.FLAGS + ["-x", "hip", "-fsyntax-only", str(src)], capture_output=True, text=True)
        assert (r.returncode == 0) == ok, r.stderr


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    found = mc.kernels(str(tmp_path_factory.mktemp("code")))
    assert len(found) > 100
    return found


def late_scalars(code):
    """Vector memory instructions that read a scalar register fewer than five wait states after a vector instruction wrote it."""
    late = []
    for i, ins in enumerate(code):
        op, _, args = ins.partition(" ")
        if not op.startswith(("buffer_", "global_")):
            continue
        reads, states = mc.scalars(args), 0
        for before in reversed(code[max(0, i - 5):i]):
            what, _, to = before.partition(" ")
            if states >= 5:
                break
            if what.startswith("v_") and reads & mc.scalars(to.split(", ")[0]):
                late.append((i, before, ins))
            states += int(to) + 1 if what == "s_nop" else 1
    return late


def own_wait(code, i):
    """Wait states that the statement of load i brings itself: what is right in front of it and only waits or sets M0 and EXEC."""
    states = 0
    for before in reversed(code[:i]):
        what, _, to = before.partition(" ")
        if what == "s_nop":
            states += int(to) + 1
        elif re.match(r"(m0|exec\w*),", to):
            states += 1
        else:
            break
    return states


def test_what_counts_as_a_late_scalar():
    load = "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"
    for code, late in (([], 0), (["v_readlane_b32 s7, v9, 3", "s_mov_b32 m0, s9", "s_nop 0"], 1), (["v_readlane_b32 s7, v9, 3", "s_nop 4"], 0),
                       (["v_readfirstlane_b32 s4, v9", "s_nop 3"], 1), (["v_cmp_gt_i32_e64 s[2:3], v1, v2"], 0), (["v_cmp_gt_i32_e64 s[6:7], v1, v2"], 1)):
        assert len(late_scalars(code + [load])) == late, code


def test_direct_loads_wait_for_their_scalars(built):
    """A scalar register that a vector instruction wrote, a reloaded spill among them, needs five wait states before a vector memory
    instruction reads it, and the compiler does not look into a load's assembly.  Where it spills scalar registers each load has to
    wait by itself, as a reload may stand in front of any of them."""
    for name, (notes, code) in built.items():
        assert not late_scalars(code), name
        if int(notes["sgpr_spill_count"]):
            for i, ins in enumerate(code):
                if re.match(r"(buffer|global)_load", ins) and "lds" in ins and "s[" in ins:
                    assert own_wait(code, i) >= 5, (name, code[max(0, i - 4):i + 1])


def test_statements_that_write_m0_say_so():
    for f in os.listdir(build.CSRC):
        text = open(os.path.join(build.CSRC, f)).read()
        for s in re.findall(r"asm volatile\((.*?)\);", text, re.S):
            assert not re.search(r"s_\w+ m0,", s) or re.search(r'"memory"[^)]*"m0"', s), (f, s)


def test_matrix_core_kernels_keep_their_vectors_in_registers(built):
    """A vector register reloaded in a loop is waited for together with the loads that the loop has on their way, the tiles of its next
    turns.  (Not asked of the fp32 backward at head sizes above 64 and of two of the 256 x 256 products, which were measured as they are.)"""
    kernels = [n for n in built if re.search(r"fa_fwd|fa_bwd|fa_f32_fwd|gemm_tile|gemm_wide|gemm_nt256", n)]
    assert len(kernels) > 40
    assert not [n for n in kernels if int(built[n][0]["vgpr_spill_count"])]
