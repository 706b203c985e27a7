"""What the build refuses, and what the machine code of libssdt.so must hold."""
import subprocess

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
