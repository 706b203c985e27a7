"""The kernels of libssdt.so as they were built: what the code objects' notes say about them, and their instructions."""
import os
import re
import struct
import subprocess

from paper_2408_10013_amd import build

LLVM = "/opt/rocm/llvm/bin/"


def _tool(name, *args):
    return subprocess.run([LLVM + name, *args], check=True, capture_output=True, text=True).stdout


def kernels(tmp, instructions=True):
    """{name: (notes, instructions)} of the gfx950 kernels; `tmp`: a folder."""
    if not os.path.exists(build.LIB):
        build.build()
    bundle = os.path.join(tmp, "bundle")
    _tool("llvm-objcopy", "--dump-section=.hip_fatbin=" + bundle, build.LIB, os.devnull)
    data, found = open(bundle, "rb").read(), {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start() + 32
        for _ in range(struct.unpack_from("<Q", data, at - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + n]
            at += 24 + n
            if not target.endswith(b"gfx950") or not size:
                continue
            obj = os.path.join(tmp, "object")
            with open(obj, "wb") as f:
                f.write(data[m.start() + off:m.start() + off + size])
            notes = {}
            for part in re.split(r"\n  - (?=\.)", _tool("llvm-readelf", "--notes", obj)):
                d = dict(re.findall(r"^ *\.(\w+): +(\S+)$", part, re.M))
                if "vgpr_spill_count" in d:
                    notes[d["symbol"].removesuffix(".kd")] = d
            code = {}
            if instructions:
                for part in _tool("llvm-objdump", "-d", "--no-show-raw-insn", obj).split("\n\n"):
                    head, _, body = part.strip().partition(":\n")
                    name = re.fullmatch(r"[0-9a-f]+ <(\S+)>", head)
                    if name:
                        code[name[1]] = [l.split("//")[0].strip() for l in body.splitlines()]
            found.update({k: (v, code.get(k)) for k, v in notes.items()})
    return found


def scalars(operands):
    """Numbers of the scalar registers that an instruction's operands name."""
    regs = set()
    for a, b, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", operands):
        regs |= {int(one)} if one else set(range(int(a), int(b) + 1))
    for name, at in (("vcc", (106, 107)), ("vcc_lo", (106,)), ("vcc_hi", (107,))):
        if re.search(r"\b%s\b" % name, operands):
            regs |= set(at)
    return regs
