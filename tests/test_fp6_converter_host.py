"""The FP6 converters write their six result registers over several passes while still reading their sources, and the compiler's
register allocator is not told: a result on top of a source gives wrong codes without any error.  The sources hold them
apart with a statement that keeps both live; this reads the library's gfx950 code and checks that they are apart."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.environ.get("LQ_LIB", os.path.join(ROOT, "paper_2604_18117_amd", "liblq.so"))
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def _code_objects():
    blob, at = open(LIB, "rb").read(), 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := blob.find(magic, at)) >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            if count > 16:  # (the bytes of the magic in something else)
                break
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + n]:
                yield blob[at + off:at + off + size]
            p += 24 + n
        at += len(magic)


def _regs(operand, width=None):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]|v(\d+)", operand)
    if not m:
        return set()  # scalar or constant
    if m[3]:
        return {int(m[3])}
    lo, hi = int(m[1]), int(m[2])
    return set(range(lo, (hi if width is None else lo + width - 1) + 1))


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_results_and_sources_are_apart(tmp_path):
    found = {"act_int_kernel": 0, "mx6_": 0}
    for i, co in enumerate(_code_objects()):
        if b"act_int_kernel" not in co and b"mx6_" not in co:
            continue
        path = tmp_path / f"co{i}"
        path.write_bytes(co)
        p = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)], stdout=subprocess.PIPE, text=True)
        kernel = ""
        for line in p.stdout:
            if line.endswith(">:\n"):
                kernel = line
            elif "cvt_scalef32" in line and "fp6" in line:
                dst, *src = [t.strip() for t in line.split("//")[0].split(None, 1)[1].split(",")]
                int_family = "act_int_kernel" in kernel  # eight values of each source's sixteen: the rest is never looked at
                read = set().union(*(_regs(s, 8 if int_family and ":" in s else None) for s in src))
                assert not _regs(dst) & read, (kernel.strip(), line.strip())
                found["act_int_kernel" if int_family else "mx6_"] += 1
        assert p.wait() == 0
    assert all(found.values()), found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_mxint_main_codes(tmp_path):
    """The same for the MXINT4 main codes: 16 values per conversion (eight dwords of each source are defined), 32 in the
    hand-off of the large tiles."""
    found = {"mxi_act_kernel": 0, "mxi_fwd_small_kernel": 0, "mxi_fwd_kernel": 0}
    for i, co in enumerate(_code_objects()):
        if b"mxi_act_kernel" not in co:
            continue
        path = tmp_path / f"co{i}"
        path.write_bytes(co)
        p = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)], stdout=subprocess.PIPE, text=True)
        kernel = ""
        for line in p.stdout:
            if line.endswith(">:\n"):
                kernel = line
            elif "cvt_scalef32" in line and "fp6" in line:
                dst, *src = [t.strip() for t in line.split("//")[0].split(None, 1)[1].split(",")]
                name = next(k for k in found if k in kernel)
                read = set().union(*(_regs(s, 8 if name != "mxi_fwd_kernel" and ":" in s else None) for s in src))
                assert not _regs(dst) & read, (kernel.strip(), line.strip())
                found[name] += 1
        assert p.wait() == 0
    assert all(found.values()), found
