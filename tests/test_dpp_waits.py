"""The wait states of hand-written DPP instructions do not rest on the order the
compiler gives: in the assembly of every kernel, each inline-assembly block that reads
a DPP operand starts with the two wait states that a vector write before it needs, and
none of its instructions reads what another of the block has written (counting every
operand, the accumulator of a multiply-add too, as the compiler's own rule does)."""
import os
import re
import subprocess

import pytest

from paper_2412_07731_amd import build

FILES = [f for f in build.SOURCES if f.endswith(".hip")
         and "_dpp" in open(os.path.join(build.SRC, f)).read()]


def regs(op):
    """numbers of a vector register operand, v7 or v[8:9]"""
    m = re.match(r"v\[(\d+):(\d+)\]$", op) or re.match(r"v(\d+)()$", op)
    return set(range(int(m[1]), int(m[2] or m[1]) + 1)) if m else set()


def faults(asm):
    """what is wrong in the asm blocks of an assembly text"""
    out, seen = [], 0
    for block in re.findall(r";#ASMSTART\n(.*?)\n\s*;?;#ASMEND", asm, flags=re.S):
        lines = [s.strip() for s in block.splitlines() if s.strip() and not s.strip().startswith(";")]
        if not any("_dpp" in s for s in lines):
            continue
        seen += 1
        if lines[0] != "s_nop 1":
            out.append(f"no wait states before {lines[0]}")
        written = set()
        for s in lines:
            if "_dpp" not in s:
                continue
            ops = [o.strip() for o in s.split(" row_")[0].split(None, 1)[1].split(",")]
            read = set().union(*(regs(o) for o in (ops if "fmac" in s else ops[1:])))
            if read & written:
                out.append(f"{s} reads what the block wrote")
            written |= regs(ops[0])
    return seen, out


def test_checker():
    ok = ";#ASMSTART\n\ts_nop 1\n\tv_fmac_f64_dpp v[2:3], v[4:5], v[6:7] row_newbcast:1\n\t;;#ASMEND"
    assert faults(ok) == (1, [])
    assert faults(ok.replace("\ts_nop 1\n", ""))[1]
    assert faults(ok.replace("\n\t;;", "\n\tv_add_u32_dpp v9, v3, v8 row_newbcast:1\n\t;;"))[1]
    assert faults(ok.replace("\n\t;;", "\n\tv_fmac_f64_dpp v[2:3], v[4:5], v[8:9] row_newbcast:2\n\t;;"))[1]
    assert not faults(ok.replace("\n\t;;", "\n\tv_fmac_f64_dpp v[8:9], v[4:5], v[10:11] row_newbcast:2\n\t;;"))[1]


@pytest.mark.parametrize("name", FILES)
def test_waits(name, tmp_path):
    try:
        cc = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = tmp_path / "k.s"
    cmd = [cc] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.SRC, name), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    seen, wrong = faults(out.read_text())
    assert seen > 0
    assert not wrong, wrong[:5]
