"""The backward kernels issue their gradient products as inline-assembly MFMAs, whose operands the
compiler's hazard handling does not see: an MFMA may not read a register that a vector instruction
wrote in the two wait states before it. The kernels are compiled to assembly here and every such
MFMA is checked, and that the accumulators are read only behind the drain's wait states."""
import os
import re
import subprocess

import pytest

from paper_2606_13872_amd import build as b


def _regs(t):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", t)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.match(r"([va])(\d+)$", t)
    return {(m.group(1), int(m.group(2)))} if m else set()


def _scan(text):
    """(asm MFMAs, hazards, accumulator reads less than 12 wait states behind the MFMA that wrote it)"""
    count, hazards, early = 0, [], []
    left = False
    prev, in_asm, now, written = [], False, 0, {}  # wait states so far; when an accumulator was written
    for n, line in enumerate(text.splitlines(), 1):
        t = line.strip()
        if t.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if t.startswith(";;#ASMEND"):
            in_asm = False
            continue
        if not t or t.startswith(";") or re.match(r"^\.(?!LBB)", t):
            continue
        if re.match(r"^[.\w$]+:", t):
            prev = []
            if left:  # nothing falls through to here
                written.clear()
            continue
        op = t.split()[0]
        left = op in ("s_branch", "s_endpgm")
        args = [x.strip() for x in t[len(op):].split(";")[0].split(",")]
        if op == "s_nop":
            prev = (prev + [set()] * (int(args[0]) + 1))[-2:]
            now += int(args[0]) + 1
            continue
        now += 1
        if in_asm and op.startswith("v_mfma"):
            count += 1
            written.update((r, now) for r in _regs(args[0]))
            use = _regs(args[1]) | _regs(args[2])
            hazards += [(n, t) for w in prev if w & use]
        if op.startswith("v_accvgpr") and len(args) > 1 and any(now - written.get(r, -99) < 12 for r in _regs(args[1])):
            early.append((n, t))
        if op.startswith("v_accvgpr_") and op != "v_accvgpr_read_b32":
            for r in _regs(args[0]):
                written.pop(r, None)
        write = set()
        if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp")):
            write = _regs(args[0])
        prev = (prev + [write])[-2:]
    return count, hazards, early


@pytest.mark.parametrize("src", ["sra_grad.hip"])
def test_assembly_mfma_operands_are_settled(src, tmp_path):
    out = tmp_path / "k.s"
    cmd = [b.hipcc(), *b.HIP_FLAGS, *b.EXTRA_FLAGS.get(src, []), *b.COMMON, "--cuda-device-only", "-S",
           os.path.join(b.CSRC, src), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=b.COMPILE_TIMEOUT_S)
    count, hazards, early = _scan(out.read_text())
    assert count >= 4 * 32  # the products are there
    assert not hazards, hazards[:5]
    assert not early, early[:5]


def test_scan_sees_a_hazard():
    text = """
	v_cvt_pk_bf16_f32 v5, v1, v2
	;;#ASMSTART
	v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[4:7], a[0:3]
	;;#ASMEND
	v_accvgpr_read_b32 v0, a0
"""
    count, hazards, early = _scan(text)
    assert (count, len(hazards), len(early)) == (1, 1, 1)
    assert _scan(text.replace(";;#ASMSTART", "s_nop 1\n\t;;#ASMSTART"))[1] == []
