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


def _merge(states):
    """What may have happened just before a label: the registers that any way there wrote in each of the two
    wait states, and the shortest time since an asm MFMA wrote an accumulator."""
    window, age = [set(), set()], {}
    for w, a in states:
        window = [x | y for x, y in zip(window, w)]
        for r, t in a.items():
            age[r] = min(t, age.get(r, t))
    return window, age


def _pass(lines, entries):
    """One walk over the listing; `entries`: label -> states at the branches to it (of the walk before).
    Returns (asm MFMAs, hazards, early reads, states at the branches of this walk)."""
    count, hazards, early, out = 0, [], [], {}
    window, age, in_asm, falls = [set(), set()], {}, False, False
    for n, t in lines:
        if t.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if t.startswith(";;#ASMEND"):
            in_asm = False
            continue
        if not t or t.startswith(";") or re.match(r"^\.(?!LBB)", t):
            continue
        label = re.match(r"^([.\w$]+):", t)
        if label:
            window, age = _merge(([(window, age)] if falls else []) + entries.get(label.group(1), []))
            falls = True
            continue
        op = t.split()[0]
        args = [x.strip() for x in t[len(op):].split(";")[0].split(",")]
        states = int(args[0]) + 1 if op == "s_nop" else 1
        age = {r: x + states for r, x in age.items() if x + states < 64}
        write = set()
        if in_asm and op.startswith("v_mfma"):
            count += 1
            use = _regs(args[1]) | _regs(args[2])
            hazards += [(n, t) for w in window if w & use]
            age.update((r, 0) for r in _regs(args[0]))
        elif op.startswith("v_accvgpr"):
            if len(args) > 1 and any(age.get(r, 99) < 12 for r in _regs(args[1])):
                early.append((n, t))
            if op != "v_accvgpr_read_b32":
                for r in _regs(args[0]):
                    age.pop(r, None)
        if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp")):
            write = _regs(args[0])
        window = (window + [write] + [set()] * (states - 1))[-2:]
        if op.startswith(("s_branch", "s_cbranch")):
            out.setdefault(args[0], []).append((window, age))
        falls = op not in ("s_branch", "s_endpgm", "s_setpc_b64")
        if not falls:
            window, age = [set(), set()], {}
    return count, hazards, early, out


def _scan(text):
    """(asm MFMAs, hazards, accumulator reads less than 12 wait states behind the MFMA that wrote it), over
    every way into a block: it falls through from the block before, and is branched to."""
    lines = [(n, x.strip()) for n, x in enumerate(text.splitlines(), 1)]
    entries = {}
    for _ in range(3):  # states travel through blocks shorter than the window
        count, hazards, early, entries = _pass(lines, entries)
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


def test_scan_looks_across_block_boundaries():
    head = "\tv_cvt_pk_bf16_f32 v5, v1, v2\n"
    mfma = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[4:7], a[0:3]\n\t;;#ASMEND\n"
    fall = "k:\n" + head + ".LBB0_1:\n" + mfma
    assert len(_scan(fall)[1]) == 1
    jump = "k:\n\ts_branch .LBB0_1\n.LBB0_2:\n\ts_nop 7\n.LBB0_1:\n" + mfma + head + "\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n"
    assert len(_scan(jump)[1]) == 1  # one wait state, the branch, between the write and the MFMA
    assert _scan(jump.replace("\ts_cbranch", "\ts_nop 0\n\ts_cbranch"))[1] == []
    read = "k:\n" + mfma + ".LBB0_1:\n\tv_accvgpr_read_b32 v0, a0\n"
    assert len(_scan(read)[2]) == 1
    assert _scan("k:\n" + head + "\ts_endpgm\nl:\n" + mfma)[1] == []
