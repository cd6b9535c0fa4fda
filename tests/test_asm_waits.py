"""Wait states around inline assembly in the compiled kernels (no GPU needed).

gfx950 needs wait states between some instructions, and the compiler, which inserts them
for its own instructions, does not look inside inline assembly.  Every source with inline
assembly is compiled to gfx950 assembly with the build's flags and each instruction
written by hand is checked against the rules that can apply to it, in program order:
  - a scalar register written by the vector ALU (v_readlane and the like) and read by the
    vector ALU: 2 wait states;
  - a vector register written by the vector ALU and read by a matrix product, a lane
    permutation or a DPP operand: 2;
  - a matrix product's result read or written, or its third source written, by the vector
    ALU: up to 18 for the 16 x 16 products; held to be waited out once any compiled
    instruction has read that result.
"""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2605_08451_amd import build as lib_build

MFMA_WAIT = 18
WINDOW = 40
_REG = re.compile(r"(?<![\w.])-?\|?([vsa])(?:(\d+)|\[(\d+):(\d+)\])\|?")


def regs(text, kinds="vs"):
    out = set()
    for kind, one, lo, hi in _REG.findall(text):
        if kind in kinds:
            out |= {(kind, int(one))} if one else {(kind, r) for r in range(int(lo), int(hi) + 1)}
    if "s" in kinds and re.search(r"(?<!\w)vcc(?!\w)", text):
        out.add(("s", "vcc"))
    return out


def parse(line):
    """(mnemonic, operand texts) of an instruction line, or None."""
    line = line.split(";")[0].strip()
    if not line or line.startswith(".") or line.endswith(":") or not re.match(r"[a-z]\w+", line):
        return None
    op, _, rest = line.partition(" ")
    return op, [o.strip() for o in re.split(r",(?![^\[]*\])", rest)] if rest else []


def hazards(asm):
    """The rules' violations in an assembly text, one message each."""
    found = []
    hist = []   # newest last: dict(ws, op, hand, vw, sw, d, c, read)
    hand = False
    for no, line in enumerate(asm.splitlines(), 1):
        if "ASMSTART" in line or "ASMEND" in line:
            hand = "ASMSTART" in line
            continue
        ins = parse(line)
        if ins is None:
            continue
        op, ops = ins
        if op in ("s_endpgm", "s_branch", "s_setpc_b64"):
            hist = []
            continue
        valu = op.startswith("v_")
        mfma = op.startswith("v_mfma")
        ndst = 0 if not valu else 2 if op.startswith("v_permlane") and "swap" in op or op.startswith("v_swap") else 1
        writes = set().union(*(regs(o) for o in ops[:ndst])) if ndst else set()
        # a store's or a compare's first operand is read as well; swaps read what they write
        srcs = ops if not valu or ndst == 2 else ops[1:]
        reads = set().union(*(regs(o) for o in srcs)) if srcs else set()
        if valu and any(m in op for m in ("_fmac_", "_dot", "_mac_")):
            reads |= writes
        ws = 0
        for prev in reversed(hist):
            if ws >= MFMA_WAIT:
                break
            if hand and valu and ws < 2 and prev["valu"]:
                bad = {r for r in prev["writes"] & reads if r[0] == "s"}
                if bad:
                    found.append(f"line {no}: {line.strip()} reads {sorted(bad, key=str)} {ws} wait states after {prev['op']}")
            needs_two = mfma or (op.startswith("v_permlane")) or op.endswith("_dpp") or " row_" in line or "quad_perm" in line
            if needs_two and prev["hand"] and prev["valu"] and ws < 2:
                bad = {r for r in prev["writes"] & reads if r[0] == "v"}
                if bad:
                    found.append(f"line {no}: {op} reads {sorted(bad)} {ws} wait states after hand-written {prev['op']}")
            if hand and valu and prev["mfma"] and not prev["done"]:
                bad = (prev["writes"] & (reads | writes)) | (prev["c"] & writes)
                if bad:
                    found.append(f"line {no}: {line.strip()} touches {sorted(bad)} {ws} wait states after {prev['op']}")
            ws += prev["ws"]
        if not hand:
            for prev in hist:
                if prev["mfma"] and prev["writes"] & reads and not mfma:
                    prev["done"] = True   # the compiler waited for it here
        states = 1 + (int(ops[0]) if op == "s_nop" else 0)
        hist.append(dict(ws=states, op=op, hand=hand, valu=valu, mfma=mfma, writes=writes, done=False,
                         c=regs(ops[3]) if mfma and len(ops) > 3 else set()))
        del hist[:-WINDOW]
    return found


def compile_asm(src):
    cmd = [lib_build.hipcc(), *lib_build._flags(), "-x", "hip", "--cuda-device-only", "-S",
           os.path.join(lib_build.CSRC, src), "-o", "-"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout


def sources_with_inline_asm():
    """Every compiled source whose text, or whose headers of this repository, has asm."""
    def has_asm(path, seen):
        if path in seen or not os.path.exists(path):
            return False
        seen.add(path)
        text = re.sub(r"//[^\n]*", "", open(path).read())
        return bool(re.search(r"\basm\b", text)) or any(
            has_asm(os.path.join(lib_build.CSRC, h), seen) for h in re.findall(r'#include "([^"]+)"', text))
    return [s for s in lib_build.SOURCES if s.endswith(".hip") and has_asm(os.path.join(lib_build.CSRC, s), set())]


@pytest.mark.parametrize("text, n", [
    ("v_readlane_b32 s0, v2, 0\n;;#ASMSTART\nv_pk_mul_f16 v8, v61, s0 op_sel_hi:[0,1]\n;;#ASMEND", 1),
    ("v_readlane_b32 s0, v2, 0\ns_nop 1\n;;#ASMSTART\nv_pk_mul_f16 v8, v61, s0\n;;#ASMEND", 0),
    (";;#ASMSTART\nv_pk_add_f16 v5, v6, v7\n;;#ASMEND\nv_mfma_f32_16x16x32_f16 v[0:3], v[8:11], v[4:7], 0", 1),
    (";;#ASMSTART\nv_pk_add_f16 v5, v6, v7\n;;#ASMEND\ns_nop 1\nv_mfma_f32_16x16x32_f16 v[0:3], v[8:11], v[4:7], 0", 0),
    ("v_mfma_f32_16x16x32_f16 v[0:3], v[8:11], v[4:7], 0\n;;#ASMSTART\nv_pk_add_f16 v5, v2, v7\n;;#ASMEND", 1),
    ("v_mfma_f32_16x16x32_f16 v[0:3], v[8:11], v[4:7], 0\nv_mov_b32_e32 v9, v3\n;;#ASMSTART\nv_pk_add_f16 v5, v2, v7\n;;#ASMEND", 0),
])
def test_checker(text, n):
    assert len(hazards(text)) == n


def test_no_hand_written_instruction_misses_a_wait():
    srcs = sources_with_inline_asm()
    assert {"col_mfma.hip", "row_dense.hip"} <= set(srcs)
    with concurrent.futures.ThreadPoolExecutor(max_workers=4) as ex:
        for src, asm in zip(srcs, ex.map(compile_asm, srcs)):
            bad = hazards(asm)
            assert not bad, f"{src}: {len(bad)}: " + "; ".join(bad[:5])
