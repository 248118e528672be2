"""The generated code of the LM head, whose products and loads into LDS are
inline assembly that the compiler's hazard recogniser does not look into. The
wait states that CDNA4 asks for around them are either in that assembly or, for
the three checked here, come from where the compiler puts its own instructions:
in the code as compiled (44 s) they have to be there on every path."""

import functools
import os
import re
import subprocess

import pytest

from paper_2505_12398_amd import build as B

pytestmark = pytest.mark.slow

# wait states between a write and the instruction that depends on it
SCALAR_TO_LOAD = 5       # vector instruction writes a scalar register, a buffer load reads it
VECTOR_TO_PRODUCT = 2    # vector instruction writes a register, a product reads it
PRODUCT_TO_OTHER = 18    # a product writes accumulators, another instruction touches them


def _regs(operand):
    """Registers named by an operand: s5, v[2:3], a[0:3], vcc."""
    operand = operand.strip("|-")
    m = re.fullmatch(r"([sva])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if m:
        lo = int(m[2] or m[3])
        return {(m[1], i) for i in range(lo, int(m[2] or m[4]) + 1)}
    return {("s", operand)} if operand in ("vcc", "m0") else set()


@functools.lru_cache(maxsize=None)
def _parse(line):
    op, _, rest = line.partition(" ")
    return op, [_regs(x) for x in re.split(r"[ ,]+(?![^\[]*\])", rest.strip()) if x]


def _vector(op):
    return op.startswith("v_") and not op.startswith("v_mfma")


def _violation(before, line):
    """What the instruction lacks, given those before it (nearest last) and
    their wait states; None if it may issue."""
    op, operands = _parse(line)
    every = set().union(*operands) if operands else set()
    states = 0
    for prev in reversed(before):
        pop, pops = _parse(prev)
        wrote = pops[0] if pops else set()
        if _vector(pop) and op.startswith("buffer_load") and states < SCALAR_TO_LOAD:
            if any(r[0] == "s" for r in wrote & every):
                return f"{prev} -> {line}: {states} states"
        if _vector(pop) and op.startswith("v_mfma") and states < VECTOR_TO_PRODUCT:
            if wrote & every:
                return f"{prev} -> {line}: {states} states"
        if pop.startswith("v_mfma") and not op.startswith("v_mfma") and wrote & every:
            return f"{prev} -> {line}: {states} states"
        states += 1 + (int(prev.split()[1], 0) if pop == "s_nop" else 0)
        if states >= PRODUCT_TO_OTHER:
            break
    return None


def violations(text):
    """Hazards of one function's assembly, along falling through and along
    every branch to its label."""
    code, labels = [], {}
    for raw in text.split("\n"):
        line = raw.split(";")[0].strip()
        if re.fullmatch(r"\.L\w+:", line):
            labels[line[:-1]] = len(code)
        elif line and not line.startswith(".") and not line.endswith(":"):
            code.append(line)
    found = []
    for i, line in enumerate(code):
        fallen = code[max(0, i - 40):i]
        for k in range(len(fallen) - 1, -1, -1):     # what precedes a jump does not fall through
            if fallen[k].startswith(("s_branch", "s_endpgm")):
                fallen = fallen[k + 1:]
                break
        found.append(_violation(fallen, line))
        if line.startswith(("s_branch", "s_cbranch")):
            start = labels[line.split()[1]]
            for j in range(start, min(start + PRODUCT_TO_OTHER, len(code))):
                found.append(_violation(code[max(0, i - 40):i + 1] + code[start:j], code[j]))
    return [f for f in found if f]


@pytest.mark.parametrize("text,hazards", [
    ("v_readlane_b32 s9, v3, 1\ns_mov_b32 m0, s2\ns_nop 0\n"
     "buffer_load_dwordx4 v1, s[4:7], s9 offen lds", 1),
    ("v_readlane_b32 s9, v3, 1\ns_mov_b32 m0, s2\ns_nop 3\n"
     "buffer_load_dwordx4 v1, s[4:7], s9 offen lds", 0),
    ("v_mov_b32_e32 v5, v9\ns_nop 0\nv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", 1),
    ("v_mov_b32_e32 v5, v9\ns_nop 1\nv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", 0),
    ("v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]\ns_nop 15\ns_nop 0\n"
     "v_accvgpr_read_b32 v1, a2", 1),
    ("v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]\ns_nop 15\ns_nop 1\n"
     "v_accvgpr_read_b32 v1, a2", 0),
    (".LBB0_1:\nv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]\ns_nop 2\n"
     "v_mov_b32_e32 v8, v20\ns_cbranch_scc1 .LBB0_1\ns_endpgm", 1),
])
def test_the_check_sees_hazards(text, hazards):
    """The check itself, on lines with too few and just enough wait states."""
    assert len(violations(text)) == hazards


def test_lmhead_wait_states(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "lmhead.s"
    flags = [f for f in B.FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run([B.HIPCC, *flags, "--cuda-device-only", "-S", "-I", B.INCLUDE, "-I", B.CSRC,
                    os.path.join(B.CSRC, "tv_lmhead.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    text = out.read_text()
    kernels = re.findall(r"^(_ZN\S*lmhead_kernel\S*):\s*;.*?\n(.*?)^\.Lfunc_end", text,
                         re.M | re.S)
    assert len(kernels) == 24          # 8 tile heights x (tiles, ranges, ranges read once)
    for name, body in kernels:
        assert "v_mfma_f32_16x16x32_bf16" in body and re.search(r"offen (nt )?lds", body)
        assert violations(body) == [], name
