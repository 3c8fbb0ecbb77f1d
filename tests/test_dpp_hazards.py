"""Wait states of the row-broadcast instructions in the built kernels (no GPU
needed).  They are inline assembly, which the compiler's hazard handling does
not see into: a DPP operand must not be read within two wait states of its
write by a vector instruction, and no operand within 19 of its write by an
FP64 matrix instruction.  The sources keep the distances by the order of
their instructions; a copy or a reload that a compiler places between them
would break that silently."""
import re

import pytest

import device_code

pytestmark = pytest.mark.skipif(not device_code.available(), reason="library or LLVM tools not there")

REG = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")


def _regs(operand):
    out = set()
    for m in REG.finditer(operand):
        lo, hi = (int(m.group(1)), int(m.group(2))) if m.group(1) else (int(m.group(3)),) * 2
        out.update(range(lo, hi + 1))
    return out


def _hazards(lines):
    """(row broadcasts read, lines that read an operand too early)."""
    ins = [ln.split("//")[0].strip() for ln in lines]
    ins = [i for i in ins if i and not i.endswith(":") and not i.startswith("<")]
    count, bad = 0, []
    for at, text in enumerate(ins):
        if "row_newbcast" not in text:
            continue
        count += 1
        ops = text.split(None, 1)[1].split(",")
        source = _regs(ops[1])
        used = _regs(text.split("row_newbcast")[0])
        states, k = 0, at - 1
        while k >= 0 and states < 19:
            prev = ins[k].split(None, 1)
            if prev[0] == "s_nop":
                states += int(prev[1], 0) + 1
            else:
                if prev[0].startswith("v_") and len(prev) > 1:
                    written = _regs(prev[1].split(",")[0])
                    if (states < 2 and written & source) or (prev[0].startswith("v_mfma") and written & used):
                        bad.append((ins[k], text, states))
                states += 1
            k -= 1
    return count, bad


def test_the_check_finds_planted_hazards():
    dpp = "v_fmac_f64_dpp v[2:3], v[68:69], v[4:5] row_newbcast:0 row_mask:0xf bank_mask:0xf"
    mfma = "v_mfma_f64_16x16x4_f64 v[2:9], v[20:21], v[22:23], 0"
    assert _hazards(["v_mov_b32_e32 v69, v1", "s_nop 0", dpp])[1]
    assert _hazards(["v_mul_f64 v[68:69], v[8:9], v[10:11]", "v_mov_b32_e32 v1, v2", dpp])[1]
    assert _hazards([mfma] + ["s_nop 7"] * 2 + [dpp])[1]
    assert not _hazards(["v_mov_b32_e32 v69, v1", "s_nop 1", dpp])[1]
    assert not _hazards(["v_mov_b32_e32 v2, v1", dpp])[1]
    assert not _hazards([mfma] + ["s_nop 7"] * 3 + [dpp])[1]


def test_row_broadcasts_read_no_operand_too_early(tmp_path):
    count, bad = 0, []
    for obj in device_code.code_objects(tmp_path):
        n, b = _hazards(device_code.assembly(obj).splitlines())
        count += n
        bad += b
    assert count > 1000
    assert not bad, (len(bad), bad[:5])
