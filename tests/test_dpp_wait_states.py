"""The factor's leaves use a DPP instruction in inline assembly, whose wait states the compiler does
not insert: a VGPR written by a vector instruction may be read through DPP two wait states later at
the earliest. Checked on the assembly that this compiler makes of the kernel."""
import re
import shutil
import subprocess

import pytest

from paper_2607_07964_amd import build as B

_REG = re.compile(r"^v(?:(\d+)|\[(\d+):(\d+)\])$")


def _vgprs(operand):
    m = _REG.match(operand.strip().rstrip(","))
    if not m:
        return set()
    return {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))


def dpp_hazards(asm: str):
    """(number of DPP instructions, those that read a register written less than two wait states
    before); straight through the text, so a branch's fall-through path is what is seen."""
    recent, found, bad = [], 0, []  # recent: (wait states since, registers written)
    for line in asm.splitlines():
        m = re.match(r"^\t([vsdgb]\w+)\s*(.*?)(?:;.*)?$", line)
        if not m:
            continue
        op, ops = m[1], re.findall(r"v\[\d+:\d+\]|[^,\s]+", m[2])
        if op.endswith("_dpp"):
            found += 1
            if any(age < 2 and regs & _vgprs(ops[1]) for age, regs in recent):
                bad.append(line.strip())
        states = int(ops[0], 0) + 1 if op == "s_nop" else 1
        recent = [(age + states, regs) for age, regs in recent if age + states < 2]
        if op.startswith("v_") and ops:
            regs = _vgprs(ops[0])
            if "swap" in op:
                regs = regs | _vgprs(ops[1])
            recent.append((0, regs))
    return found, bad


def test_dpp_hazard_rule():
    head = "\tv_add_f32_e32 v1, v2, v3\n"
    dpp = "\tv_fmac_f32_dpp v4, v1, v5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
    one = "\tv_mul_f32_e32 v9, v8, v8\n"
    assert len(dpp_hazards(head + dpp)[1]) == 1
    assert len(dpp_hazards(head + one + dpp)[1]) == 1
    assert len(dpp_hazards(head + "\ts_nop 0\n" + dpp)[1]) == 1
    assert dpp_hazards(head + one + one + dpp) == (1, [])
    assert dpp_hazards(head + "\ts_nop 1\n" + dpp) == (1, [])
    assert len(dpp_hazards("\tv_permlane32_swap_b32_e32 v7, v1\n" + dpp)[1]) == 1


@pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="no hipcc here")
def test_chol_dpp_wait_states(tmp_path):
    out = tmp_path / "chol.s"
    subprocess.run([B.HIPCC, *B.FLAGS, "-x", "hip", "--offload-device-only", "-S",
                    f"{B.CSRC}/chol.hip", "-o", str(out)], check=True, capture_output=True)
    found, bad = dpp_hazards(out.read_text())
    assert found > 1000 and bad == []
