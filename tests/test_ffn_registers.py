"""The bf16 expert products name their accumulation registers in asm statements.  That holds as long as the compiler itself uses
none of them and no operand of a matrix instruction is written by a vector instruction within the two wait states that the
hardware asks for: both are read off the assembly that it writes for these kernels."""
import os
import re
import subprocess

import pytest

from paper_2503_05066_amd import build


def _registers(operand):
    m = re.match(r"^([av])(?:\[(\w+):(\w+)\]|\[(\w+)\]|(\d+))$", operand.strip())
    if not m:
        return set()
    low = int(m[2] or m[4] or m[5], 0)
    return {(m[1], r) for r in range(low, (int(m[3], 0) if m[3] else low) + 1)}


def test_accumulators_belong_to_the_asm_statements(tmp_path):
    try:
        hipcc = build._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = tmp_path / "ffn.s"
    subprocess.run([hipcc, *build.COMMON, "--cuda-device-only", "-S", os.path.join(build.CSRC, "ffn.hip"), "-o", str(out)],
                   check=True, capture_output=True, timeout=600)
    inside, code, matrix = False, [], 0
    for line in out.read_text().splitlines():
        line = line.strip()
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
        elif line and not line.startswith((";", ".")) and not line.endswith(":") and re.match(r"^[a-z]+_", line):
            line = line.split(";")[0]
            name, _, rest = line.partition(" ")
            operands = [_registers(o) for o in re.split(r",\s*", rest)]
            if not inside:
                assert not any(kind == "a" for o in operands for kind, _ in o), line
            code.append((name, operands, line))
    for at, (name, operands, line) in enumerate(code):
        if not name.startswith("v_mfma"):
            continue
        matrix += 1
        used, states, back = set().union(*operands), 0, at - 1
        assert operands[0] and operands[1] and operands[2], line
        while states < 2 and back >= 0:
            other, written, text = code[back]
            if other == "s_nop":
                states += int(text.split()[1])
            elif other.startswith("v_") and not other.startswith("v_mfma"):
                wrote = written[0] | (written[1] if "swap" in other else set())
                assert not wrote & used, (text, line)
            states += 1
            back -= 1
    assert matrix > 5000  # every height of a tile, twice (how its weights are fetched), in three kernels
