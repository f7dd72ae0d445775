"""The issue-rate probe writes its matrix instructions as inline assembly, whose hazards the compiler does not handle: the
waits around them have to stand where the generated code needs them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2301_10936_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_waits_between_accumulator_moves_and_matrix_instructions(tmp_path):
    out = str(tmp_path / "probe.s")
    cmd = ["hipcc", *build.FLAGS, "--cuda-device-only", "-S", "-o", out, os.path.join(build.CSRC, "pit_probe.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    text = open(out).read()
    body = text[re.search(r"^_Z\S*k_rate_16x16x32\S*:", text, re.M).start():]
    ops = re.findall(r"^\s+(s_nop \d+|v_mfma\w+|v_accvgpr_(?:write|read)\w*|v_mov\w+)\b", body[:body.index("s_endpgm")], re.M)
    mfma = [i for i, op in enumerate(ops) if op.startswith("v_mfma")]
    states = lambda span: sum(int(op.split()[1]) + 1 for op in span if op.startswith("s_nop"))
    before = max(i for i in range(mfma[0]) if not ops[i].startswith("s_nop"))
    assert states(ops[before + 1:mfma[0]]) >= 2             # a vector write of an operand, then the matrix instruction
    after = next(i for i in range(mfma[-1] + 1, len(ops)) if ops[i].startswith("v_accvgpr_read"))
    assert states(ops[mfma[-1] + 1:after]) >= 11            # eight passes of the last matrix instruction, then a read
