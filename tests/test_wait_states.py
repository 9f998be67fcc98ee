"""Compiler output check (no GPU): the broadcasting multiply-adds of the eigensolver are inline assembly, and the compiler keeps no
wait states for those: two must lie between a vector instruction that writes a register and a multiply-add that broadcasts it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _registers(operand):
    m = re.match(r"-?v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"-?v(\d+)\b", operand)
    return {int(m[1])} if m else set()


def broadcasts_too_early(text):
    """(number of broadcasting multiply-adds, those whose broadcast register a vector instruction may have written less than two
    wait states before, on any way there)."""
    code, at, jumps = [], {}, {}   # instructions (opcode, operands, line); label -> its instruction; label -> branches to it
    for number, line in enumerate(text.splitlines(), 1):
        line = line.split(";")[0].strip()
        label = re.match(r"([.\w$]+):", line)
        if label:
            at[label[1]] = len(code)
        elif line and not line.startswith("."):
            op, _, rest = line.partition(" ")
            args = [a.strip() for a in rest.split(",")]
            if op.startswith(("s_branch", "s_cbranch")):
                jumps.setdefault(args[0], []).append(len(code))
            code.append((op, args, number))
    came = {}   # instruction -> branches that lead to it
    for label, sites in jumps.items():
        came.setdefault(at[label], []).extend(sites)

    def written(i, source, states):   # within `states` wait states in front of instruction i
        if states <= 0:
            return False
        ways = list(came.get(i, []))
        if i > 0 and code[i - 1][0] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            ways.append(i - 1)
        for j in ways:
            op, args, _ = code[j]
            if op.startswith("v_") and _registers(args[0]) & source:
                return True
            if written(j, source, states - (1 + int(args[0], 0) if op == "s_nop" else 1)):
                return True
        return False

    places = [i for i, (op, _, _) in enumerate(code) if op == "v_fmac_f64_dpp"]
    assert all(_registers(code[i][1][1]) for i in places)
    return len(places), [code[i] for i in places if written(i, _registers(code[i][1][1]), 2)]


def test_the_check_finds_a_planted_violation():
    good = "v_mul_f64 v[2:3], v[4:5], v[6:7]\ns_nop 1\nv_fmac_f64_dpp v[8:9], v[2:3], v[0:1] row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
    assert broadcasts_too_early(good) == (1, [])
    jump = ".LBB0_1:\n" + good.replace("v_mul_f64 v[2:3], v[4:5], v[6:7]\ns_nop 1\n", "") + "s_nop 0\nv_mov_b32_e32 v2, v9\ns_cbranch_vccnz .LBB0_1\n"
    assert broadcasts_too_early(jump.replace("s_cbranch", "s_nop 1\ns_cbranch")) == (1, [])
    for bad in (good.replace("s_nop 1\n", ""), good.replace("s_nop 1", "s_nop 0"), good.replace("s_nop 1", "s_nop 1\nv_mov_b32_e32 v3, v9"),
                good.replace("s_nop 1\n", ".LBB0_1:\n"), jump):
        assert len(broadcasts_too_early(bad)[1]) == 1, bad


@pytest.mark.parametrize("name", ["tridiag", "tdeig"])
def test_broadcast_registers_have_settled(name, tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    from paper_2503_10501_amd import build
    out = tmp_path / (name + ".s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, name + ".hip"), "-o", str(out)], check=True,
                   capture_output=True, timeout=600)
    count, early = broadcasts_too_early(out.read_text())
    assert count > 100
    assert not early, early[:5]
