"""The built two-label aggregation kernels keep the wait states that the
compiler cannot see: v_min_u32_sdwa is written in inline assembly, and a DPP
instruction that reads its result needs two instructions (or wait states)
between.  Checked on the disassembly of the objects the library is linked
from."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2112_00821_amd", "_build")
LLVM = "/opt/rocm/llvm/bin"


def _instructions(name, tmp):
    obj = os.path.join(BUILD, name)
    if not os.path.exists(obj):
        pytest.skip(f"{name} is not here (the build's objects stay where it ran)")
    co = str(tmp / "code.co")
    subprocess.run(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", obj, str(tmp / "fat")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={tmp / 'fat'}", f"--output={co}"], check=True)
    out = subprocess.run([f"{LLVM}/llvm-objdump", "-d", co], check=True, capture_output=True, text=True).stdout
    for line in out.splitlines():
        m = re.match(r"\s+([vsdgb]\w+)\s*(.*?)\s*//", line)
        if m:
            yield m[1], m[2]


def _registers(operand):
    m = re.fullmatch(r"v(\d+)", operand) or re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    return set(range(int(m[1]), int(m[m.lastindex]) + 1)) if m else set()


@pytest.mark.parametrize("pairs", [1, 2, 3, 4])
def test_sdwa_before_dpp(tmp_path, pairs):
    pending = {}     # register -> wait states since a v_min_u32_sdwa wrote it
    seen = 0
    for op, args in _instructions(f"k_sgm_pk{pairs}.o", tmp_path):
        operands = [a.strip().split()[0] for a in args.split(",") if a.strip()]
        if "dpp" in op or "row_" in args or "quad_perm" in args:
            for o in operands[1:]:
                for r in _registers(o):
                    assert pending.get(r, 9) >= 2, (op, args)
        states = int(args) + 1 if op == "s_nop" else 1
        pending = {r: n + states for r, n in pending.items() if n + states < 2}
        if op.startswith("v_") and operands:
            for r in _registers(operands[0]):
                pending.pop(r, None)
        if op == "v_min_u32_sdwa":
            seen += 1
            pending.update({r: 0 for r in _registers(operands[0])})
    assert seen > 0
