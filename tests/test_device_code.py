"""The compiled gfx950 code of the library (no GPU needed): orderings inside
inline assembly that the compiler does not check.

A load into LDS takes its LDS base from M0.  CDNA needs one wait state between a
scalar write of M0 and such a load, and five between a vector instruction's
write of a scalar register and a vector-memory instruction that reads it; the
compiler places them around its own instructions only.
"""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2608_02123_amd import build as B
from paper_2608_02123_amd import pctree as P

LLVM = "/opt/rocm/llvm/bin"


def _instructions(path, tmp):
    """The library's device code: {kernel: [instruction]}."""
    fat, obj = str(tmp / "fatbin"), str(tmp / "gfx950.o")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", path,
                    str(tmp / "rest")], check=True)
    code, blob = {}, open(fat, "rb").read()
    # one bundle per source file, each at its own magic
    at = [m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob)] + [len(blob)]
    for i in range(len(at) - 1):
        part = str(tmp / f"part{i}")
        open(part, "wb").write(blob[at[i]:at[i + 1]])
        subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle",
                        f"--targets=hipv4-amdgcn-amd-amdhsa--{B.ARCH}", f"--input={part}",
                        f"--output={obj}"], check=True)
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn",
                               "--no-leading-addr", obj], check=True, capture_output=True,
                              text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"\s*<(\S+)>:$", line)
            if m:
                name = m.group(1)
                code[name] = []
            elif name and line.startswith(("\t", " ")) and line.strip():
                code[name].append(line.split("//")[0].strip())
    return code


def _wait_states(ins):
    m = re.match(r"s_nop (\d+)", ins)
    return int(m.group(1)) + 1 if m else 1


def _scalars(operands):
    """Scalar registers named in an operand string."""
    regs = set()
    for a, b, c in re.findall(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)", operands):
        regs |= set(range(int(a), int(b) + 1)) if a else {int(c)}
    return regs


@pytest.mark.parametrize("which", ["LIB_PATH", "TIMELINE_LIB_PATH"])
def test_lds_loads_wait_for_their_registers(which, tmp_path):
    code = _instructions(getattr(P, which), tmp_path)
    assert any("attn_direct_kernel" in n for n in code) and any("round_kernel" in n for n in code)
    loads = 0
    for name, ins in code.items():
        for i, line in enumerate(ins):
            if not re.match(r"(global|buffer)_load_lds|global_load_\S* .*\blds\b", line):
                continue
            loads += 1
            states, reads = 0, _scalars(line)
            for back in ins[max(0, i - 8):i][::-1]:
                if re.match(r"s_\w+ m0\b", back):
                    assert states >= 1, f"{name}: {back} / {line}"
                if re.match(r"v_(readfirstlane|readlane|cmp)", back):
                    dst = _scalars(back.split(",")[0])
                    assert not (dst & reads) or states >= 5, f"{name}: {back} / {line}"
                states += _wait_states(back)
    assert loads > 100, loads
