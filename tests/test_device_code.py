"""The device code that the build produced, read back (no GPU).

The copies from memory into LDS are written as inline assembly, inside which the
compiler inserts no wait states, so what the hardware asks for has to hold in the
code as built: one between a scalar write of m0 and the copy that reads it.
"""
import os
import re
import subprocess

import pytest

from paper_2607_05147_amd import build

LLVM = "/opt/rocm/llvm/bin"


def _code_object(src, tmp_path):
    obj = os.path.join(build.OBJDIR, os.path.basename(src) + ".o")
    if not os.path.exists(obj):
        build.build()
    fat, co = str(tmp_path / "fat"), str(tmp_path / "co")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", obj, str(tmp_path / "rest")],
                   check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={co}",
                    f"--targets=hipv4-amdgcn-amd-amdhsa--{build.ARCH}"], check=True)
    return co


def _instructions(co):
    """(kernel, opcode, operands) of every instruction, in program order."""
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", co], check=True, capture_output=True,
                          text=True).stdout
    kernel = None
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if m:
            kernel = m[1]
        elif line.startswith("\t"):
            words = line.split("//")[0].strip().split(None, 1)
            yield kernel, words[0], [x.strip() for x in words[1].split(",")] if len(words) > 1 else []


def _hazards(code):
    """Copies into LDS that come right after the write of m0 that they read."""
    found, copies, last = [], 0, (None, None, [""])
    for kernel, op, args in code:
        if op.startswith("global_load_lds"):
            copies += 1
            if last[0] == kernel and last[2][:1] == ["m0"]:
                found.append(f"{kernel}: {last[1]} {last[2]} right before {op} {args}")
        last = kernel, op, args
    return found, copies


def test_the_scan_sees_a_missing_wait():
    copy = ("k", "global_load_lds_dwordx4", ["v1", "s[0:1]"])
    m0, nop = ("k", "s_mov_b32", ["m0", "s4"]), ("k", "s_nop", ["0"])
    assert len(_hazards([m0, copy])[0]) == 1 and _hazards([m0, nop, copy]) == ([], 1)


@pytest.mark.parametrize("name", [os.path.basename(s) for s in build.sources()])
def test_copies_into_lds_wait_for_m0(name, tmp_path):
    found, copies = _hazards(_instructions(_code_object(os.path.join(build.CSRC, name), tmp_path)))
    assert not found, f"{len(found)} of {copies}: " + "; ".join(found[:3])
    assert copies > 0 or not name.startswith(("attn_m", "attn_stream"))
