"""The device code that the build produced, read back (no GPU).

The copies from memory into LDS are written as inline assembly, inside which the
compiler inserts no wait states, so what the hardware asks for has to hold in the
code as built: one between a scalar write of m0 and the copy that reads it, and five
between a vector instruction's write of a scalar register and the copy that takes its
address from there.

The latent attention kernel keeps a few bytes of scratch memory that it does not use, for
the sake of what runs after it on the queue; how many it has is up to the compiler.
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


def _sgprs(operand):
    m = re.match(r"s\[(\d+):(\d+)\]|s(\d+)", operand)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def _hazards(code):
    """Copies into LDS that come too soon after the write of a scalar register that they
    read: m0, and the address registers written by a vector instruction."""
    m0, address, copies, before, now = [], [], 0, [], None
    for kernel, op, args in code:
        if kernel != now:
            before, now = [], kernel
        if op.startswith("global_load_lds"):
            copies += 1
            reads = set().union(*(_sgprs(a) for a in args))
            states = 0
            for o, a in reversed(before):
                if states < 1 and a[:1] == ["m0"]:
                    m0.append(f"{kernel}: {o} {a} right before {op} {args}")
                if o.startswith("v_") and a and _sgprs(a[0]) & reads:
                    address.append(f"{kernel}: {o} {a} {states} states before {op} {args}")
                states += int(a[0], 0) + 1 if o == "s_nop" else 1
                if states >= 5:
                    break
        before = before[-8:] + [(op, args)]
    return m0, address, copies


def test_the_scan_sees_a_missing_wait():
    copy, nop = ("k", "global_load_lds_dwordx4", ["v1", "s[0:1]"]), lambda n: ("k", "s_nop", [str(n)])
    m0, lane = ("k", "s_mov_b32", ["m0", "s4"]), ("k", "v_readfirstlane_b32", ["s1", "v2"])
    assert len(_hazards([m0, copy])[0]) == 1 and _hazards([m0, nop(0), copy]) == ([], [], 1)
    assert len(_hazards([lane, nop(3), copy])[1]) == 1 and _hazards([lane, nop(4), copy]) == ([], [], 1)


@pytest.fixture(scope="module", params=[os.path.basename(s) for s in build.sources()])
def copies(request, tmp_path_factory):
    code = _code_object(os.path.join(build.CSRC, request.param), tmp_path_factory.mktemp("code"))
    m0, address, n = _hazards(_instructions(code))
    assert n > 0 or not request.param.startswith(("attn_m", "attn_stream"))
    return m0, address, n


def test_copies_into_lds_wait_for_m0(copies):
    m0, _, n = copies
    assert not m0, f"{len(m0)} of {n}: " + "; ".join(m0[:3])


def test_copies_into_lds_wait_for_their_address(copies):
    _, address, n = copies
    assert not address, f"{len(address)} of {n}: " + "; ".join(address[:3])


def _scratch_bytes(co):
    """Scratch bytes per lane of every kernel."""
    text = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", co], check=True, capture_output=True, text=True).stdout
    names = re.findall(r"\.name: +(_Z\w+)", text)
    sizes = re.findall(r"\.private_segment_fixed_size: +(\d+)", text)
    assert len(names) == len(sizes) > 0
    return dict(zip(names, map(int, sizes)))


def test_latent_scratch_is_no_multiple_of_4_kb(tmp_path):
    # waves' scratch lies as far apart as the largest kernel run on the queue asked for, in
    # whole kilobytes; a multiple of 4 KB puts the spills of the drafter's kernels into few
    # cache sets
    sizes = _scratch_bytes(_code_object(os.path.join(build.CSRC, "attn_mla.hip"), tmp_path))
    (latent,) = [n for name, n in sizes.items() if "mla_kernel" in name]
    stride = -(-latent * 64 // 1024) * 1024
    assert stride % 4096, f"{latent} bytes a lane, {stride} a wave"
    drafter = _scratch_bytes(_code_object(os.path.join(build.CSRC, "markov.hip"), tmp_path))
    assert max(drafter.values()) < latent  # else the drafter's own size decides, and the bytes are for nothing
