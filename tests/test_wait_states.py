"""What the compiler does not look after in inline assembly, checked in the device code as it was built (no GPU).

gfx950 wants two wait states between a vector instruction that writes a scalar register (v_readlane, v_readfirstlane, a
compare) and a vector instruction that reads it.  The compiler keeps to that between instructions of its own, but does
not look into inline assembly."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_05346_amd import build as B

LLVM = "/opt/rocm/llvm/bin/"
WRITES_SCALAR = re.compile(r"v_(readlane|readfirstlane|cmp)")
pytestmark = pytest.mark.skipif(shutil.which(LLVM + "llvm-objdump") is None, reason="no llvm-objdump of ROCm")


def _scalars(operand):
    regs = set()
    for lo, hi, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", operand):
        regs |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return regs


def too_early(listing):
    """Pairs (writer, reader) with fewer than two wait states between them.  An instruction is one wait state, s_nop n is n + 1."""
    found, recent = [], []  # recent: (wait states since, registers, instruction)
    for line in listing.splitlines():
        line = line.split("//")[0].strip()
        if line.endswith(">:"):  # a function begins
            recent = []
        m = re.match(r"([a-z]+_\S+)\s*(.*)$", line)
        if not m or line.endswith(":"):
            continue
        op, args = m.groups()
        args = [a.strip() for a in re.split(r",(?![^\[]*\])", args)]
        waits = int(args[0], 0) + 1 if op == "s_nop" else 1
        if op.startswith("v_"):
            read = set().union(*(_scalars(a) for a in args[1:])) if len(args) > 1 else set()
            found += [(w, line) for _, regs, w in recent if regs & read]
        recent = [(n + waits, regs, w) for n, regs, w in recent if n + waits < 2]
        if WRITES_SCALAR.match(op) and _scalars(args[0]):
            recent.append((0, _scalars(args[0]), line))
    return found


def test_the_check_finds_what_it_looks_for():
    read, use = "\tv_readlane_b32 s80, v35, 1", "\tv_bfi_b32 v54, s80, 0, v51"
    other = "\tv_mul_f32_e32 v1, v2, v3"
    assert len(too_early("\n".join([read, use]))) == 1
    assert len(too_early("\n".join([read, other, use]))) == 1
    assert len(too_early("\n".join([read, "\ts_nop 0", use]))) == 1
    assert not too_early("\n".join([read, "\ts_nop 1", use]))
    assert not too_early("\n".join([read, other, "\tv_cmp_gt_f32_e64 s[4:5], v1, v2", use]))
    assert len(too_early("\n".join(["\tv_cmp_gt_f32_e64 s[4:5], v1, v2", "\tv_cndmask_b32_e64 v0, v1, v2, s[4:5]"]))) == 1


@pytest.mark.parametrize("source", B.SOURCES)
def test_vector_instructions_wait_for_scalars_from_vector_instructions(source, tmp_path):
    obj = os.path.join(B.OBJ, source.replace(".hip", ".o"))
    if not os.path.exists(obj):
        B.build()
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code.o")
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + bundle, obj, str(tmp_path / "rest.o")],
                   check=True)
    subprocess.run([LLVM + "clang-offload-bundler", "--unbundle", "--type=o",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + bundle, "--output=" + code], check=True)
    text = subprocess.run([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", code], check=True,
                          capture_output=True, text=True).stdout
    found = too_early(text)
    assert not found, (len(found), found[:3])
