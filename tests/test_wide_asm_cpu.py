"""The wide GEMM issues its matrix instructions as inline asm, whose results the compiler does not wait for.  Every built instance is
therefore read back: nothing but matrix instructions touches an accumulator near a matrix instruction that writes it."""
import os
import re
import subprocess

import pytest

from paper_2406_13170_amd import build as bld

LLVM = "/opt/rocm/llvm/bin"
OBJ = os.path.join(bld.HERE, "_build", "gemm_skinny.o")
REG = re.compile(r"\ba(?:\[(\d+):(\d+)\]|(\d+)\b)")
# 16 x 16 instructions take 4 passes in bf16 and 8 in float32: their results are there for other units after at most 11 wait
# states; 4 lie between another unit's write and a matrix instruction's read
AFTER, BEFORE = 12, 4


def listing(tmp_path):
    fat, elf = str(tmp_path / "fat"), str(tmp_path / "dev.elf")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", OBJ, str(tmp_path / "copy.o")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}",
                    f"--output={elf}"], check=True)
    return subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", elf], check=True, capture_output=True, text=True).stdout


def regs(text):
    for m in REG.finditer(text):
        lo = int(m.group(1) or m.group(3))
        yield from range(lo, int(m.group(2) or lo) + 1)


def faults(lines):
    """Accesses of accumulators that come too early (in listing order), and the number of matrix instructions."""
    now, mfma, other, bad, n = 0, {}, {}, [], 0
    for line in lines:
        ins = line.strip().split("//")[0].strip()
        if not ins:
            continue
        now += int(ins.split()[1]) + 1 if ins.startswith("s_nop") else 1
        if ins.startswith("v_mfma"):
            n += 1
            dst, srcs = ins.split(",", 1)
            bad += [ins for r in regs(srcs.rsplit(",", 1)[1]) if now - other.get(r, -99) < BEFORE]
            mfma.update((r, now) for r in regs(dst))
        elif "a" in ins:
            for r in regs(ins):
                if now - mfma.get(r, -99) < AFTER:
                    bad.append(ins)
                other[r] = now
    return bad, n


def test_the_scan_sees_an_early_access():
    mm = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"
    assert faults([mm, "s_nop 15", "v_accvgpr_read_b32 v0, a3"]) == ([], 1)
    assert faults([mm, "s_nop 1", "v_accvgpr_read_b32 v0, a3"])[0]
    assert faults([mm] + ["v_add_u32_e32 v1, v1, v2"] * 8 + ["scratch_store_dwordx4 off, a[0:3], off"])[0]
    assert faults(["v_accvgpr_write_b32 a2, 0", mm])[0]


@pytest.mark.skipif(not (os.path.exists(OBJ) and os.path.exists(f"{LLVM}/llvm-objdump")), reason="no built object or no disassembler")
def test_nothing_touches_an_accumulator_too_early(tmp_path):
    kernels = 0
    for part in re.split(r"^<(\S+)>:$", listing(tmp_path), flags=re.M)[1:]:
        if part.startswith("_ZN4amph11k_gemm_wide"):
            name = part
            continue
        if not part.startswith("\n") or "v_mfma" not in part or "name" not in locals() or name is None:
            continue
        bad, n = faults(part.splitlines())
        assert n > 0 and not bad, (name, bad[:4])
        kernels, name = kernels + 1, None
    assert kernels == 72                                       # 56 instances in bf16, 16 in float32
