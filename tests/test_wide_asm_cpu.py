"""The wide GEMM issues its matrix instructions as inline asm, of which the compiler knows neither how long an operand must have been
there nor how long a result takes.  Every built instance is therefore read back, along every path through its code: nothing but matrix
instructions touches an accumulator near a matrix instruction that writes it, and no vector instruction writes an operand just ahead of one
that reads it."""
import os
import re
import subprocess

import pytest

from paper_2406_13170_amd import build as bld

LLVM = "/opt/rocm/llvm/bin"
OBJ = os.path.join(bld.HERE, "_build", "gemm_skinny.o")
# 16 x 16 instructions take 4 passes in bf16 and 8 in float32: their results are there for other units after at most 11 wait
# states; 4 lie between another unit's write of an accumulator and a matrix instruction's read, 2 behind a vector instruction's write of
# one of the two factors
AFTER, BEFORE, FACTOR = 12, 4, 3


def listing(tmp_path):
    fat, elf = str(tmp_path / "fat"), str(tmp_path / "dev.elf")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", OBJ, str(tmp_path / "copy.o")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}",
                    f"--output={elf}"], check=True)
    return subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", elf], check=True, capture_output=True, text=True).stdout


def regs(kind, text):
    out = set()
    for m in re.finditer(rf"\b{kind}(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        lo = int(m.group(1) or m.group(3))
        out.update(range(lo, int(m.group(2) or lo) + 1))
    return out


class Ins:
    """One instruction: its wait states, the accumulators it touches, the vector registers that it writes on the vector unit, and, of a
    matrix instruction, its result, addend and factors."""

    def __init__(self, text):
        self.text = text
        op, _, args = text.partition(" ")
        args = [a.strip() for a in re.split(r",(?![^\[]*\])", args)]
        self.op, self.args = op, args
        self.states = int(args[0], 0) + 1 if op == "s_nop" else 1
        self.mfma = op.startswith("v_mfma")
        self.acc = regs("a", text) if not self.mfma else set()
        self.dst = regs("a", args[0]) if self.mfma else set()
        self.addend = regs("a", args[3]) if self.mfma else set()
        self.factors = regs("v", args[1]) | regs("v", args[2]) if self.mfma else set()
        written = args[:2] if "swap" in op else args[:1]
        self.writes = set().union(*(regs("v", a) for a in written)) if op.startswith("v_") and not self.mfma else set()


def flow(lines):
    """Instructions, and the places that each may be followed by."""
    code, at, names = [], {}, []
    for line in lines:
        m = re.match(r"\s+(\S.*?)\s*//\s*([0-9A-F]+):\s*((?:[0-9A-F]{8}\s*)+)", line)
        if not m:
            continue
        at[int(m.group(2), 16)] = len(code)
        names.append((int(m.group(2), 16), 4 * len(m.group(3).split())))
        code.append(Ins(m.group(1)))
    follow = []
    for i, (ins, (a, size)) in enumerate(zip(code, names)):
        nxt = [i + 1] if i + 1 < len(code) else []
        if ins.op.startswith(("s_cbranch", "s_branch")):
            off = int(ins.args[0], 0)
            to = at[a + size + 4 * (off - 65536 if off >= 32768 else off)]
            nxt = [to] if ins.op == "s_branch" else nxt + [to]
        elif ins.op == "s_setpc_b64":                             # a far branch: s_getpc, s_add, s_addc, s_setpc
            assert [c.op for c in code[i - 3:i]] == ["s_getpc_b64", "s_add_u32", "s_addc_u32"] and code[i - 1].args[2] == "0"
            nxt = [at[names[i - 2][0] + int(code[i - 2].args[2], 0)]]
        elif ins.op == "s_endpgm":
            nxt = []
        else:
            assert not ins.op.startswith(("s_call", "s_swappc", "s_rfe", "s_cbranch_i")), ins.text
        follow.append(nxt)
    return code, follow


def faults(lines):
    """Pairs of instructions that follow each other too closely, and the number of matrix instructions."""
    code, follow = flow(lines)

    def within(i, limit):
        """What is issued fewer than `limit` wait states behind instruction i, on any path."""
        seen, todo = {}, [(j, code[i].states) for j in follow[i]]
        while todo:
            j, t = todo.pop()
            if t >= limit or seen.get(j, limit) <= t:
                continue
            seen[j] = t
            todo += [(k, t + code[j].states) for k in follow[j]]
        return seen

    bad, n = [], 0
    for i, ins in enumerate(code):
        if ins.mfma:
            n += 1
            bad += [(ins.text, code[j].text) for j in within(i, AFTER) if code[j].acc & ins.dst]
        else:
            near = within(i, BEFORE if ins.acc else FACTOR) if ins.acc or ins.writes else {}
            bad += [(ins.text, code[j].text) for j, t in near.items() if code[j].mfma and
                    ((ins.acc & code[j].addend and t < BEFORE) or (ins.writes & code[j].factors and t < FACTOR))]
    return bad, n


def lines_of(*texts):
    return [f"\t{t} // {4 * i:012X}: 00000000" for i, t in enumerate(texts)]


def test_the_scan_sees_an_early_access():
    mm = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"
    assert faults(lines_of(mm, mm, "s_nop 15", "v_accvgpr_read_b32 v8, a3")) == ([], 2)
    assert faults(lines_of(mm, "s_nop 1", "v_accvgpr_read_b32 v0, a3"))[0]
    assert faults(lines_of(mm, *["v_add_u32_e32 v9, v9, v2"] * 8, "scratch_store_dwordx4 off, a[0:3], off"))[0]
    assert faults(lines_of("v_accvgpr_write_b32 a2, 0", mm))[0]
    assert faults(lines_of("v_add_u32_e32 v5, v9, v2", "s_nop 0", mm))[0]
    assert faults(lines_of("v_permlane32_swap_b32_e32 v9, v0", mm))[0]
    assert not faults(lines_of("v_add_u32_e32 v9, v0, v4", mm))[0]
    assert not faults(lines_of("v_add_u32_e32 v5, v9, v2", "s_nop 1", mm))[0]


def test_the_scan_follows_branches():
    mm = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"
    read = "v_accvgpr_read_b32 v8, a3"
    assert faults(lines_of(read, "s_nop 7", mm, "s_cbranch_scc1 65532", "s_endpgm"))[0] == [(mm, read)]      # round a loop
    assert faults(lines_of(mm, "s_cbranch_scc0 2", "s_nop 15", "s_endpgm", read, "s_endpgm"))[0] == [(mm, read)]
    assert faults(lines_of(mm, "s_branch 1", read, "s_endpgm"))[0] == []                                     # never reached from there
    far = [mm, "s_getpc_b64 s[0:1]", "s_add_u32 s0, s0, 0x14", "s_addc_u32 s1, s1, 0", "s_setpc_b64 s[0:1]", "s_endpgm", "s_endpgm"]
    assert faults(lines_of(*far, read))[0] == [(mm, read)]
    assert faults(lines_of(*far, "s_endpgm", read))[0] == []


@pytest.mark.skipif(not (os.path.exists(OBJ) and os.path.exists(f"{LLVM}/llvm-objdump")), reason="no built object or no disassembler")
def test_nothing_touches_an_operand_too_early(tmp_path):
    assert bld.built_from() == bld.sources_digest(), "the built objects are not those of the sources: build again"
    kernels = 0
    for name, part in re.findall(r"^[0-9a-f]+ <(_ZN4amph11k_gemm_wide\w+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", listing(tmp_path), flags=re.M | re.S):
        bad, n = faults(part.splitlines())
        assert n > 0 and not bad, (name, bad[:4])
        kernels += 1
    assert kernels == 72                                       # 56 instances in bf16, 16 in float32
