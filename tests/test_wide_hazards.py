"""Inline asm of the tiled kernels, around which the compiler puts no wait states: the built code must leave the distances that
the hardware needs (in wait states; an instruction is at least one).  Matrix instructions of ffn_wide.h: 2 from a vector
instruction that writes a register to a matrix instruction that reads it, 11 from a matrix instruction to any other instruction
that reads or writes its result (16 x 16 x 32 in bf16: 8 passes).  Direct loads to LDS (ffn_wide.h, ffn_tile.hip): 1 from a write
of m0, which holds their LDS address."""
import os
import re
import subprocess

import pytest

from paper_2201_05596_amd import build as B

LLVM = "/opt/rocm/llvm/bin"
BEFORE, AFTER = 2, 11
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def registers(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        out |= {(kind, i) for i in range(int(lo or one), int(hi or one) + 1)}
    return out


def operands(line):
    """(mnemonic, registers of the first operand, registers of the others)"""
    name, _, rest = line.partition(" ")
    first, _, others = rest.partition(",")
    return name, registers(first), registers(others)


def states(name, line):
    return int(line.split()[1], 0) + 1 if name == "s_nop" else 1


def find_hazards(code):
    """code: instruction lines of one kernel in memory order.  Branches are taken for falling through, and what precedes a
    branch target in memory for one of its predecessors; a backward branch is followed once from its loop's end to its start."""
    bad, pending, written = [], {}, {}      # register -> states since a matrix instruction / another vector instruction wrote it

    def walk(lines):
        for line in lines:
            name, first, others = operands(line)
            if name.startswith("v_mfma"):
                reads = others
                bad.extend((line, r, "before") for r in reads if written.get(r, BEFORE) < BEFORE)
                # a result that goes on as the same accumulator is forwarded; as an A or B operand it is not
                ab = registers(",".join(line.partition(" ")[2].split(",")[1:3]))
                bad.extend((line, r, "after") for r in ab if pending.get(r, AFTER) < AFTER)
            elif name.startswith(("v_", "ds_", "global_", "scratch_", "buffer_", "flat_")):
                bad.extend((line, r, "after") for r in first | others if pending.get(r, AFTER) < AFTER)
            n = states(name, line)
            for table, limit in ((pending, AFTER), (written, BEFORE)):
                for r in [r for r, d in table.items() if d + n >= limit]:
                    del table[r]
                for r in table:
                    table[r] += n
            if name.startswith("v_mfma"):
                pending.update((r, 0) for r in first)
            elif name.startswith("v_") and not name.startswith("v_cmp"):
                written.update((r, 0) for r in first)

    walk([line for _, line in code])
    index = {a: i for i, (a, _) in enumerate(code)}
    for i, (address, line) in enumerate(code):
        m = re.match(r"s_c?branch\S* (\d+)", line)
        if m:
            off = int(m.group(1))
            target = address + 4 + 4 * (off - 65536 if off >= 32768 else off)
            if target in index:
                pending.clear()
                written.clear()
                walk([text for _, text in code[max(0, i - 40):i + 1]])
                found = len(bad)
                walk([text for _, text in code[index[target]:index[target] + 20]])
                bad[found:] = [b + ("over a branch",) for b in bad[found:]]
    return bad


def find_m0_hazards(code):
    """Direct loads whose predecessor in memory writes m0.  (A predecessor over a branch is the branch: a wait state.)"""
    return [line for (_, before), (_, line) in zip(code, code[1:])
            if "_lds_" in line.split()[0] and re.match(r"s_\S+ m0\b", before)]


WIDE = ("wide_store", "wide_gelu", "wide_scatter")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    return disassemble(WIDE, tmp_path_factory)


@pytest.fixture(scope="module")
def tiled_kernels(tmp_path_factory):
    return disassemble(("tile",), tmp_path_factory)


def disassemble(names, tmp_path_factory):
    objs = [os.path.join(B.HERE, "_build", f"ffn_{n}.o") for n in names]
    if not all(map(os.path.exists, objs)) or not os.path.exists(LLVM + "/llvm-objdump"):
        pytest.skip("needs the built object files and llvm-objdump")
    found = {}
    for n, obj in enumerate(objs):
        fat = str(tmp_path_factory.mktemp("co") / f"{n}.fat")
        out = fat[:-4] + ".co"
        subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj, os.devnull], check=True, capture_output=True)
        subprocess.run([LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                        "--input=" + fat, "--output=" + out], check=True, capture_output=True)
        text = subprocess.run([LLVM + "/llvm-objdump", "-d", out], check=True, capture_output=True, text=True).stdout
        current = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                current = found.setdefault(m.group(1), [])
            elif current is not None and "//" in line:
                body, _, tail = line.partition("//")
                current.append((int(tail.strip().split(":")[0], 16), " ".join(body.split())))
    return {n: c for n, c in found.items() if "wide_kernel" in n or "tgemm_kernel" in n}


def test_built_code_keeps_the_distances(kernels):
    assert kernels
    for name, code in kernels.items():
        assert sum(line.startswith("v_mfma") for _, line in code) >= 224
        assert not find_hazards(code), name


def test_direct_loads_wait_for_m0(kernels, tiled_kernels):
    assert kernels and tiled_kernels
    for name, code in [*kernels.items(), *tiled_kernels.items()]:
        assert sum("_lds_" in line.split()[0] for _, line in code) >= 8
        assert not find_m0_hazards(code), name


def test_finds_planted_hazards():
    mfma = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"

    def hazards(*lines):
        return find_hazards([(4 * i, line) for i, line in enumerate(lines)])

    assert hazards(mfma, "v_accvgpr_mov_b32 a9, a2") and hazards(mfma, "s_nop 9", "v_accvgpr_read_b32 v9, a0")
    assert not hazards(mfma, "s_nop 10", "v_accvgpr_mov_b32 a9, a2") and not hazards(mfma, mfma)
    assert hazards("v_mov_b32_e32 v4, v9", mfma) and hazards("v_accvgpr_write_b32 a3, v9", "s_nop 0", mfma)
    assert not hazards("v_mov_b32_e32 v4, v9", "s_nop 1", mfma)
    assert hazards("v_accvgpr_read_b32 v9, a0", "s_nop 1", mfma, "s_cbranch_scc1 65532")

    def m0_hazards(*lines):
        return find_m0_hazards([(4 * i, line) for i, line in enumerate(lines)])

    load = "global_load_lds_dwordx4 v[2:3], off"
    assert m0_hazards("s_mov_b32 m0, s3", load) and m0_hazards("s_nop 0", "s_add_u32 m0, s3, 0x400", load)
    assert not m0_hazards("s_mov_b32 m0, s3", "s_nop 0", load) and not m0_hazards("s_mov_b32 s4, m0", load, load)
