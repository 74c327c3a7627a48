"""The MFMAs of the 256 x 256 tile and of the one-workgroup chain, and the transfers from memory to LDS of
every tile, are inline assembly.  The compiler then knows neither what they take nor how long they
run, so nothing that it puts around them is held back for them: a copy of an accumulator next to an
MFMA would read an unfinished result, an operand moved into place just ahead of one would be read
before it is there, and so would the resource of a transfer.  The built library is disassembled and
must hold no such code, along any path (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2505_23725_amd as mlc
from paper_2505_23725_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
GEMMS = ["ns_gemm_bf16_kernelILi256ELi256ELb0E", "ns_gemm_bf16_kernelILi256ELi256ELb1E"]
CHAINS = ["ns_chain_multi_kernelE", "ns_chain_small_kernelILi1E", "ns_chain_small_kernelILi2E", "ns_chain_small_kernelILi4E"]
# the compiler's own MFMAs, with transfers in assembly
SMALL = ["ns_gemm_bf16_kernelILi%dELi%dELb%dELi%dE" % (t, t, k, r) for t, r in ((64, 9), (128, 5), (128, 9)) for k in (0, 1)]
KERNELS = sorted(GEMMS + CHAINS + SMALL)
TWO_FORMS = [k for k in SMALL if "ILi64E" in k]       # results written through to memory, and not
# wait states (instructions, s_nop n counting n + 1) between
ACC_TO_READ = 11       # v_mfma_f32_16x16x32_bf16 (4 passes of 4 cycles) and a read of its result by another instruction
VALU_TO_MFMA = 2       # a vector instruction's result and an MFMA that has it as operand
VALU_TO_VMEM = 5       # a scalar register written by a vector instruction and a memory operation that reads it
M0_TO_LDS = 1          # a write of m0 and a transfer to LDS


class Instruction:
    def __init__(self, text, target=None):
        self.text = text
        self.op, _, rest = text.partition(" ")
        # an operand's modifiers ("offen lds", "offset:16") follow it after a space
        self.operands = [(p.split() or [""])[0] for p in rest.split(",")] if rest else []
        self.to_lds = self.op.startswith("buffer_load") and rest.split()[-1] == "lds"
        self.target = target               # index of the instruction that a branch goes to

    def registers(self, kind, operands=None):
        out = set()
        for o in self.operands if operands is None else operands:
            o = o.strip("-|")
            m = re.fullmatch(kind + r"\[(\d+):(\d+)\]", o) or re.fullmatch(kind + r"(\d+)", o)
            if m:
                out |= {kind + str(i) for i in range(int(m[1]), int(m[m.lastindex]) + 1)}
        return out

    def destinations(self):
        """Operands that a vector instruction writes."""
        if self.op.startswith(("v_swap", "v_permlane16_swap", "v_permlane32_swap", "v_div_scale", "v_mad_u64", "v_mad_i64")) or "_co_" in self.op:
            return self.operands[:2]
        return self.operands[:1]

    @property
    def mfma(self):
        return self.op.startswith(("v_mfma", "v_smfma"))

    @property
    def valu(self):
        return self.op.startswith("v_") and not self.mfma

    @property
    def vmem(self):
        return self.op.startswith(("buffer_", "global_", "flat_", "scratch_"))


def faults(code, mfma_by_hand):
    """What is wrong with a kernel's instructions.  A state says which registers are not there yet, and
    for how many wait states; where paths meet it is the longer wait of either."""
    found = set()
    joins = {ins.target for ins in code}

    def check(i, state):
        ins = code[i]

        def early(kind, regs):
            if any((kind, r) in state for r in regs):
                found.add("too early: " + ins.text)
        if ins.op.startswith(("s_setpc", "s_swappc", "s_call")):
            found.add("leaves the kernel: " + ins.text)
        if ins.vmem:
            early("lane", ins.registers("s") | {o for o in ins.operands if o in ("vcc", "m0")})
        if ins.to_lds:
            early("m0", ["m0"])
        if not mfma_by_hand:
            return
        if ins.op.startswith("scratch_"):
            found.add("spills: " + ins.text)
        if ins.mfma:
            if ins.operands[3] not in (ins.operands[0], "0"):
                found.add("adds to another accumulator: " + ins.text)
            early("operand", ins.registers("v", ins.operands[1:3]))
            if ins.registers("a", ins.operands[1:3]) or not ins.registers("a", ins.operands[:1]):
                found.add("operand out of place: " + ins.text)
        elif ins.op.startswith("v_accvgpr_read"):
            early("result", ins.registers("a"))
        elif ins.registers("a"):
            found.add("accumulators belong to MFMAs: " + ins.text)

    def after(i, state):
        ins = code[i]
        passed = int(ins.operands[0], 0) + 1 if ins.op == "s_nop" else 1
        out = {k: t - passed for k, t in state.items() if t > passed}
        if ins.mfma:
            out.update({("result", r): ACC_TO_READ for r in ins.registers("a", ins.operands[:1])})
        elif ins.valu:
            out.update({("operand", r): VALU_TO_MFMA for r in ins.registers("v", ins.destinations())})
            lane = ins.registers("s", ins.destinations()) | {o for o in ins.destinations() if o in ("vcc", "m0")}
            out.update({("lane", r): VALU_TO_VMEM for r in lane})
        if ins.op.startswith("s_") and ins.operands and ins.operands[0] == "m0":
            out[("m0", "m0")] = M0_TO_LDS
        return out

    entry = {0: {}}
    todo = [0]
    while todo:
        i = todo.pop()
        state = entry[i]
        while True:
            check(i, state)
            state = after(i, state)
            nexts = [] if code[i].op in ("s_endpgm", "s_branch") else [i + 1]
            if code[i].target is not None:
                nexts.append(code[i].target)
            if nexts == [i + 1] and i + 1 not in entry and i + 1 not in joins:
                i += 1
                continue
            for n in nexts:
                old = entry.get(n)
                new = {k: max((old or {}).get(k, 0), state.get(k, 0)) for k in {**(old or {}), **state}}
                if old is None or new != old:
                    entry[n] = new
                    todo.append(n)
            break
    return sorted(found)


def parse(lines):
    """Instructions from a listing with addresses: "op operands // 000000001234: words <symbol+0x10>"."""
    rows = []
    for line in lines:
        m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(?:.*<[^>+]*(?:\+(0x[0-9a-f]+))?>)?", line)
        if m:
            rows.append((m[1], int(m[2], 16), m[3]))
    at = {addr: i for i, (_, addr, _) in enumerate(rows)}
    return [Instruction(text, at[rows[0][1] + int(off or "0", 0)] if text.startswith(("s_branch", "s_cbranch")) else None)
            for text, _, off in rows]


def listing(tmp):
    shutil.copy(build.LIB_PATH, os.path.join(tmp, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(tmp)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp, check=True,
                              capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            head, _, body = part.partition("\n")
            for k in KERNELS:
                if k in head:                       # (a kernel's forms have its name in common)
                    out.setdefault(k, []).append(parse(body.splitlines()))
    return out


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_copy_of_an_accumulator_follows_its_mfma(tmp_path):
    mlc.library()
    code = listing(str(tmp_path))
    assert sorted(code) == KERNELS, sorted(code)
    assert {k: len(v) for k, v in code.items() if len(v) > 1} == {k: 2 for k in TWO_FORMS}
    for name, ins in ((k, one) for k, forms in code.items() for one in forms):
        mfmas = sum(i.mfma for i in ins)
        reads = sum(i.op.startswith("v_accvgpr_read") for i in ins)
        if name in GEMMS:      # 128 MFMAs a K tile in the unrolled ones and in the loop, 256 reads an epilogue
            assert mfmas % 128 == 0 and mfmas >= 5 * 128, (name, mfmas)
            assert reads % 256 == 0 and reads >= 5 * 256, (name, reads)
        else:
            assert mfmas and reads, (name, mfmas, reads)
        assert name in CHAINS or any(i.to_lds for i in ins), name
        assert not faults(ins, name not in SMALL), (name, faults(ins, name not in SMALL)[:5])


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_all_wavefronts_of_a_chain_meet_at_the_same_barriers(tmp_path):
    """Every barrier in the source stands once in the code of each form of the chain: none lies in a part that is
    compiled for some of a workgroup's wavefronts and again for others."""
    source = open(os.path.join(build.CSRC, "ns_chain_small.hip")).read()
    body = source[source.index("ns_chain_body(const ChainArgs"):source.index("ns_chain_small_kernel(ChainArgs")]
    barriers = body.count("__syncthreads();")
    assert barriers
    mlc.library()
    code = listing(str(tmp_path))
    for name in CHAINS:
        forms = 3 if "multi" in name else 1
        assert [sum(i.op == "s_barrier" for i in ins) for ins in code[name]] == [forms * barriers], name


MFMA = "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], a[0:3]"
LOAD = "buffer_load_dwordx4 v1, s[8:11], s12 offen lds"
GOOD = [
    [MFMA, "s_nop 10", "v_accvgpr_read_b32 v0, a3"],
    ["v_mov_b32_e32 v9, v0", "s_nop 1", MFMA],
    ["v_readfirstlane_b32 s12, v0", "s_nop 4", LOAD],
    ["s_add_u32 m0, s0, s1", "s_nop 0", LOAD],
    [MFMA, "s_branch 4", "v_accvgpr_read_b32 v0, a3", "s_endpgm", "s_nop 15", "v_accvgpr_read_b32 v0, a3"],
]
BAD = [
    [MFMA, "s_nop 9", "v_accvgpr_read_b32 v0, a3"],
    [MFMA, "s_nop 15", "v_accvgpr_mov_b32 a7, a3"],
    [MFMA, "s_nop 15", "v_accvgpr_write_b32 a3, v0"],
    [MFMA, "s_nop 15", "buffer_store_dwordx4 a[0:3], v1, s[8:11], 0 offen"],
    ["ds_read_b128 a[0:3], v1", "s_nop 15", MFMA],
    ["v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], a[4:7]"],
    ["v_mov_b32_e32 v15, v0", "s_nop 0", MFMA],
    ["v_swap_b32 v0, v8", "s_nop 0", MFMA],
    ["v_readlane_b32 s11, v0, 3", "s_nop 3", LOAD],
    ["v_cmp_eq_u32_e64 s[12:13], v0, v1", "s_nop 3", LOAD],
    ["s_add_u32 m0, s0, s1", LOAD],
    ["scratch_store_dword off, v0, s0"],
    ["s_swappc_b64 s[0:1], s[2:3]"],
    # along a branch: past what lies between, round a loop, and from the longer way of two that meet
    [MFMA, "s_branch 4", "s_nop 15", "s_endpgm", "v_accvgpr_read_b32 v0, a3"],
    ["v_accvgpr_read_b32 v0, a3", "s_nop 3", MFMA, "s_cbranch_scc1 0"],
    [MFMA, "s_cbranch_scc1 4", "s_nop 15", "v_add_u32_e32 v2, v2, v3", "v_accvgpr_read_b32 v0, a3"],
]


def assembled(lines):
    out = [Instruction(l) for l in lines]
    for ins in out:
        if ins.op.startswith(("s_branch", "s_cbranch")):
            ins.target = int(ins.operands[0])                 # here the index of an instruction
    return out + [Instruction("s_endpgm")]


@pytest.mark.parametrize("lines", GOOD)
def test_sound_listings_are_accepted(lines):
    assert not faults(assembled(lines), True)


@pytest.mark.parametrize("lines", BAD)
def test_faulty_listings_are_refused(lines):
    assert faults(assembled(lines), True)
