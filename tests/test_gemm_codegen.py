"""The MFMAs of the 256 x 256 tile and of the one-workgroup chain are written as inline assembly, so that
the compiler keeps every accumulator where it is.  It then also knows nothing of their latency: a copy
of an accumulator that it put next to one would read an unfinished result.  The built library is
disassembled and must hold no such copy (no GPU needed)."""
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
KERNELS = sorted(GEMMS + CHAINS)
# v_mfma_f32_16x16x32_bf16 takes 4 passes of 4 cycles; its result may be read 11 wait states after it
WAIT_STATES = 11


def listing(tmp):
    shutil.copy(build.LIB_PATH, os.path.join(tmp, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(tmp)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", f], cwd=tmp, check=True,
                              capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]* ?<)", text):
            head, _, body = part.partition("\n")
            for k in KERNELS:
                if k in head:
                    out[k] = [l.split("//")[0].strip() for l in body.splitlines() if l.strip()]
    return out


def accumulators(operand):
    m = re.match(r"a\[(\d+):(\d+)\]$", operand) or re.match(r"a(\d+)$", operand)
    return range(int(m[1]), int(m[m.lastindex]) + 1) if m else range(0)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_copy_of_an_accumulator_follows_its_mfma(tmp_path):
    mlc.library()
    code = listing(str(tmp_path))
    assert sorted(code) == KERNELS, sorted(code)
    for name, lines in code.items():
        busy = {}                                  # accumulator -> wait states until it may be read
        mfmas = reads = 0
        for line in lines:
            op, _, rest = line.partition(" ")
            assert not op.startswith("scratch_"), f"{name}: spills: {line}"
            assert not op.startswith("v_accvgpr_write"), f"{name}: accumulators are written by MFMAs only: {line}"
            passed = int(rest.split()[0], 0) + 1 if op == "s_nop" else 1
            busy = {a: t - passed for a, t in busy.items() if t > passed}
            regs = [r.strip() for r in rest.split(",")]
            if op.startswith("v_mfma"):
                mfmas += 1
                assert regs[3] in (regs[0], "0"), f"{name}: an MFMA adds to another accumulator: {line}"
                for a in accumulators(regs[0]):
                    busy[a] = WAIT_STATES
            elif op.startswith("v_accvgpr_read"):
                reads += 1
                late = [a for a in accumulators(regs[1]) if a in busy]
                assert not late, f"{name}: read too early: {line}"
        if name in GEMMS:      # 128 MFMAs a K tile in the unrolled ones and in the loop, 256 reads an epilogue
            assert mfmas % 128 == 0 and mfmas >= 5 * 128, (name, mfmas)
            assert reads % 256 == 0 and reads >= 5 * 256, (name, reads)
        else:
            assert mfmas and reads, (name, mfmas, reads)
