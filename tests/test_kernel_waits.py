"""Waits that inline assembly has to spell out, checked in the machine code of the built library: the compiler places
them for its own instructions but does not look inside an asm string."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2408_00264_amd import clover

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel name: its instructions in program order}"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(clover.LIB_PATH):
        from paper_2408_00264_amd import build
        build.build()
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(clover.LIB_PATH, d)            # (the code objects are written beside their library)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, capture_output=True)
    out, ins = {}, None
    for name in sorted(os.listdir(d)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", name], cwd=d, check=True, capture_output=True, text=True).stdout
        for line in text.splitlines():
            head = re.match(r"[0-9a-f]+ <(.*)>:$", line)
            if head:
                ins = out.setdefault(head[1], [])
            elif ins is not None and line.startswith("\t"):
                ins.append(line.split("//")[0].strip())
    return out


def wait_states(ins):
    """of one instruction: s_nop N stands for N + 1 of them"""
    return int(ins.split()[1], 0) + 1 if ins.startswith("s_nop") else 1


def test_lds_loads_wait_for_their_m0(kernels):
    """gfx950: one wait state between a scalar write of M0 and a load to the LDS that takes its address from it"""
    n = 0
    for name, code in kernels.items():
        for i, ins in enumerate(code):
            if not re.match(r"(global|buffer)_load_lds_", ins):
                continue
            n += 1
            states = 0
            for before in reversed(code[max(0, i - 8):i]):
                if re.match(r"s_\w+ m0,", before):
                    assert states >= 1, (name, before, ins)
                    break
                states += wait_states(before)
    assert n > 100, n                                # the GEMM's and the attention's staging loads


def test_accumulators_are_read_behind_the_wait(kernels):
    """The GEMM's matrix instructions are asm statements: 8 wait states (what the compiler places for its own) between the
    last of them and the first read of an accumulator must come from a no-op, not from whatever was scheduled in between."""
    n = 0
    for name, code in kernels.items():
        if "gemm_tile_kernel" not in name:
            continue
        nop = 0
        for ins in code:
            if ins.startswith("v_mfma"):
                nop = 0
            elif ins.startswith("s_nop"):
                nop = max(nop, wait_states(ins))
            elif ins.startswith("v_accvgpr_read"):
                assert nop >= 8, (name, ins)
                n += 1
    assert n > 100, n


def test_every_lds_load_of_the_gemm_has_an_m0_of_its_own(kernels):
    """The GEMM writes M0 in one asm statement and loads in a later one, and the load does not say that it reads M0: between two
    loads there must be exactly one write of M0, the GEMM's own, and no jump between it and its load."""
    n = 0
    for name, code in kernels.items():
        if "gemm_tile_kernel" not in name:
            continue
        since = []                                   # writes of M0, and jumps behind the last of them
        for ins in code:
            if re.match(r"global_load_lds_", ins):
                assert len(since) == 1 and since[0].startswith("s_add_u32 m0,"), (name, since, ins)
                n, since = n + 1, []
            elif re.match(r"[sv]_\w+ m0\b", ins):
                since.append(ins)
            elif since and re.match(r"s_c?branch|s_setpc|s_swappc|s_call", ins):
                since.append(ins)
    assert n > 1000, n
