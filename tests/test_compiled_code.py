"""CPU-side checks of the built library's gfx950 code: rules that the hardware does not enforce and
that the compiler keeps for its own instructions only."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_20022_amd import build, flexdraft as fd

WAIT_STATES = 5            # between a vector instruction that writes a scalar register and a memory instruction that reads it


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel name -> its instructions, in order."""
    objdump = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc()))), "llvm", "bin", "llvm-objdump")
    if not os.path.exists(objdump):
        objdump = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
    fd.load()
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(fd.LIB_PATH, d / "lib.so")
    subprocess.run([objdump, "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=d)
    out = {}
    for obj in glob.glob(str(d / "lib.so.*gfx950")):
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
        code = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
            if m:
                code = out.setdefault(m[1], [])
            elif code is not None and line.split("//")[0].strip():
                code.append(line.split("//")[0].strip())
    return out


def _scalar_registers(operands):
    regs = set()
    for lo, hi, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", operands):
        regs |= set(range(int(lo), int(hi) + 1)) if lo else {int(one)}
    return regs


def _early_scalar_reads(code):
    """Memory instructions that read a scalar register too soon after a vector instruction wrote it."""
    found, age = [], {}                                      # age: wait states since the write, while below WAIT_STATES
    for ins in code:
        op, _, operands = ins.partition(" ")
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            if any(r in age for r in _scalar_registers(operands)):
                found.append(ins)
        n = 1 + (int(operands, 0) if op == "s_nop" else 0)
        age = {r: a + n for r, a in age.items() if a + n < WAIT_STATES}
        if op.startswith("v_"):
            dst = [x.strip() for x in operands.split(",")]
            two = re.search(r"_co_|div_scale|mad_u64|mad_i64", op)      # the carry is a second destination
            for x in dst[:2 if two else 1]:
                if re.fullmatch(r"s\[\d+:\d+\]|s\d+", x):
                    age.update((r, 0) for r in _scalar_registers(x))
    return found


def test_the_check_finds_an_early_read():
    spill = ["v_readlane_b32 s7, v9, 3", "s_mov_b32 s2, m0", "s_mov_b32 m0, s83"]
    load = ["buffer_load_dwordx4 v1, s[4:7], 0 offen lds"]
    assert _early_scalar_reads(spill + ["s_nop 0"] + load) == load
    assert _early_scalar_reads(spill + ["s_nop 1"] + load) == load
    assert _early_scalar_reads(spill + ["s_nop 2"] + load) == []
    assert _early_scalar_reads(["v_readlane_b32 s8, v9, 3"] + load) == []


def test_memory_instructions_keep_their_distance_to_vector_written_scalars(kernels):
    assert any(" lds" in ins for name, code in kernels.items() if "attn_mfma_kernel" in name for ins in code)
    bad = {name: ins for name, code in kernels.items() for ins in [_early_scalar_reads(code)] if ins}
    assert not bad, bad


def test_new_length_is_stored_past_a_barrier(kernels):
    """fd_append_kv in place: every wave reads the old length before any wave may store the new one."""
    found = [code for name, code in kernels.items() if "append_kv_kernel" in name]
    assert len(found) == 2                                   # one per data type
    for code in found:
        store = [i for i, ins in enumerate(code) if re.match(r"global_store_dword ", ins)]          # (cache rows are dwordx4)
        assert len(store) == 1
        barrier = [i for i, ins in enumerate(code) if ins.startswith("s_barrier")]
        assert barrier and barrier[0] < store[0]
        copies = [i for i, ins in enumerate(code) if ins.startswith("global_store_dwordx4")]
        assert copies and max(copies) < barrier[0]
