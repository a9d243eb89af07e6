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


def _llvm(tool):
    exe = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc()))), "llvm", "bin", tool)
    return exe if os.path.exists(exe) else shutil.which(tool) or "/opt/rocm/llvm/bin/" + tool


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    fd.load()
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(fd.LIB_PATH, d / "lib.so")
    subprocess.run([_llvm("llvm-objdump"), "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=d)
    return glob.glob(str(d / "lib.so.*gfx950"))


@pytest.fixture(scope="module")
def kernels(code_objects):
    """Kernel name -> its instructions, in order."""
    out = {}
    for obj in code_objects:
        text = subprocess.run([_llvm("llvm-objdump"), "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
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


def test_combine_kernel_requests_a_batch_at_once(kernels):
    """Twelve pieces of a row, or six where four lane groups share it: two vector loads each, and no wait for one of them before the last is requested."""
    seen = 0
    for name, code in kernels.items():
        m = re.search(r"attn_mfma_combine_kernelILi[24]ELi\d+ELi([14])E", name)
        if not m:
            continue
        seen += 1
        run = longest = 0
        for ins in code:
            if ins.startswith("global_load"):
                run += 1
                longest = max(longest, run)
            elif ins.startswith("s_waitcnt") and ("vmcnt" in ins or ins.split()[1] == "0"):
                run = 0
        assert longest >= (24 if m[1] == "1" else 12), (name, longest)
    assert seen == 8                                         # 64 and 128 rows, head dims 64 and 128, one lane group a row and four


def test_planned_kernels_along_the_line_spill_few_scalars(code_objects):
    """Each spilled scalar is a vector instruction where it is stored or used.  A branch before the walk over items doubled them (312 in the 64-row
    variant, 221 in the 128-row one: planned calls 2 to 16 % slower); without it there are 145 to 164."""
    spills = {}
    for obj in code_objects:
        notes = subprocess.run([_llvm("llvm-readelf"), "--notes", obj], check=True, capture_output=True, text=True).stdout
        names = re.findall(r"\.name: +(_ZN2fd\w+)", notes)
        counts = re.findall(r"\.sgpr_spill_count: +(\d+)", notes)
        assert len(names) == len(counts)
        spills.update(zip(names, map(int, counts)))
    planned = {m[1]: n for name, n in spills.items() for m in [re.search(r"attn_mfma_kernelI(Li[24]ELb1ELi\d+ELi0E)", name)] if m}
    assert len(planned) == 4 and max(planned.values()) <= 200, planned         # 64 and 128 rows, head dims 64 and 128
