"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header
declares, and its pure-host entry points (workspace queries, argument validation)
behave.  No kernel is launched here."""
import ctypes as C
import os
import re

import pytest

from paper_2605_20022_amd import flexdraft as fd

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "flexdraft.h")).read()
    return re.findall(r"FD_API\s+[\w\s\*]+?\b(fd_\w+)\s*\(", text)


def test_header_symbols_are_exported():
    lib = fd.load()
    names = _declared_symbols()
    assert len(names) >= 10 and set(names) == set(fd.EXPORTS)
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in flexdraft.h but not exported"
    assert fd.fd_version().startswith("flexdraft-gfx950")


def test_struct_layout_matches_header():
    """The ctypes mirror must have the size the C compiler gives the struct (checked via a
    tiny C program compiled on the spot with the host compiler)."""
    import subprocess, tempfile
    src = '#include <stdio.h>\n#include "flexdraft.h"\nint main(){printf("%zu %zu %zu\\n", sizeof(fd_attn_args), ' \
          '__builtin_offsetof(fd_attn_args, k_cache), __builtin_offsetof(fd_attn_args, status));return 0;}\n'
    with tempfile.TemporaryDirectory() as d:
        open(os.path.join(d, "t.c"), "w").write(src)
        subprocess.check_call(["gcc", "-I", os.path.join(ROOT, "include"), os.path.join(d, "t.c"), "-o", os.path.join(d, "t")])
        size, off_k, off_s = map(int, subprocess.check_output([os.path.join(d, "t")]).split())
    assert size == C.sizeof(fd.fd_attn_args)
    assert off_k == fd.fd_attn_args.k_cache.offset and off_s == fd.fd_attn_args.status.offset


def _args(**kw):
    a = fd.fd_attn_args()
    a.batch = 4; a.num_q_heads = 32; a.num_kv_heads = 8; a.head_dim = 128; a.page_size = 16
    a.dtype = fd.FD_BF16; a.total_rows = 128; a.max_kv_len = 32768; a.max_new_rows = 32; a.num_pages = 9000
    for k, v in kw.items():
        setattr(a, k, v)
    return a


def test_attention_workspace_query_and_validation():
    a = _args()
    need = fd.fd_verify_draft_attn_workspace(a)
    # MFMA path: two split-partial slots of 128 rows x (D + 2) floats per persistent work-group,
    # independent of the sequence lengths, plus two small per-item index arrays
    per_slot = 128 * (128 + 2) * 4
    assert need % 256 == 0 and need >= 2 * 256 * per_slot and need <= 2 * 2048 * per_slot + (1 << 20)
    assert fd.fd_verify_draft_attn_workspace(_args(max_kv_len=1 << 20)) == need
    # scalar path: chunks * rows * heads * (D + 2) floats; an explicit chunk size fixes the count
    g = _args(flags=fd.FD_ATTN_FORCE_GENERIC, kv_chunk=4096)
    assert fd.fd_verify_draft_attn_workspace(g) == 8 * 128 * 32 * (128 + 2) * 4
    assert fd.fd_verify_draft_attn_workspace(_args(num_kv_heads=5)) == 0
    assert fd.fd_verify_draft_attn_workspace(_args(head_dim=100)) == 0
    assert fd.fd_verify_draft_attn_workspace(_args(kv_chunk=100)) == 0
    for bad, code in ((dict(num_kv_heads=5), 1), (dict(head_dim=256), 2), (dict(page_size=0), 1), (dict(dtype=7), 1)):
        with pytest.raises(fd.FlexDraftError) as e:
            fd._check(fd.load().fd_verify_draft_attn(C.byref(_args(**bad)), None))
        assert e.value.code == code
    # missing pointers are rejected before anything is launched
    with pytest.raises(fd.FlexDraftError) as e:
        fd._check(fd.load().fd_verify_draft_attn(C.byref(_args()), None))
    assert e.value.code == 1 and "NULL" in str(e.value)


def test_most_rows_of_one_launch():
    """max_new_rows x heads is bounded: 65535 groups of sixteen (fp32 kernel), 64 or 128 tile rows."""
    f32 = dict(dtype=fd.FD_F32, num_q_heads=8, num_kv_heads=8, total_rows=1, max_kv_len=64)
    assert fd.fd_verify_draft_attn_workspace(_args(max_new_rows=131056, **f32)) > 0                # 8 x 8191
    assert fd.fd_verify_draft_attn_workspace(_args(max_new_rows=131057, **f32)) == 0               # 8 x 8192
    with pytest.raises(fd.FlexDraftError) as e:
        fd._check(fd.load().fd_verify_draft_attn(C.byref(_args(max_new_rows=131057, **f32)), None))
    assert e.value.code == 2
    bf16 = dict(batch=1, num_q_heads=8, num_kv_heads=8, total_rows=1, max_kv_len=64)
    assert fd.fd_verify_draft_attn_workspace(_args(max_new_rows=8191 * 128, **bf16)) > 0
    assert fd.fd_verify_draft_attn_workspace(_args(max_new_rows=8191 * 128 + 1, **bf16)) == 0


def test_plan_entry_point_validates_on_the_host():
    """fd_verify_draft_plan takes the same argument struct; a planned attention call needs the length of
    the page list (the plan's page ids are checked against it)."""
    lib = fd.load()
    assert lib.fd_verify_draft_plan(None, None) == 1
    assert lib.fd_verify_draft_plan(C.byref(_args(num_kv_heads=5)), None) == 1
    assert lib.fd_verify_draft_plan(C.byref(_args()), None) == 1 and b"NULL" in lib.fd_last_error()
    assert lib.fd_verify_draft_plan(C.byref(_args(batch=0)), None) == 0            # nothing to plan
    a = _args(flags=fd.FD_ATTN_PLANNED, page_indices_len=0)
    p = 4096                                                                       # never dereferenced: rejected on the host
    for name in ("page_indptr", "page_indices", "kv_len", "row_indptr", "verify_len", "q", "k_new", "v_new", "out",
                 "k_cache", "v_cache", "workspace"):
        setattr(a, name, p)
    a.workspace_bytes = 1 << 30
    a.cache_stride_page, a.cache_stride_head, a.cache_stride_token = 8 * 16 * 128, 16 * 128, 128
    assert lib.fd_verify_draft_attn(C.byref(a), None) == 1 and b"page_indices_len" in lib.fd_last_error()


def test_negative_page_list_length_is_rejected():
    assert fd.fd_verify_draft_attn_workspace(_args(page_indices_len=-1)) == 0
    assert fd.fd_verify_draft_attn_workspace(_args(page_indices_len=0)) > 0


def test_accept_workspace_query_and_validation():
    g = fd.fd_accept_workspace(16, 128, 151936, False)
    s = fd.fd_accept_workspace(4, 64, 151936, True)
    assert g > 0 and s > g and g % 256 == 0 and s % 256 == 0
    assert fd.fd_accept_workspace(1, 1, 0, False) == 0
    lib = fd.load()
    rc = lib.fd_accept_greedy(None, fd.FD_BF16, 10, 20, None, None, 1, 1, 1, None, None, None, None, 0, None)
    assert rc == 1 and b"row_stride" in lib.fd_last_error()
    rc = lib.fd_accept_sample(None, None, fd.FD_BF16, 20, 20, 1.0, None, None, None, None, 0, 0, 0, None, None, None, 0, None)
    assert rc == 0      # empty batch: nothing to do


def test_widened_entry_points_validate_on_the_host():
    """fd_draft_select, fd_select_branch, fd_append_kv: workspace query and the argument errors that
    are detected before anything is launched."""
    lib = fd.load()
    ws = fd.fd_draft_select_workspace(480, 151936)
    assert ws > 0 and ws % 256 == 0 and fd.fd_draft_select_workspace(1, 0) == 0
    f = lib.fd_draft_select
    # temperature must be positive; the threshold finite; the row stride at least the vocabulary
    assert f(None, fd.FD_BF16, 100, 100, 0.0, 0.3, None, 1, 1, 1, None, None, None, None, 0, None) == 1
    assert b"temperature" in lib.fd_last_error()
    assert f(None, fd.FD_BF16, 100, 100, 1.0, float("nan"), None, 1, 1, 1, None, None, None, None, 0, None) == 1
    assert f(None, fd.FD_BF16, 50, 100, 1.0, 0.3, None, 1, 1, 1, None, None, None, None, 0, None) == 1
    assert b"row_stride" in lib.fd_last_error()
    assert f(None, fd.FD_BF16, 100, 100, 1.0, 0.3, None, 0, 0, 0, None, None, None, None, 0, None) == 0   # empty batch
    assert f(None, fd.FD_BF16, 100, 100, 1.0, 0.3, None, 1, 1, 1, None, None, None, None, 0, None) == 1   # NULL pointers
    # branch selection
    assert lib.fd_select_branch(None, None, None, None, None, None, -1, 0, 0, None, None, None) == 1
    assert lib.fd_select_branch(None, None, None, None, None, None, 0, 0, 0, None, None, None) == 0
    assert lib.fd_select_branch(None, None, None, None, None, None, 2, 4, 2, None, None, None) == 1
    p = C.c_void_p(4096)                                  # never dereferenced: the call fails on the host
    assert lib.fd_select_branch(p, p, p, p, None, None, 2, 4, 2, p, None, None) == 1 and b"verify_len" in lib.fd_last_error()
    # commit of accepted rows
    assert lib.fd_append_kv(None, None, None, None, None, None) == 1
    a = fd.fd_attn_args()
    a.dtype = fd.FD_BF16; a.batch = 0; a.num_kv_heads = 8; a.head_dim = 128; a.page_size = 16
    assert lib.fd_append_kv(C.byref(a), None, None, None, None, None) == 0       # empty batch
    a.batch = 2
    assert lib.fd_append_kv(C.byref(a), None, None, None, None, None) == 1 and b"NULL" in lib.fd_last_error()
    a.head_dim = 100
    assert lib.fd_append_kv(C.byref(a), None, None, None, None, None) == 1


def test_header_declares_only_the_methods_calls():
    """Measurement helpers live in a library of their own, not in the product's header or exports."""
    names = _declared_symbols()
    assert not [n for n in names if "probe" in n or "profile" in n or "stream_" in n]
    lib = fd.load()
    for n in ("fd_stream_copy", "fd_stream_read", "fd_profile_begin", "fd_profile_end"):
        assert not hasattr(lib, n)


def test_measurement_probes_validate_on_the_host():
    """The benchmark's probe library rejects NULL pointers and sizes that are not whole units."""
    from paper_2605_20022_amd import probes
    lib = probes.load()
    assert lib.fdp_stream_copy(None, None, 16, None) == 1
    assert lib.fdp_stream_read(None, 32768, None, None) == 1
    assert lib.fdp_stream_read(C.c_void_p(4096), 1000, C.c_void_p(4096), None) == 1
