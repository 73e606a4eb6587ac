"""Calls of the C ABI that pass validation, for the sanitizer build only
(its launches are stand-ins that check the host layer's launch arguments;
with the real library these calls would launch kernels). Run by
tests/test_sanitize_cpu.py in a process with AddressSanitizer preloaded."""
import ctypes

import pytest

from paper_2607_03612_amd import binding as B

OK = ctypes.c_void_p(0x10000)  # never dereferenced by the stand-ins


def _p(heads, frames, T, dtype=B.BF16):
    return B.Problem(heads, frames, T, 64, 64, dtype)


TABLES = [
    # every class on a small ragged layer
    (12, 3, 261, [(B.DENSE, 0), (B.FRAME_LOCAL, 0), (B.TOPK, 5), (B.ANCHOR, 0), (B.ANCHOR, 2),
                  (B.STRIDE, 1), (B.STRIDE, 7), (B.STRIDE, 783), (B.GLOBAL_PROBE, 3),
                  (B.COSINE_TOPK, 1), (B.COSINE_TOPK, 2), (B.SKIP, 0)]),
    # the split: a 274800-token layer with long lists and a dense head
    (6, 200, 1374, [(B.TOPK, 959), (B.GLOBAL_PROBE, 400), (B.COSINE_TOPK, 3), (B.DENSE, 0),
                    (B.FRAME_LOCAL, 0), (B.STRIDE, 9)]),
    # the largest problem: 2^20 tokens, the most blocks
    (3, 8, 131072, [(B.TOPK, 164), (B.FRAME_LOCAL, 0), (B.TOPK, 16384)]),
    # the most heads, cycling through the classes
    (256, 2, 300, [[(B.DENSE, 0), (B.FRAME_LOCAL, 0), (B.TOPK, 3), (B.ANCHOR, 1), (B.STRIDE, 5),
                    (B.GLOBAL_PROBE, 2), (B.COSINE_TOPK, 1), (B.SKIP, 0)][h % 8] for h in range(256)]),
]


@pytest.mark.parametrize("heads,frames,T,table", TABLES)
@pytest.mark.parametrize("dtype", [B.BF16, B.F32])
def test_valid_calls_reach_consistent_launches(heads, frames, T, table, dtype):
    lib = B.load()
    p = _p(heads, frames, T, dtype)
    t = B.head_table(table)
    cap = lib.saf3r_index_capacity(ctypes.byref(p), t)
    assert cap >= 1
    assert lib.saf3r_estimate_blocks(ctypes.byref(p), t, OK, OK, OK, OK, None) == 0
    sel = lib.saf3r_select_blocks
    ws = lib.saf3r_select_workspace_bytes(ctypes.byref(p), t)
    # single-launch path (when its score rows fit in LDS), full and one-head workspaces
    nb = lib.saf3r_num_blocks(ctypes.byref(p))
    if nb <= 8192:
        assert sel(ctypes.byref(p), t, OK, OK, OK, OK, cap, None, None, 0, None) == 0
    assert sel(ctypes.byref(p), t, OK, OK, OK, OK, cap, OK, OK, max(ws, 16), None) == 0
    n_topk = sum(1 for c, _ in table if c == B.TOPK)
    if n_topk > 1:
        assert sel(ctypes.byref(p), t, OK, OK, OK, OK, cap, None, OK, ws // n_topk, None) == 0
    att = lib.saf3r_sparse_attention
    aws = lib.saf3r_attention_workspace_bytes(ctypes.byref(p), t)
    assert att(ctypes.byref(p), t, OK, OK, OK, OK, OK, cap, OK, OK, None, 0, None) == 0
    assert att(ctypes.byref(p), t, OK, OK, OK, OK, OK, cap, OK, None, OK, max(aws, 16), None) == 0
    if any(c == B.COSINE_TOPK for c, _ in table):
        cws = lib.saf3r_cosine_workspace_bytes(ctypes.byref(p), 96)
        assert lib.saf3r_cosine_select(ctypes.byref(p), t, OK, 96, OK, cws, OK, OK, cap, None) == 0
    nws = lib.saf3r_nmse_workspace_bytes(ctypes.byref(p))
    assert lib.saf3r_nmse(ctypes.byref(p), OK, OK, OK, nws, OK, None) == 0
    assert lib.saf3r_nmse_noalloc(ctypes.byref(p), OK, OK, OK, None) == 0


# four rows to a workgroup, in one launch, up to 256 blocks and 512 workgroups
@pytest.mark.parametrize("heads,nb,small", [(1, 17, True), (30, 65, True), (31, 65, False), (16, 128, True),
                                            (17, 128, False), (8, 256, True), (9, 256, False), (16, 256, False),
                                            (1, 257, False)])
def test_small_layers_select_in_one_launch(heads, nb, small):
    lib = B.load()
    p = _p(heads, 1, 64 * nb)
    t = B.head_table([(B.TOPK, 3)] * heads)
    ws = lib.saf3r_select_workspace_bytes(ctypes.byref(p), t)
    rows = lib.saf3r_stub_topk_rows_per_group
    for workspace, expect in ((None, 4 if small else 16), (OK, 4 if small else 0)):
        assert lib.saf3r_select_blocks(ctypes.byref(p), t, OK, OK, OK, OK, 3, None, workspace,
                                       ws if workspace else 0, None) == 0
        assert rows() == expect


# rows that four waves share in bf16: beside short lists, in key ranges (with the workspace), strided, odd block counts
@pytest.mark.parametrize("heads,frames,T,table", [
    (4, 1, 520, [(B.DENSE, 0), (B.TOPK, 8), (B.TOPK, 1), (B.STRIDE, 1)]),
    (5, 2, 1000, [(B.DENSE, 0), (B.TOPK, 31), (B.FRAME_LOCAL, 0), (B.ANCHOR, 1), (B.TOPK, 3)]),
    (1, 1, 8190, [(B.DENSE, 0)]),
    (16, 8, 1374, [(B.FRAME_LOCAL, 0)] * 6 + [(B.DENSE, 0)] + [(B.TOPK, 13)] * 9),
    (3, 4, 1374, [(B.STRIDE, 3), (B.STRIDE, 500), (B.STRIDE, 11)]),
    (12, 20, 1001, [(B.DENSE, 0)] * 3 + [(B.FRAME_LOCAL, 0)] * 4 + [(B.TOPK, 32)] * 5),
])
@pytest.mark.parametrize("workspace", [False, True])
def test_shared_rows_reach_consistent_launches(heads, frames, T, table, workspace):
    lib = B.load()
    p = _p(heads, frames, T)
    t = B.head_table(table)
    cap = max(lib.saf3r_index_capacity(ctypes.byref(p), t), 1)
    aws = lib.saf3r_attention_workspace_bytes(ctypes.byref(p), t)
    launches = lib.saf3r_stub_attention_launches
    before = launches(4)
    assert lib.saf3r_sparse_attention(ctypes.byref(p), t, OK, OK, OK, OK, OK, cap, OK, OK,
                                      OK if workspace else None, max(aws, 16) if workspace else 0, None) == 0
    assert launches(4) > before


# a global-probe head's one workgroup writes nb * cap entries: beside the Top-K launch up to 2^17 of them for each turn of
# 256 groups of 16 Top-K rows, twice that in one launch
@pytest.mark.parametrize("topk,nb,cap,with_ws,without", [
    (1, 512, 256, 1, 1), (1, 512, 257, 0, 1), (1, 512, 512, 0, 1), (1, 1024, 128, 1, 1), (1, 1024, 256, 0, 1),
    (1, 1024, 257, 0, 0), (1, 1025, 4, 0, 0), (1, 256, 512, 1, 1), (4, 1024, 129, 0, 1), (5, 1024, 256, 1, 1),
    (5, 1024, 257, 0, 1), (10, 1024, 384, 1, 1), (10, 1024, 768, 0, 1), (10, 1024, 769, 0, 0)])
def test_global_probe_lists_beside_the_topk_launch(topk, nb, cap, with_ws, without):
    lib = B.load()
    t = B.head_table([(B.TOPK, 3)] * topk + [(B.GLOBAL_PROBE, 4)])
    p = _p(topk + 1, 1, 64 * nb)
    ws = lib.saf3r_select_workspace_bytes(ctypes.byref(p), t)
    for workspace, fused in ((OK, with_ws), (None, without)):
        assert lib.saf3r_select_blocks(ctypes.byref(p), t, OK, OK, OK, OK, cap, None, workspace,
                                       ws if workspace else 0, None) == 0
        assert lib.saf3r_stub_topk_global() == fused, workspace


# equal rows: shared while that takes fewer turns of the chip (one workgroup per CU), not beyond
@pytest.mark.parametrize("heads,nb,k,waves", [
    (1, 130, 8, 4), (1, 653, 8, 1), (8, 86, 8, 1), (1, 512, 16, 4), (1, 520, 16, 1), (1, 800, 16, 1), (1, 653, 48, 4),
    (4, 203, 12, 1), (8, 640, 128, 1), (1, 130, 7, 1),
])
def test_equal_rows_are_shared_where_that_takes_fewer_turns(heads, nb, k, waves):
    lib = B.load()
    p = _p(heads, 1, 64 * nb)
    t = B.head_table([(B.TOPK, k)] * heads)
    launches = lib.saf3r_stub_attention_launches
    before = [launches(1), launches(4)]
    assert lib.saf3r_sparse_attention(ctypes.byref(p), t, OK, OK, OK, OK, OK, k, OK, None, None, 0, None) == 0
    assert [launches(1) - before[0], launches(4) - before[1]] == [int(waves == 1), int(waves == 4)]


def test_all_dense_table_is_one_launch():
    lib = B.load()
    p = _p(16, 100, 1374)
    t = B.head_table([(B.DENSE, 0)] * 16)
    assert lib.saf3r_sparse_attention(ctypes.byref(p), t, OK, OK, OK, None, None, 0, OK, None,
                                      None, 0, None) == 0


@pytest.mark.parametrize("heads,frames,T,table", TABLES)
def test_list_check_reaches_a_consistent_launch(heads, frames, T, table):
    lib = B.load()
    p = _p(heads, frames, T)
    t = B.head_table(table)
    cap = lib.saf3r_index_capacity(ctypes.byref(p), t)
    first = ctypes.c_int32(-1)
    assert lib.saf3r_validate_index(ctypes.byref(p), t, OK, OK, cap, OK, ctypes.byref(first), None) == 0
