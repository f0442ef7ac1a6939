"""Host logic without a GPU: the tables of workgroups behind the grouped launches.

Whatever the shapes, every element of every matrix must belong to exactly one workgroup of a
launch (per rank slice for compression), the workgroups that share the columns of a row block
must agree on where their partial products and their arrival counter live, and no two groups
may share either.  The tables come from the library's own builders through a host-only hook.
"""
import numpy as np
import pytest
from hypothesis import given, settings, strategies as st

from paper_2402_03293_amd import flora, workloads

COLS = dict(mat=0, row0=1, rows=2, col0=3, slice=4, rblock=5, col1=6, part=7, nparts=8, cidx=9, poff=10)
RANKS = [8, 16, 32, 64, 128, 256]

shape_lists = st.lists(st.tuples(st.integers(1, 5000), st.integers(1, 9000)), min_size=1, max_size=5)
aligned_shape_lists = st.lists(st.tuples(st.integers(1, 5000), st.integers(1, 1100).map(lambda x: 8 * x)),
                               min_size=1, max_size=5)


def check_compress(shapes, r, gdt):
    items, info = flora.debug_work_items(0, shapes, r, gdt)
    mt, _, kc, ws_floats, ws_counters = (int(x) for x in info)
    c = COLS
    if r <= 32:
        rows_per_wg, slice_w, nslices, rp = 64 * mt, None, 1, max(16, r)
    else:
        wide = mt >= 8
        rows_per_wg = 512 if mt == 8 else 256 if mt == 16 else 128 if mt == 32 else 128 * mt
        slice_w = (64 if r == 64 else 128) if wide else 64
        nslices, rp = r // slice_w, slice_w
    groups = {}
    for i, it in enumerate(items):
        groups.setdefault((it[c["mat"]], it[c["rblock"]], it[c["slice"]] if r > 32 else 0), []).append(it)
    # rows: per (matrix, slice) the row blocks tile [0, n)
    for l, (n, m) in enumerate(shapes):
        for s in range(nslices):
            blocks = sorted({(g[0][c["row0"]], g[0][c["rows"]]) for k, g in groups.items() if k[0] == l and k[2] == s})
            assert blocks, (l, s)
            pos = 0
            for row0, rows in blocks:
                assert row0 == pos and 1 <= rows <= rows_per_wg
                pos += rows
            assert pos == n
    seen_counters, spans = set(), []
    for key, g in groups.items():
        n, m = shapes[key[0]]
        g = sorted(g, key=lambda it: it[c["part"]])
        nparts = g[0][c["nparts"]]
        assert [it[c["part"]] for it in g] == list(range(nparts)) and nparts >= 1
        pos = 0
        for it in g:
            assert it[c["nparts"]] == nparts and it[c["row0"]] == g[0][c["row0"]] and it[c["rows"]] == g[0][c["rows"]]
            assert it[c["col0"]] == pos and it[c["col0"]] % 64 == 0 and it[c["col1"]] > it[c["col0"]]
            pos = it[c["col1"]]
        assert pos == m
        if nparts > 1:
            assert len({it[c["cidx"]] for it in g}) == 1 and len({it[c["poff"]] for it in g}) == 1
            cidx, poff = g[0][c["cidx"]], g[0][c["poff"]]
            assert 0 <= cidx < ws_counters and cidx not in seen_counters
            seen_counters.add(cidx)
            spans.append((poff, poff + nparts * rows_per_wg * rp))
    spans.sort()
    for (a0, a1), (b0, b1) in zip(spans, spans[1:]):
        assert a1 <= b0
    if spans:
        assert spans[0][0] >= 0 and spans[-1][1] <= ws_floats
    assert len(seen_counters) == ws_counters
    return items, info


def check_decompress(shapes, r, dtype=flora.F32, kind=1):
    items, info = flora.debug_work_items(kind, shapes, r, dtype)
    vec = int(info[1])
    cols = 256 if vec else 128
    c = COLS
    if vec:
        assert r >= 64 and all(m % 4 == 0 for _, m in shapes)
    per_mat = {}
    for it in items:
        per_mat.setdefault(it[c["mat"]], []).append(it)
    assert sorted(per_mat) == list(range(len(shapes)))
    for l, (n, m) in enumerate(shapes):
        its = per_mat[l]
        nchunks = (m + cols - 1) // cols
        blocks = sorted({(it[c["rblock"]], it[c["row0"]], it[c["rows"]]) for it in its})
        pos = 0
        for rb, (rblock, row0, rows) in enumerate(blocks):
            assert rblock == rb and row0 == pos and rows >= 1
            if rb + 1 < len(blocks):
                assert rows % 32 == 0
            pos += rows
        assert pos == n
        assert len(its) == len(blocks) * nchunks
        assert sorted(it[c["part"]] for it in its) == list(range(len(its)))       # slots of per-workgroup sums
        for it in its:
            cc = it[c["slice"]]
            assert 0 <= cc < nchunks and it[c["col0"]] == cc * cols
            assert it[c["part"]] == it[c["rblock"]] * nchunks + cc
    return items, info


@settings(max_examples=60, deadline=None)
@given(shape_lists, st.sampled_from([8, 16, 32]), st.sampled_from([flora.F32, flora.BF16]))
def test_fp32_compress_tables_cover_every_element_once(shapes, r, gdt):
    check_compress(shapes, r, gdt)


# 128 rows per workgroup (bf16 at r = 32): the last block short or a single row, pieces and whole rows.
@pytest.mark.parametrize("shapes,kc", [([(257, 2048)] * 80, 512), ([(320, 4096)] * 40, 512), ([(65537, 80)] * 8, 0), ([(1281, 1024)] * 30, 1024), (workloads.workload(2).shapes, 1024),
                                       (workloads.workload(5).shapes, 0)])
def test_bf16_compress_tables_of_128_rows(shapes, kc):
    _, info = check_compress(shapes, 32, flora.BF16)
    assert (int(info[0]), int(info[2])) == (2, kc)


@settings(max_examples=60, deadline=None)
@given(st.one_of(shape_lists, aligned_shape_lists), st.sampled_from([64, 128, 256]))
def test_bf16_compress_tables_cover_every_element_once(shapes, r):
    check_compress(shapes, r, flora.BF16)


# Pieces of columns between the halvings of 1536 (bf16 and fp32 gradients, whole and ragged rows).
@pytest.mark.parametrize("shapes,r", [([(768, 2304), (768, 768), (768, 3072), (3072, 768)] * 4, 128), ([(300, 8192)] * 8, 64), ([(640, 12001)], 256),
                                      ([(129, 5003)] * 12, 128), ([(8192, 8192)], 256), ([(1000, 1500)] * 10, 256)])
def test_bf16_compress_tables_of_finer_pieces(shapes, r):
    check_compress(shapes, r, flora.BF16)
    check_compress(shapes, r, flora.F32)


# ... are tried with every number of rows, whatever was the last to be tried with another (us with what was chosen else: 147 / 110,
# 271 / 195, 123 / 82), and at r = 256 fewer rows of fp32 gradients only where they are ahead by a margin (55 / 41).
@pytest.mark.parametrize("shapes,r,mt,shared", [([(1664, 1600)] * 47 + [(64, 6976)] * 26, 64, 32, True), ([(980, 67)] * 3 + [(5305, 2145)] * 12 + [(2186, 7856)] * 2, 64, 32, True),
                                                ([(64, 1792)] * 115 + [(64, 4672)] * 75, 128, 32, True), ([(4488, 5584)], 256, 16, True)])
def test_finer_pieces_with_every_number_of_rows(shapes, r, mt, shared):
    _, info = check_compress(shapes, r, flora.F32)
    assert int(info[0]) == mt and (int(info[3]) > 0) == shared


@settings(max_examples=60, deadline=None)
@given(st.one_of(shape_lists, aligned_shape_lists), st.sampled_from(RANKS))
def test_decompress_tables_cover_every_element_once(shapes, r):
    check_decompress(shapes, r)


# Rows chosen by the rounds of a launch: sets at and beside 256 workgroups, single rows, the longest and shortest blocks.
@pytest.mark.parametrize("shapes,r", [([(777, 2008)] * 9, 128), ([(768, 2304), (768, 768), (768, 3072), (3072, 768)] * 4, 256),
                                      ([(1, 8)], 256), ([(1024, 256)] * 256, 256), ([(1025, 256)] * 257, 256), ([(32, 64), (16384, 1024)], 256),
                                      ([(33, 252)] * 3, 256), ([(100, 256)] * 300, 128), ([(2304, 1024)] * 40, 64)])
def test_decompress_tables_by_rounds(shapes, r):
    check_decompress(shapes, r)


def test_bf16_rows_at_rank_64_take_128_rows_in_large_launches():
    """bf16 outputs and weights alike; fp32 ones 64."""
    gpt, xl = (workloads.workload(i).shapes for i in (3, 5))
    for shapes in (gpt, gpt * 2, xl[:48], xl, [(1100, 1003)] * 100, [(2304, 1024)] * 40):
        for kind in (1, 5):
            for dtype, rows in ((flora.F32, 64), (flora.BF16, 128)):
                items, _ = check_decompress(shapes, 64, dtype, kind)
                assert max(it[COLS["rows"]] for it in items) == rows, (shapes[0], len(shapes), kind, dtype)


@settings(max_examples=30, deadline=None)
@given(shape_lists, st.sampled_from(RANKS))
def test_transfer_row_blocks(shapes, r):
    items, _ = flora.debug_work_items(2, shapes, r)
    for l, (n, m) in enumerate(shapes):
        its = sorted((it[1], it[2]) for it in items if it[0] == l)
        pos = 0
        for row0, rows in its:
            assert row0 == pos and 1 <= rows <= (64 if r >= 64 else 32)
            pos += rows
        assert pos == n
    # T = A^T A' at ranks 64 and above: every slab of rows of T sees every column exactly once
    titems, _ = flora.debug_work_items(3, shapes, r)
    if r < 64:
        assert len(titems) == 0
        return
    slabs = r // min(r, 128)
    for l, (n, m) in enumerate(shapes):
        for s_ in range(slabs):
            its = sorted((it[7], it[3], it[6]) for it in titems if it[0] == l and it[4] == s_)
            pos = 0
            for c, (part, col0, col1) in enumerate(its):
                assert part == c and col0 == pos and col0 < col1 <= col0 + 1024
                pos = col1
            assert pos == m


@pytest.mark.parametrize("index", [1, 2, 3, 4, 5])
def test_tables_of_the_five_workloads(index):
    wl = workloads.workload(index)
    gdt = flora.F32 if wl.grad_dtype == "f32" else flora.BF16
    items, info = check_compress(wl.shapes, wl.r, gdt)
    ditems, dinfo = check_decompress(wl.shapes, wl.r)
    if wl.r >= 64:
        assert int(info[0]) >= 8 and int(dinfo[1]) == 1          # wide compress, 16-byte decompress
    # launches of the full-size workloads fill the chip: more workgroups than compute units
    if index >= 2:
        assert len(items) >= 256 and len(ditems) >= 256


def test_row_blocks_of_a_bundle_share_an_xcd():
    # workgroup ids go round-robin over 8 XCDs: the column chunks of one row block of the state
    # (decompress) are placed 8 apart so that they meet in one L2
    shapes = [(2048, 2048)] * 4
    items, _ = flora.debug_work_items(1, shapes, 256)
    where = {}
    for i, it in enumerate(items):
        where.setdefault((it[0], it[5]), set()).add(i % 8)
    assert all(len(v) == 1 for v in where.values())


def test_hook_rejects_bad_arguments():
    L = flora.lib()
    mats = flora.matrices([(4, 4)])
    assert L.flora_debug_work_items(0, mats, 1, 12, 0, None, 0, None) == flora.ERR_UNSUPPORTED
    assert L.flora_debug_work_items(7, mats, 1, 16, 0, None, 0, None) == flora.ERR_INVALID
    assert L.flora_debug_work_items(0, flora.matrices([(0, 4)]), 1, 16, 0, None, 0, None) == flora.ERR_INVALID
    assert L.flora_debug_work_items(0, mats, 1, 16, 0, None, 0, None) == 1


def test_filled_updates_at_small_ranks_take_128_rows():
    """The rows per workgroup that launches filling the chip were measured to be fastest with, at every such size."""
    t5s, gpt = (workloads.workload(i).shapes for i in (2, 3))
    for shapes in (t5s, gpt, [(768, 3072)] * 24, [(1024, 2048)] * 36, [(2048, 2048)] * 8):
        for r in (8, 16, 32):
            items, _ = check_decompress(shapes, r)
            assert max(it[COLS["rows"]] for it in items) == 128, (shapes[0], len(shapes), r)


def test_fp32_compress_pieces_by_how_much_they_would_cut():
    """Pieces of 1024 columns only where they were measured to be no slower than 512: large sets, and sets of matrices
    that they mostly do not cut."""
    t5s, gpt = (workloads.workload(i).shapes for i in (2, 3))
    for shapes, kc in ((t5s, 1024), ([(768, 768)] * 96, 1024), ([(1600, 6400)] * 12, 1024), ([(2340, 3032)] * 9, 512),
                       ([(1600, 6400)] * 8, 512), ([(4096, 4096)] * 6, 512), (gpt, 512), ([(1024, 1024)], 256), ([(64, 48)], 256)):
        for r in (8, 16, 32):
            _, info = check_compress(shapes, r, flora.BF16)
            assert int(info[2]) == kc, (shapes[0], len(shapes), r)


def test_bf16_updates_are_streamed_by_the_kernel_of_whole_lines_only():
    """bf16 weights: the hint where a wave moves whole 128-byte lines, which ranks <= 32 and the 4-byte-per-lane
    kernel never do, and from 256 MiB on."""
    xl = workloads.workload(5).shapes
    sgd = flora.sgd_update(1e-3)
    for r in RANKS:
        whole = r >= 64
        assert flora.debug_access_policy(flora.matrices(xl), r, flora.BF16, sgd) == ((3, 3, 0, 1) if whole else (0, 0, 0, 0))
        assert flora.debug_access_policy(flora.matrices(xl[:8]), r, flora.BF16, sgd) == (0, 0, 0, 0)
        assert flora.debug_access_policy(flora.matrices([(n, m + 8) for n, m in xl]), r, flora.BF16, sgd) == (0, 0, 0, int(whole))
        try:
            flora.set_tuning("decompress_vec", 1)          # 4 bytes per lane
            assert flora.debug_access_policy(flora.matrices(xl), r, flora.BF16, sgd) == (0, 0, 0, 0)
        finally:
            flora.set_tuning("decompress_vec", 0)


def test_unfactored_policy_by_what_w_and_v_take():
    """The unfactored rule's plan for the last-level cache: from 192 MiB of W and V on, with bf16 weights from 256 MiB,
    to 768 MiB of V; V stays in the cache as a whole up to 256 MiB."""
    u = flora.unfactored_update(1e-3, 1.0, 0.9, 1e-30, 1.0)
    for count, f32, bf16 in ((24, (0, 0, 0, 0), (0, 0, 0, 0)),           # 192 and 144 MiB
                             (25, (0, 3, 1, 0), (0, 0, 0, 0)),           # 200, 150
                             (42, (0, 3, 1, 0), (0, 0, 0, 0)),           # 336, 252
                             (43, (0, 3, 1, 0), (0, 3, 1, 0)),           # 344, 258
                             (65, (2, 3, 1, 0), (2, 3, 1, 0)),           # V of 260 MiB
                             (192, (2, 3, 1, 0), (2, 3, 1, 0))):         # V of 768 MiB
        mats = flora.matrices([(1024, 1024)] * count)
        for r in RANKS:
            assert flora.debug_access_policy(mats, r, flora.F32, u) == f32, (count, r)
            assert flora.debug_access_policy(mats, r, flora.BF16, u) == bf16, (count, r)
