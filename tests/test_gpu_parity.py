"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs.  Layout arrays must be bit-equal; y must satisfy
|y - y_ref| <= 1e-5 * sum_j |a_ij x_j| per row (the tolerance the benchmark spec states)."""
import os

import numpy as np
import pytest

from workloads import make_config, random_csr, worked_example_8x8

pytestmark = pytest.mark.gpu

TOL = 1e-5
# fp64 handles: the same multiple (168) of the unit roundoff as 1e-5 is of fp32's; the reference
# is accumulated in extended precision and rounded once
TOL_F64 = 168 * 2.0**-53
LAYOUT_ARRAYS = ("blk_bm", "blk_bn", "slot_ptr", "blk_group_ptr", "col_blk_ptr", "stripe_ptr", "stripe_blk",
                 "group_ptr", "group_slot", "group_rounds", "col_group_ptr", "comp_lo", "comp_col", "fixed_start", "fixed_col",
                 "unit_ptr", "unit_stripe", "unit_k", "multi_stripes", "row_local", "seg_len", "slot_key", "blk_shift", "col_local",
                 "data", "add_sign")


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2504_08860_amd as H
    H.lib()
    return H


def to_dev(m):
    import torch
    t = lambda a: torch.from_numpy(a).cuda()
    return t(m.ptr), t(m.col), t(m.val), t(m.x)


def check_against_oracle(H, oracle, m, check_add_sign=True, **params):
    import torch
    ptr, col, val, x = to_dev(m)
    f64 = m.val.dtype == np.float64
    tol = TOL_F64 if f64 else TOL
    build, spmv = (H.hbp_build_f64, H.hbp_spmv_f64) if f64 else (H.hbp_build, H.hbp_spmv)
    print(f"[case] {m.name} rows={m.n_rows} cols={m.n_cols} nnz={m.nnz} {m.val.dtype} params={params}", flush=True)
    h = build(ptr, col, val, m.n_rows, m.n_cols, keep_keys=True, **params)   # the keys themselves are compared too
    try:
        info = H.hbp_get_info(h)
        shift = (-2 if params.get("no_reorder") else -3 if params.get("key_length") else -4 if params.get("block_shift")
                 else params.get("hash_shift", -1))
        o = oracle.OracleHbp(m.ptr, m.col, m.val, m.n_rows, m.n_cols, R=info.rows_per_block, C=info.cols_per_block,
                             W=info.group_width, hash_shift=shift,
                             num_workers=info.num_workers, fixed_q8=info.fixed_fraction_q8,
                             slot_weight=info.slot_weight, unit_slots=info.combine_unit_slots,
                             round_weight=info.round_weight, group_weight=info.group_weight, column_weight=info.column_weight,
                             paper_schedule=bool(params.get("paper_schedule")))
        assert info.first_ticket_block == o.first_ticket_block
        assert (info.nnz, info.blocks, info.slots, info.groups) == (o.nnz, o.B, o.S, o.G)
        assert info.hash_shift == o.a and info.value_bytes == m.val.dtype.itemsize
        assert (info.combine_units, info.split_row_blocks) == (o.U, o.NM)
        assert info.hash_b == max(1, info.rows_per_block // 9)
        for name in LAYOUT_ARRAYS:
            if name == "add_sign" and not check_add_sign:
                continue
            got, want = H.hbp_export(h, name), o.array(name)
            if name == "data":
                assert got.dtype == want.dtype == m.val.dtype
                bits = np.uint64 if f64 else np.uint32
                got, want = got.view(bits), want.view(bits)
            assert got.shape == want.shape, name
            assert np.array_equal(got, want), f"{name} differs at {np.flatnonzero(got != want)[:5]}"
        y_ref, s_abs = oracle.csr_spmv_f64(m.ptr, m.col, m.val, m.x)
        y = torch.full((m.n_rows,), float("nan"), device="cuda", dtype=x.dtype)
        for rep in range(2):  # the second call checks that the ticket counter was re-armed
            y.fill_(float("nan"))
            spmv(h, x, y)
            torch.cuda.synchronize()
            yh = y.cpu().numpy().astype(np.float64)
            bad = np.flatnonzero(~(np.abs(yh - y_ref) <= tol * s_abs))
            assert bad.size == 0, f"rep {rep}: rows {bad[:5]} y {yh[bad[:5]]} ref {y_ref[bad[:5]]}"
            assert np.all(yh[np.diff(m.ptr) == 0] == 0.0)
        # per-slot partial sums against the oracle's walk through the layout, each on the scale of its own
        # segment's absolute products
        _, p_ref, p_abs = o.spmv(m.x, with_abs=True)
        p = H.hbp_export(h, "partial").astype(np.float64)
        bad = np.flatnonzero(~(np.abs(p - p_ref) <= tol * p_abs))
        assert bad.size == 0, f"partial sums of slots {bad[:5]}: {p[bad[:5]]} against {p_ref[bad[:5]]}"
        o.close()
        return info
    finally:
        H.hbp_free(h)


def test_worked_example(H, oracle):
    check_against_oracle(H, oracle, worked_example_8x8(), rows_per_block=4, cols_per_block=4, group_width=2, hash_shift=0)


SMALL = [
    # rows, cols, density, seed, R, C, W, shift
    (40, 40, 0.2, 1, 8, 8, 4, -1),
    (77, 53, 0.3, 2, 16, 10, 4, 0),
    (64, 200, 0.15, 3, 64, 32, 8, 1),
    (129, 65, 0.5, 4, 32, 16, 3, 2),
    (30, 300, 0.4, 5, 7, 50, 64, -1),
    (200, 30, 0.1, 6, 512, 4096, 64, -1),
    (1000, 1000, 0.02, 7, 100, 333, 64, -1),     # ragged everywhere, several tiles of 64 nonzeros
    (5000, 3000, 0.01, 8, 512, 1024, 32, -1),
    (3000, 9000, 0.05, 9, 8192, 32768, 64, -1),  # the largest block the library accepts
    (2500, 700, 0.3, 10, 1, 1, 1, 0),            # degenerate 1 x 1 blocks
]


@pytest.mark.parametrize("case", SMALL)
def test_small_random(H, oracle, case):
    nr, nc, dens, seed, R, C, W, shift = case
    m = random_csr(nr, nc, dens, seed, empty_row_frac=0.15)
    check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C, group_width=W, hash_shift=shift)


@pytest.mark.parametrize("P,q8,chunk,gw,cw", [(1, 0, 1, 0, 0), (3, 256, 1, 50, 400), (7, 100, 5, 1024, 4096), (2000, 200, 2, 7, 0),
                                               (5, 30, 64, 0, 33)])
def test_schedule_variants(H, oracle, P, q8, chunk, gw, cw):
    """y does not depend on how blocks are split into fixed and competitive parts."""
    m = random_csr(3000, 3000, 0.01, 21, empty_row_frac=0.1)
    info = check_against_oracle(H, oracle, m, rows_per_block=64, cols_per_block=128, num_workers=P,
                                fixed_fraction_q8=q8, claim_chunk=chunk, round_weight=gw, group_weight=cw,
                                slot_weight=0 if cw == 33 else -1)
    assert info.num_workers == P and info.claim_chunk == chunk


@pytest.mark.parametrize("number,scale,R,C", [(1, 1.0, 512, 4096), (2, 0.02, 512, 4096), (2, 0.02, 256, 32768),
                                              (3, 2**-6, 256, 1024), (4, 2**-7, 512, 2048), (5, 0.01, 512, 4096),
                                              (5, 0.01, 2048, 32768)])
def test_configs_reduced(H, oracle, number, scale, R, C):
    check_against_oracle(H, oracle, make_config(number, scale), rows_per_block=R, cols_per_block=C)


def test_long_rows_and_heavy_tail(H, oracle):
    """A few rows far longer than the rest (one fills a whole block row), inside one group."""
    rng = np.random.default_rng(3)
    lens = np.r_[rng.integers(0, 6, 500), [4096, 3000, 1], rng.integers(0, 6, 300)]
    n_cols = 4096
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    ptr = np.r_[0, np.cumsum(lens)].astype(np.int32)
    from workloads import CsrMatrix
    m = CsrMatrix("heavy", len(lens), n_cols, ptr, col, rng.standard_normal(len(col)).astype(np.float32),
                  rng.uniform(-1, 1, n_cols).astype(np.float32))
    check_against_oracle(H, oracle, m, rows_per_block=256, cols_per_block=4096)
    check_against_oracle(H, oracle, m, rows_per_block=256, cols_per_block=512)


def test_empty_matrix_and_empty_rows(H, oracle):
    import torch
    ptr = torch.zeros(11, dtype=torch.int32, device="cuda")
    col = torch.zeros(1, dtype=torch.int32, device="cuda")
    val = torch.zeros(1, dtype=torch.float32, device="cuda")
    h = H.hbp_build(ptr, col, val, 10, 5)
    info = H.hbp_get_info(h)
    assert (info.nnz, info.blocks, info.slots, info.groups) == (0, 0, 0, 0)
    y = torch.full((10,), float("nan"), device="cuda")
    H.hbp_spmv(h, torch.ones(5, device="cuda"), y)
    assert torch.all(y == 0)
    H.hbp_free(h)
    # a single nonzero in the last row and column
    m = random_csr(1, 1, 1.1, 0)
    check_against_oracle(H, oracle, m)


def test_invalid_inputs_are_errors(H):
    import torch
    m = random_csr(50, 60, 0.2, 1)
    ptr, col, val, x = to_dev(m)
    with pytest.raises(H.HbpError) as e:                      # column beyond n_cols
        H.hbp_build(ptr, col, val, m.n_rows, 10)
    assert e.value.status == -3
    bad = col.clone(); bad[1], bad[0] = col[0].item(), col[1].item()
    if m.ptr[1] >= 2:                                          # unsorted inside row 0
        with pytest.raises(H.HbpError) as e:
            H.hbp_build(ptr, bad, val, m.n_rows, m.n_cols)
        assert e.value.status == -3
    p2 = ptr.clone(); p2[3] = p2[2] - 1 if p2[2] > 0 else 99999
    with pytest.raises(H.HbpError) as e:                      # decreasing row pointer
        H.hbp_build(p2, col, val, m.n_rows, m.n_cols)
    assert e.value.status == -2
    for kw in (dict(rows_per_block=8193), dict(cols_per_block=32769), dict(group_width=65), dict(hash_shift=13)):
        with pytest.raises(H.HbpError) as e:
            H.hbp_build(ptr, col, val, m.n_rows, m.n_cols, **kw)
        assert e.value.status == -1
    with pytest.raises(H.HbpError) as e:                      # block table too large
        H.hbp_build(ptr, col, val, m.n_rows, 2**30, rows_per_block=1, cols_per_block=1)
    assert e.value.status == -4


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("params", [dict(), dict(rows_per_block=512, rounds_per_batch=8)])
@pytest.mark.parametrize("first_row,n_rows", [(7, 5000), (4999, 1), (3000, 2000)])
def test_row_slices_without_rebased_pointers_are_errors(H, first_row, n_rows, params, f64):
    """The pointers of a row slice, not rebased, with the slice's own columns: ptr[0] = b, ptr[n] = b + nnz, nnz
    columns.  Refused, with the parameters chosen from the matrix (a sampling pass) or given."""
    m = random_csr(first_row + n_rows, 700, 0.05, 3)
    ptr, col, val, _ = to_dev(m)
    b, e = int(m.ptr[first_row]), int(m.ptr[-1])
    assert b > 0
    build = H.hbp_build_f64 if f64 else H.hbp_build
    with pytest.raises(H.HbpError) as err:
        build(ptr[first_row:].clone(), col[b:e].clone(), (val.double() if f64 else val)[b:e].clone(), n_rows, m.n_cols, **params)
    assert err.value.status == -2
    h = build((ptr[first_row:] - b).contiguous(), col[b:e].clone(), (val.double() if f64 else val)[b:e].clone(), n_rows, m.n_cols, **params)
    H.hbp_free(h)


@pytest.mark.parametrize("kind", [0, 1, 2, 4, 8, 16, 32])
def test_csr_baselines(H, oracle, kind):
    import torch
    for m in (make_config(1), make_config(5, 0.01), random_csr(300, 200, 0.2, 4, empty_row_frac=0.2)):
        ptr, col, val, x = to_dev(m)
        y = torch.full((m.n_rows,), float("nan"), device="cuda")
        H.hbp_csr_spmv(kind, ptr, col, val, x, y)
        torch.cuda.synchronize()
        y_ref, s_abs = oracle.csr_spmv_f64(m.ptr, m.col, m.val, m.x)
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= TOL * s_abs)


def test_csr_baseline_rejects_unknown_kind(H):
    import torch
    m = make_config(1)
    ptr, col, val, x = to_dev(m)
    y = torch.zeros(m.n_rows, device="cuda")
    for kind in (3, 64, -1):
        with pytest.raises(H.HbpError) as e:
            H.hbp_csr_spmv(kind, ptr, col, val, x, y)
        assert e.value.status == -1


def _mixed_matrix(seed=5):
    """Rows of equal length in bulk (full equal groups -> aligned wide loads), a band of short
    rows (packs of several groups), and a few very long rows (deep batches, whole-wavefront
    spans), all inside one block column so that they share groups."""
    from workloads import CsrMatrix
    rng = np.random.default_rng(seed)
    n_cols = 6000
    lens = np.r_[np.full(1500, 12), rng.integers(1, 4, 2000), np.full(700, 5), [5000, 3000, 2999, 800, 799, 300, 64, 63],
                 rng.integers(0, 40, 600), np.full(640, 9)]
    rng.shuffle(lens)
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    ptr = np.r_[0, np.cumsum(lens)].astype(np.int32)
    return CsrMatrix("mixed", len(lens), n_cols, ptr, col, rng.standard_normal(len(col)).astype(np.float32),
                     rng.uniform(-1, 1, n_cols).astype(np.float32))


@pytest.mark.parametrize("rounds", [2, 4, 8, 9, 16])
@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_kernel_variants(H, oracle, rounds, threads):
    """Every instantiation of the SpMV-part kernel (rounds per batch x workgroup size) for workers of few groups, on a
    matrix that reaches all three walking modes, with and without a competitive part.  (Of many: test_steps_*.)"""
    m = _mixed_matrix()
    for q8, workers in ((256, 7), (160, 5)):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=1024, cols_per_block=8192,
                             rounds_per_batch=rounds, threads_per_worker=threads, fixed_fraction_q8=q8,
                             num_workers=workers, slot_weight=3)


@pytest.mark.parametrize("column_weight,ranges_open", [(0, 4), (1, 4), (100, 4), (450, 2), (2000, 0), (-1, 0)])
@pytest.mark.parametrize("workers", [1, 5])
def test_ranges_worth_entering_and_not(H, oracle, column_weight, ranges_open, workers):
    """The library's own share: competitive groups that weigh at least twice the column weight are claimed (those of all ranges that
    have any, of some, of none), the others are run like the fixed part."""
    m = _mixed_matrix()
    info = check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=1024, cols_per_block=2048,
                                rounds_per_batch=4, num_workers=workers, slot_weight=1, group_weight=10, round_weight=1,
                                column_weight=column_weight)
    o = oracle.OracleHbp(m.ptr, m.col, m.val, m.n_rows, m.n_cols, R=1024, C=2048, W=64, num_workers=workers, fixed_q8=info.fixed_fraction_q8,
                         slot_weight=1, round_weight=1, group_weight=10, column_weight=info.column_weight)
    before = o.array("group_ptr").astype(np.int64) + o.array("group_slot") + o.array("group_rounds") + 10 * np.arange(o.G + 1)
    lo, end = o.array("comp_lo"), o.array("fixed_start")[1:]
    is_open = (lo < end) & (before[end] - before[np.minimum(lo, end)] >= 2 * info.column_weight)
    assert is_open.sum() == (ranges_open if workers == 5 else column_weight >= 0)
    o.close()


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("blocks,lens", [
    (30, [127, 128, 129, 130, 200]),       # lists first: heavy from 8192 nonzeros on
    (1100, [255, 256, 257, 258, 300]),     # 1024 groups and more, lists last: never
])
def test_groups_heavy_by_their_nonzeros(H, oracle, blocks, lens, f64):
    """Groups of 64 rows of up to 300 nonzeros, just under, at and over the line, among blocks of one nonzero: each has more than an
    eighth of the range's nonzeros."""
    from workloads import widen_to_f64
    m = _matrix_of_lengths(np.concatenate([np.repeat(lens, 64), np.tile([1] + [0] * 63, blocks)]), 4000, seed=blocks)
    if f64:
        m = widen_to_f64(m)
    check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=64, cols_per_block=4096, rounds_per_batch=4,
                         num_workers=1, threads_per_worker=1024, fixed_fraction_q8=256)


@pytest.mark.parametrize("f64", [False, True])
def test_given_heavy_group_rounds_decide_alone(H, f64):
    """A group that would be shared for its nonzeros is not where the caller's heavy_group_rounds are more than its rows have: its
    sums have the order that they have where no group is listed at all."""
    import torch
    from workloads import widen_to_f64
    m = _matrix_of_lengths(np.r_[np.full(32, 1600), np.full(32, 1601), np.full(640, 3)], 4000, seed=4)
    if f64:
        m = widen_to_f64(m)
    ptr, col, val, x = to_dev(m)
    build, spmv = (H.hbp_build_f64, H.hbp_spmv_f64) if f64 else (H.hbp_build, H.hbp_spmv)
    ys = {}
    for heavy in (0, 100000, 2**30):
        h = build(ptr, col, val, m.n_rows, m.n_cols, rows_per_block=64, cols_per_block=4096, rounds_per_batch=16, num_workers=1,
                  threads_per_worker=1024, fixed_fraction_q8=256, heavy_group_rounds=heavy)
        try:
            ys[heavy] = torch.empty(m.n_rows, device="cuda", dtype=x.dtype)
            spmv(h, x, ys[heavy])
            torch.cuda.synchronize()
        finally:
            H.hbp_free(h)
    assert torch.equal(ys[100000], ys[2**30]) and not torch.equal(ys[0], ys[2**30])


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("blocks", [5, 1100])                      # lists first and last
@pytest.mark.parametrize("big", [0, 63, 64, 65, 71])
def test_heavy_groups_of_both_kinds(H, oracle, big, blocks, f64):
    """Groups with a row of more than 2048 nonzeros, up to more than their list holds, and three that are heavy because they
    outweigh the others; no such group among a hundred of them."""
    from workloads import widen_to_f64
    rows = lambda n, length: np.r_[np.full(n, length), np.zeros(64 - n, int)]
    others = [rows(1, 2100)] * big if big else [rows(64, 150)] * 100
    lens = np.concatenate([rows(64, 500)] * 3 + others + [rows(1, 1)] * blocks)
    m = _matrix_of_lengths(lens, 4000, seed=big)
    if f64:
        m = widen_to_f64(m)
    for q8 in (256, 128):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=64, cols_per_block=4096, rounds_per_batch=4,
                             num_workers=1, threads_per_worker=1024, fixed_fraction_q8=q8)


@pytest.mark.parametrize("threads", [256, 512, 1024])
@pytest.mark.parametrize("q8", [256, 100])
def test_steps_of_short_rows(H, oracle, threads, q8):
    """1024 groups per worker and more, fp32, short batches: runs of groups with rows of one nonzero (longer than a step and
    than a draw, full and not), groups that just fit the wavefront's place in LDS (224 elements) and that just do not,
    a long row among short ones.  64 rows per block, so that the rows of a group are known."""
    rows = lambda *parts: np.concatenate([np.full(n, v) for n, v in parts])
    one = rows((64, 1))
    pattern = [one] * 13 + [rows((64, 3)), one, rows((32, 3), (32, 4)), one, one, rows((33, 4), (31, 3)), rows((31, 4), (33, 3)),
                            rows((1, 161), (63, 1)), rows((1, 162), (63, 1)), rows((5, 1), (59, 0)), rows((17, 2), (47, 0)), one,
                            rows((64, 8)), rows((63, 1), (1, 2)), rows((64, 2)), rows((1, 300), (63, 3))]
    m = _matrix_of_lengths(np.concatenate((pattern * 40)[:1061] + [np.full(37, 1)]), 4000, seed=threads)
    check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=64, cols_per_block=4096, rounds_per_batch=4,
                         threads_per_worker=threads, num_workers=1, fixed_fraction_q8=q8)


@pytest.mark.parametrize("threads", [256, 1024])
@pytest.mark.parametrize("heavy", [0, 16])
def test_steps_of_groups_that_nearly_fit(H, oracle, threads, heavy):
    """224 elements are a wavefront's place in LDS, 256 a step's loads; between them the first two rounds make room for the
    others, in groups of 36 rows and more.  Beside short groups, so that the average one fits."""
    rows = lambda *parts: np.concatenate([np.full(n, v) for n, v in parts] + [np.zeros(64 - sum(n for n, _ in parts), int)])
    nearly = [rows((64, 4)), rows((63, 4), (1, 3)), rows((33, 4), (31, 3)), rows((32, 4), (32, 3)), rows((1, 193), (63, 1)), rows((1, 162), (63, 1)),
              rows((64, 2)), rows((36, 7)), rows((36, 7), (1, 4)), rows((4, 8), (32, 7)), rows((35, 7)), rows((34, 7), (1, 18)), rows((37, 6), (1, 34)),
              rows((1, 256)), rows((2, 128)), rows((40, 6), (1, 17)), rows((51, 5), (1, 1)), rows((51, 5), (1, 2)), rows((1, 221), (35, 1)),
              rows((1, 222), (34, 1)), rows((1, 220), (36, 1)), rows((64, 3)), rows((32, 7), (32, 1)), rows((33, 7), (25, 1))]
    m = _matrix_of_lengths(np.concatenate([g for group in nearly for g in (group, rows((64, 1)), rows((3, 2)))] * 15), 4000, seed=threads)
    check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=64, cols_per_block=4096, rounds_per_batch=4,
                         threads_per_worker=threads, num_workers=1, fixed_fraction_q8=200, heavy_group_rounds=heavy)


@pytest.mark.parametrize("rounds,threads", [(2, 256), (4, 1024)])
@pytest.mark.parametrize("heavy", [0, 16])
def test_packs_of_many_groups(H, oracle, rounds, threads, heavy):
    """1024 groups per worker and more whose average does not fit the steps: packs, with the lists last (and without lists)."""
    rows = lambda *parts: np.concatenate([np.full(n, v) for n, v in parts] + [np.zeros(64 - sum(n for n, _ in parts), int)])
    pattern = [rows((64, 5)), rows((64, 4)), rows((60, 6), (3, 40)), rows((64, 1)), rows((33, 7), (20, 3)), rows((64, 5)), rows((1, 200), (40, 5))]
    m = _matrix_of_lengths(np.concatenate((pattern * 160)[:1063]), 4000, seed=rounds)
    assert m.nnz > 224 * 1063
    for q8 in (256, 100):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=64, cols_per_block=4096, rounds_per_batch=rounds,
                             threads_per_worker=threads, num_workers=1, fixed_fraction_q8=q8, heavy_group_rounds=heavy)


def test_many_columns_competition(H, oracle):
    """More block columns than a wavefront has lanes (the scan for the fullest column loops), tiny
    tickets, more workers than groups."""
    m = random_csr(1500, 9000, 0.01, 31, empty_row_frac=0.2)
    check_against_oracle(H, oracle, m, rows_per_block=128, cols_per_block=64, fixed_fraction_q8=64, claim_chunk=1,
                         num_workers=300, threads_per_worker=256)
    check_against_oracle(H, oracle, m, rows_per_block=128, cols_per_block=64, fixed_fraction_q8=0, claim_chunk=3,
                         num_workers=32, threads_per_worker=512, rounds_per_batch=4)


@pytest.mark.parametrize("unit_slots", [64, 300, 5000])
def test_split_row_blocks(H, oracle, unit_slots):
    """Row blocks cut into several combine units (their sums meet in y through atomic adds), next
    to row blocks with one unit and empty row blocks; R both below and above the 128/256-thread
    switch of the combine kernel."""
    m = _mixed_matrix(seed=41)
    for R in (256, 2048):
        info = check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=512, combine_unit_slots=unit_slots)
        if unit_slots == 64:
            assert info.split_row_blocks > 0


@pytest.mark.parametrize("heavy", [1, 5, 60, 700])
@pytest.mark.parametrize("rounds,threads", [(2, 256), (4, 512), (8, 1024), (9, 1024), (16, 512)])
def test_heavy_groups_shared_by_a_worker(H, oracle, heavy, rounds, threads):
    """Groups with a row longer than heavy_group_rounds are walked by all wavefronts of a worker,
    each taking an equal share of the group's nonzeros.  heavy = 1 makes nearly every group heavy
    (the worker's list overflows and the rest is walked the ordinary way); the larger values
    leave a mix; with and without a competitive part."""
    m = _mixed_matrix(seed=7)
    for q8, workers in ((256, 3), (128, 6)):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=2048, cols_per_block=8192,
                             rounds_per_batch=rounds, threads_per_worker=threads, fixed_fraction_q8=q8,
                             num_workers=workers, heavy_group_rounds=heavy)


def _matrix_of_lengths(lens, n_cols, seed):
    from workloads import CsrMatrix
    rng = np.random.default_rng(seed)
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    ptr = np.r_[0, np.cumsum(lens)].astype(np.int32)
    return CsrMatrix("lengths", len(lens), n_cols, ptr, col, rng.standard_normal(len(col)).astype(np.float32),
                     rng.uniform(-1, 1, n_cols).astype(np.float32))


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("threads", [256, 1024])
@pytest.mark.parametrize("groups", [1, 2, 3, 4, 5, 9])
def test_heavy_groups_walked_side_by_side(H, oracle, groups, threads, f64):
    """One, two or four heavy groups at a time, the last turn with fewer than that; known before the range is walked (first
    case) and found among the claimed groups (second)."""
    from workloads import widen_to_f64
    m = _matrix_of_lengths(np.concatenate([np.arange(64 * groups) % 190 + 65, np.full(100, 3)]), 4000, seed=groups)
    if f64:
        m = widen_to_f64(m)
    for q8 in (256, 0):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=1024, cols_per_block=4096, rounds_per_batch=4,
                             threads_per_worker=threads, num_workers=1, fixed_fraction_q8=q8, heavy_group_rounds=64)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("threads", [256, 1024])
def test_heavy_groups_have_one_order_whoever_claims_them(H, threads, f64):
    """Every group competitive: how many heavy ones a worker claims depends on the number of workers and on timing, a group's sum
    does not."""
    import torch
    from workloads import widen_to_f64
    m = _matrix_of_lengths(np.concatenate([np.arange(64 * 40) % 190 + 65, np.full(3000, 3)]), 4000, seed=40)
    if f64:
        m = widen_to_f64(m)
    ptr, col, val, x = to_dev(m)
    build, spmv = (H.hbp_build_f64, H.hbp_spmv_f64) if f64 else (H.hbp_build, H.hbp_spmv)
    first = None
    for workers in (1, 40, 5):
        h = build(ptr, col, val, m.n_rows, m.n_cols, rows_per_block=1024, cols_per_block=4096, rounds_per_batch=4, claim_chunk=1,
                  threads_per_worker=threads, num_workers=workers, fixed_fraction_q8=0, heavy_group_rounds=64)
        try:
            assert H.hbp_get_info(h).split_row_blocks == 0
            for rep in range(10):
                y = torch.full((m.n_rows,), float("nan"), device="cuda", dtype=x.dtype)
                spmv(h, x, y)
                first = y if first is None else first
                assert torch.equal(y, first), (workers, rep)
        finally:
            H.hbp_free(h)


@pytest.mark.parametrize("seed", range(int(os.environ.get("HBP_RANDOM_CASES", "24"))))  # more seeds for a soak run
def test_random_parameters(H, oracle, seed):
    """Seeded random draws over matrix shape and every build parameter (block sizes, group
    width, workers, fixed share, claim size, weights, kernel variant, combine units, heavy
    threshold): layout bit-exact, y and partial sums within tolerance, twice in a row."""
    rng = np.random.default_rng(1000 + seed)
    n_rows = int(rng.integers(1, 6000))
    n_cols = int(rng.integers(1, 9000))
    density = float(rng.choice([0.002, 0.01, 0.05, 0.2]))
    m = random_csr(n_rows, n_cols, density, 500 + seed, empty_row_frac=float(rng.choice([0.0, 0.3])))
    if seed % 4 == 0:   # a few long rows on top, so that deep batches, spans and heavy groups occur
        m = _with_long_rows(m, rng)
    threads = int(rng.choice([256, 512, 1024]))
    params = dict(
        rows_per_block=int(rng.choice([1, 7, 64, 512, 2048, 8192])),
        cols_per_block=int(rng.choice([1, 33, 256, 4096, 32768])),
        group_width=int(rng.choice([1, 5, 32, 64])),
        num_workers=int(rng.choice([0, 1, 3, 17, 300])),
        fixed_fraction_q8=int(rng.choice([0, 77, 192, 255, 256])),
        claim_chunk=int(rng.choice([0, 1, 3, 50])),
        threads_per_worker=threads,
        rounds_per_batch=int(rng.choice([2, 4, 8, 9, 16])),
        slot_weight=int(rng.choice([0, 1, 4, 64])),
        group_weight=int(rng.choice([0, 10, 4096])),
        round_weight=int(rng.choice([0, 8, 1024])),
        column_weight=int(rng.choice([0, 0, 50, 100000])),
        combine_unit_slots=int(rng.choice([0, 64, 1000])),
        heavy_group_rounds=int(rng.choice([0, 1, 20, 300])),
        hash_shift=int(rng.choice([-1, 0, 3, 12])),
    )
    if params["rows_per_block"] * params["cols_per_block"] < 64 and n_rows * n_cols > 4_000_000:
        params["rows_per_block"] = 64   # keep the block table of the tiny-block cases small
    check_against_oracle(H, oracle, m, check_add_sign=seed % 3 == 0, **params)


def _with_long_rows(m, rng):
    """m with a handful of rows replaced by rows that fill 10 to 90 % of the columns."""
    from workloads import CsrMatrix
    lens = np.diff(m.ptr).astype(np.int64)
    rows = [m.col[m.ptr[i]:m.ptr[i + 1]] for i in range(m.n_rows)]
    for i in rng.choice(m.n_rows, size=min(m.n_rows, 6), replace=False):
        k = max(1, int(m.n_cols * rng.uniform(0.1, 0.9)))
        rows[i] = np.sort(rng.choice(m.n_cols, k, replace=False)).astype(np.int32)
        lens[i] = k
    col = np.concatenate(rows).astype(np.int32) if lens.sum() else np.zeros(0, np.int32)
    ptr = np.r_[0, np.cumsum(lens)].astype(np.int32)
    return CsrMatrix(m.name + "+long", m.n_rows, m.n_cols, ptr, col, rng.standard_normal(len(col)).astype(np.float32), m.x)


@pytest.mark.parametrize("R", [65, 129, 130, 257, 300, 1000, 4097, 8192])
@pytest.mark.parametrize("mode", ["hash", "no_reorder", "key_length", "block_shift"])
def test_block_ordering_paths(H, oracle, R, mode):
    """Both ways a block's slots are ordered (a bitonic network up to 256 slots, counting passes
    through a row table above), with R off the multiples of 64 and of the powers of two, and
    blocks from nearly empty to full: one dense and one sparse column block side by side."""
    rng = np.random.default_rng(R)
    n_rows, n_cols = 2 * R + 17, 600
    lens = np.where(rng.random(n_rows) < 0.9, rng.integers(1, 40, n_rows), 0)
    lens[rng.integers(0, n_rows, 5)] = 500
    cols = []
    for n in lens:
        dense = np.sort(rng.choice(512, min(int(n), 512), replace=False))
        extra = 512 + np.sort(rng.choice(88, 1, replace=False)) if rng.random() < 0.05 else np.empty(0, np.int64)
        cols.append(np.r_[dense, extra])
    ptr = np.zeros(n_rows + 1, np.int32)
    np.cumsum([len(c) for c in cols], out=ptr[1:])
    col = np.concatenate(cols).astype(np.int32)
    from workloads import CsrMatrix
    m = CsrMatrix(name=f"ordering_{R}", n_rows=n_rows, n_cols=n_cols, ptr=ptr, col=col,
                  val=rng.standard_normal(len(col)).astype(np.float32), x=rng.uniform(-1, 1, n_cols).astype(np.float32))
    kw = {} if mode == "hash" else {mode: True}
    check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=512, **kw)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("row_blocks,col_blocks", [(70, 5), (65, 40), (129, 2)])
def test_fill_by_row_block(H, oracle, row_blocks, col_blocks, f64):
    """Short row segments in large blocks over at least 64 row blocks: the build fills the blocks
    row block by row block (several workgroups per row block, a number of row blocks that is no
    multiple of 8, a ragged last one)."""
    from workloads import CsrMatrix, widen_to_f64
    rng = np.random.default_rng(row_blocks * 100 + col_blocks)
    R, C = 512, 256
    n_rows, n_cols = row_blocks * R - 499, col_blocks * C
    per_block = rng.integers(1, 4, (n_rows, col_blocks))          # 1..3 nonzeros of every row in every column block
    per_block[rng.random((n_rows, col_blocks)) < 0.05] = 0        # a few empty segments
    starts = rng.integers(0, C - 3, (n_rows, col_blocks)) + np.arange(col_blocks)[None, :] * C
    lens = per_block.sum(1)
    ptr = np.zeros(n_rows + 1, np.int32)
    np.cumsum(lens, out=ptr[1:])
    col = np.concatenate([np.arange(s, s + k) for s, k in zip(starts.ravel(), per_block.ravel()) if k]).astype(np.int32)
    m = CsrMatrix(name=f"fill_{row_blocks}x{col_blocks}", n_rows=n_rows, n_cols=n_cols, ptr=ptr, col=col,
                  val=rng.standard_normal(len(col)).astype(np.float32), x=rng.uniform(-1, 1, n_cols).astype(np.float32))
    if f64:
        m = widen_to_f64(m)
    info = check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C)
    assert info.row_blocks == row_blocks and info.nnz < 4 * info.slots and info.slots >= 256 * info.blocks


@pytest.mark.parametrize("R,C", [(64, 128), (512, 4096)])
def test_plain_2d_partition(H, oracle, R, C):
    """HBP_FLAG_NO_REORDER: the plain 2D-partitioning method of Section 4 (no hash reorder)."""
    m = _mixed_matrix(seed=3)
    check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C, no_reorder=True)


@pytest.mark.parametrize("R,C", [(64, 128), (2048, 8192)])
def test_length_key(H, oracle, R, C):
    """HBP_FLAG_KEY_LENGTH (hash study): slots in ascending (length, row) order."""
    m = _mixed_matrix(seed=11)
    check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C, key_length=True)
    check_against_oracle(H, oracle, make_config(4, 2**-7), rows_per_block=512, cols_per_block=2048, key_length=True)


def test_hash_values_all_lengths(H, oracle):
    """The device's hash function, value by value: every length a block can hold (0..C with C the
    largest block width), every shift 0..12, for block heights that exercise the clamp to R - 1
    (R = 1, 4), a band of one (R = 9), the paper's 512 and the largest the library accepts."""
    import torch
    n = np.arange(0, 32768 + 1, dtype=np.uint32)
    n_dev = torch.from_numpy(n.astype(np.int32)).cuda()
    for R in (1, 4, 9, 512, 8192):
        for a in range(13):
            got = H.hbp_hash_keys(n_dev, a, R).cpu().numpy().view(np.uint32)
            want = oracle.hash_keys(n, a, R)
            assert np.array_equal(got, want), f"R={R} a={a}: first difference at n={np.flatnonzero(got != want)[:3]}"
    with pytest.raises(H.HbpError):
        H.hbp_hash_keys(n_dev, 13, 512)
    with pytest.raises(H.HbpError):
        H.hbp_hash_keys(n_dev, 0, 8193)


@pytest.mark.parametrize("R,C", [(64, 128), (512, 4096), (2048, 8192)])
def test_block_shift(H, oracle, R, C):
    """HBP_FLAG_BLOCK_SHIFT (hash study): one shift per block, taken from the block's own rows."""
    m = _mixed_matrix(seed=13)
    info = check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C, block_shift=True)
    check_against_oracle(H, oracle, make_config(4, 2**-7), rows_per_block=512, cols_per_block=2048, block_shift=True)
    check_against_oracle(H, oracle, make_config(5, 0.01), rows_per_block=R, cols_per_block=C, block_shift=True)


@pytest.mark.parametrize("P,q8", [(1, 256), (3, 224), (7, 0), (64, 128), (500, 255)])
def test_paper_schedule(H, oracle, P, q8):
    """HBP_FLAG_PAPER_SCHEDULE: Section 3.3 read literally (equal block counts per worker, a single
    ticket counter over the rest).  Schedule arrays bit-equal to the oracle's, y within tolerance,
    twice in a row (the ticket counter is re-armed)."""
    m = random_csr(3000, 3000, 0.01, 21, empty_row_frac=0.1)
    info = check_against_oracle(H, oracle, m, rows_per_block=64, cols_per_block=128, num_workers=P, fixed_fraction_q8=q8,
                                paper_schedule=True)
    assert info.first_ticket_block == P * ((info.blocks * q8) // (256 * P))
    check_against_oracle(H, oracle, _mixed_matrix(seed=17), check_add_sign=False, rows_per_block=1024, cols_per_block=2048,
                         num_workers=P, fixed_fraction_q8=q8, paper_schedule=True, threads_per_worker=512, rounds_per_batch=4)


@pytest.mark.parametrize("q8", [256, 128])
def test_hip_graph_replay(H, oracle, q8):
    """hbp_spmv allocates nothing and records no memset (the combine part re-arms the claim
    counters), so a call can be captured into a HIP graph.  Replays, with eager calls and
    synchronisations in between and x changing under the graph, must each give what an eager
    call gives for the same x (bit for bit: without split row blocks every sum has one order)."""
    import torch
    m = random_csr(4000, 5000, 0.01, 77, empty_row_frac=0.1)
    ptr, col, val, x = to_dev(m)
    h = H.hbp_build(ptr, col, val, m.n_rows, m.n_cols, rows_per_block=256, cols_per_block=1024, fixed_fraction_q8=q8,
                    num_workers=24)
    try:
        assert H.hbp_get_info(h).split_row_blocks == 0
        y_eager = torch.empty(m.n_rows, device="cuda")
        y_graph = torch.full((m.n_rows,), float("nan"), device="cuda")
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):                 # first launches configure the kernels: not under capture
            H.hbp_spmv(h, x, y_graph)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            H.hbp_spmv(h, x, y_graph)
        for rep in range(4):
            x.mul_(1.25).add_(0.01 * rep)
            H.hbp_spmv(h, x, y_eager)
            torch.cuda.synchronize()
            y_graph.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y_graph, y_eager), f"replay {rep}"
            y_ref, s_abs = oracle.csr_spmv_f64(m.ptr, m.col, m.val, x.cpu().numpy())
            assert np.all(np.abs(y_graph.cpu().numpy().astype(np.float64) - y_ref) <= TOL * s_abs)
    finally:
        H.hbp_free(h)


def test_two_handles_on_two_streams(H, oracle):
    """Two handles may run at the same time on different streams (workers never wait for another
    workgroup); each result equals what the handle gives alone."""
    import torch
    ms = [random_csr(6000, 7000, 0.004, 91, empty_row_frac=0.1), make_config(5, 0.01)]
    hs, xs, ys, refs = [], [], [], []
    for m in ms:
        ptr, col, val, x = to_dev(m)
        hs.append(H.hbp_build(ptr, col, val, m.n_rows, m.n_cols, rows_per_block=512, cols_per_block=2048, fixed_fraction_q8=200))
        xs.append(x)
        y = torch.empty(m.n_rows, device="cuda")
        H.hbp_spmv(hs[-1], x, y)
        torch.cuda.synchronize()
        refs.append(y.clone())
        ys.append(torch.full((m.n_rows,), float("nan"), device="cuda"))
    try:
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        for rep in range(3):
            for y in ys:
                y.fill_(float("nan"))
            torch.cuda.synchronize()
            for h, x, y, s in zip(hs, xs, ys, streams):
                for _ in range(4):                      # several calls in a row on each stream
                    H.hbp_spmv(h, x, y, stream=s)
            torch.cuda.synchronize()
            for m, y, ref in zip(ms, ys, refs):
                y_ref, s_abs = oracle.csr_spmv_f64(m.ptr, m.col, m.val, m.x)
                assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= TOL * s_abs), f"rep {rep} {m.name}"
    finally:
        for h in hs:
            H.hbp_free(h)


def _short_rows_with_a_few_long_ones():
    from workloads import CsrMatrix
    rng = np.random.default_rng(12)
    n_cols = 3000
    lens = np.r_[rng.integers(3, 11, 30000), [900, 40, 35], rng.integers(0, 3, 2000)]
    rng.shuffle(lens)
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    ptr = np.r_[0, np.cumsum(lens)].astype(np.int32)
    return CsrMatrix("long_list", len(lens), n_cols, ptr, col, rng.standard_normal(len(col)).astype(np.float32),
                     rng.uniform(-1, 1, n_cols).astype(np.float32))


@pytest.mark.parametrize("rounds,threads", [(4, 512), (8, 1024)])
def test_long_group_list_overflows(H, oracle, rounds, threads):
    """Nearly every group has a row of more than heavy_group_rounds / 8 nonzeros and the workers have fewer than 1024
    groups each: a range's own long groups wait on a list (1024 entries, enough here) and go first, the claimed ones on
    another one (256 entries); a few rows are long enough for the cooperative heavy path as well.  Lists that do
    overflow: test_full_lists_of_long_groups."""
    m = _short_rows_with_a_few_long_ones()
    for workers, q8 in ((1, 256), (3, 128)):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=4096, cols_per_block=4096,
                             rounds_per_batch=rounds, threads_per_worker=threads, num_workers=workers,
                             fixed_fraction_q8=q8, heavy_group_rounds=16)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("rounds,threads", [(4, 512), (8, 1024)])
@pytest.mark.parametrize("workers,W,q8", [
    (1, 64, 0),      # lists first: all groups are claimed, more long ones than the list of claimed groups holds
    (1, 2, 256),     # lists last (1024 groups and more per worker): more long ones in the range than the list holds
    (3, 2, 100),     # the same, in the fixed parts and among the claimed groups
    (20, 2, 256),    # lists first: ranges with few long groups and with many
])
def test_full_lists_of_long_groups(H, oracle, workers, W, q8, rounds, threads, f64):
    """Long groups that do not fit their list are walked where they were drawn."""
    from workloads import widen_to_f64
    m = _short_rows_with_a_few_long_ones()
    if f64:
        m = widen_to_f64(m)
    heavy, params = 16, dict(rows_per_block=4096, cols_per_block=4096, group_width=W, rounds_per_batch=rounds, threads_per_worker=threads,
                             num_workers=workers, fixed_fraction_q8=q8, heavy_group_rounds=16)
    ptr, col, val, _ = to_dev(m)
    h = (H.hbp_build_f64 if f64 else H.hbp_build)(ptr, col, val, m.n_rows, m.n_cols, **params)
    try:
        longest = np.diff(H.hbp_export(h, "group_rounds"))
        start, comp = H.hbp_export(h, "fixed_start"), H.hbp_export(h, "comp_lo")
    finally:
        H.hbp_free(h)
    first = len(longest) < 1024 * workers
    is_long = (longest > max(1, heavy // 64, min(heavy // 8, 32)) if first else longest > heavy // 8) & (longest <= heavy)
    own = [int(is_long[a:b].sum()) for a, b in zip(start[:-1], comp)]                 # fixed parts
    claimed = [int(is_long[a:b].sum()) for a, b in zip(comp, start[1:])]
    if workers == 1 and q8 == 0:
        assert first and claimed[0] > 256
    elif workers < 20:
        assert not first and max(own) > 256
    else:
        assert first and max(own) > 256
    check_against_oracle(H, oracle, m, check_add_sign=False, **params)


def test_release_workspace(H, oracle):
    """The build's scratch memory is kept between builds and can be given back; builds before
    and after that are the same."""
    m = random_csr(3000, 2000, 0.01, 61)
    check_against_oracle(H, oracle, m, rows_per_block=128, cols_per_block=256)
    H.hbp_release_workspace()
    H.hbp_release_workspace()           # nothing held: still fine
    check_against_oracle(H, oracle, make_config(3, 2**-6), rows_per_block=256, cols_per_block=1024)
    check_against_oracle(H, oracle, m, rows_per_block=128, cols_per_block=256)   # a smaller one in the kept memory


def test_maximum_workers(H, oracle):
    """The largest worker count the library accepts (65536 ranges, nearly all of them empty), with
    and without a competitive part, and one more than that refused."""
    m = random_csr(2000, 3000, 0.01, 71, empty_row_frac=0.2)
    for q8 in (256, 100):
        info = check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=64, cols_per_block=256,
                                    num_workers=65536, threads_per_worker=256, fixed_fraction_q8=q8)
        assert info.num_workers == 65536
    ptr, col, val, x = to_dev(m)
    with pytest.raises(H.HbpError) as e:
        H.hbp_build(ptr, col, val, m.n_rows, m.n_cols, num_workers=65537)
    assert e.value.status == -1


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("lens,n_cols,R,C,W", [
    ([1], 1, 512, 512, 64),                                          # a single nonzero
    ([0, 0, 3, 0], 5, 2, 8, 64),                                     # empty row blocks, empty first and last rows
    ([5] * 1000 + [0] * 40 + [4] * 30, 600, 512, 1024, 64),          # one wavefront per group, rows without a slot
    ([5] * 1000 + [0] * 40 + [4] * 30, 600, 512, 100, 64),           # the same over several block columns
    ([32] * 64 + [33] * 64 + [31] * 7, 4096, 512, 4096, 64),         # 2048 nonzeros a group, and 64 more
    ([64] * 20 + [65] * 20 + [9] * 100, 3000, 64, 3000, 20),         # rows around 64 nonzeros, narrow groups
    ([1] * 300 + [3000, 2500, 17] + [2] * 300, 4000, 512, 4000, 64), # a long group that is nearly all one row
    ([1] * 300 + [3000, 2500, 17] + [2] * 300, 4000, 200, 1500, 64),
    ([700] * 130, 1400, 8, 1400, 3),                                 # more long groups than others
])
def test_small_matrices_without_workers(H, oracle, lens, n_cols, R, C, W, f64):
    """Small matrices run without the workers' schedule: one wavefront or four per group, a workgroup
    for a long group, y written directly where there is one block column."""
    from workloads import CsrMatrix, widen_to_f64
    rng = np.random.default_rng(len(lens) + n_cols)
    lens = np.asarray(lens)
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    m = CsrMatrix("small", len(lens), n_cols, np.r_[0, np.cumsum(lens)].astype(np.int32), col,
                  rng.standard_normal(len(col)).astype(np.float32), rng.uniform(-1, 1, n_cols).astype(np.float32))
    if f64:
        m = widen_to_f64(m)
    info = check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C, group_width=W)
    assert (info.bytes_combine == 0) == (info.col_blocks == 1)     # y written by the one launch there is
    # an infinity in x reaches the rows that hold its column and no other
    import torch
    ptr, cols, val, x = to_dev(m)
    c = int(m.col[len(m.col) // 2])
    x[c] = float("inf")
    build, spmv = (H.hbp_build_f64, H.hbp_spmv_f64) if f64 else (H.hbp_build, H.hbp_spmv)
    h = build(ptr, cols, val, m.n_rows, m.n_cols, rows_per_block=R, cols_per_block=C, group_width=W)
    try:
        y = torch.zeros(m.n_rows, device="cuda", dtype=x.dtype)
        spmv(h, x, y)
        rows = np.repeat(np.arange(m.n_rows), lens)
        assert np.array_equal(np.flatnonzero(~np.isfinite(y.cpu().numpy())), rows[m.col == c])
    finally:
        H.hbp_free(h)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("heavy", [0, 64, 700])
@pytest.mark.parametrize("rounds,threads", [(2, 256), (4, 512), (8, 1024), (9, 256), (16, 512)])
def test_infinities_and_nan_stay_in_their_rows(H, rounds, threads, heavy, f64):
    """An infinity or NaN in x reaches the rows that hold its column and no other, through every walk of the
    workers' kernel but the steps (next test; a small matrix without workers: test_small_matrices_without_workers)."""
    import torch
    from workloads import widen_to_f64
    m = _mixed_matrix(seed=19)
    if f64:
        m = widen_to_f64(m)
    ptr, cols, val, x = to_dev(m)
    rows = np.repeat(np.arange(m.n_rows), np.diff(m.ptr))
    used = np.bincount(m.col, minlength=m.n_cols)
    rare = np.argsort(used, kind="stable")[:3]                  # columns of few rows
    build, spmv = (H.hbp_build_f64, H.hbp_spmv_f64) if f64 else (H.hbp_build, H.hbp_spmv)
    for C in (m.n_cols, 2048):
        h = build(ptr, cols, val, m.n_rows, m.n_cols, rows_per_block=2048, cols_per_block=C, rounds_per_batch=rounds,
                  threads_per_worker=threads, num_workers=5, heavy_group_rounds=heavy)
        try:
            # each column block's first column is what lanes without an element read
            for bad in ({int(rare[0]): float("inf")}, {int(rare[1]): float("nan"), int(rare[2]): float("-inf")},
                        {c: float("inf") for c in range(0, m.n_cols, C)}):
                xb = x.clone()
                for c, v in bad.items():
                    xb[c] = v
                y = torch.zeros(m.n_rows, device="cuda", dtype=x.dtype)
                spmv(h, xb, y)
                hit = np.unique(rows[np.isin(m.col, list(bad))])
                assert np.array_equal(np.flatnonzero(~np.isfinite(y.cpu().numpy())), hit), (C, bad)
        finally:
            H.hbp_free(h)


@pytest.mark.parametrize("threads", [256, 1024])
@pytest.mark.parametrize("heavy", [0, 64])    # without and with lists
def test_infinities_and_nan_stay_in_their_rows_in_steps(H, threads, heavy):
    """1024 groups per worker and more, fp32, short batches: groups that fit a wavefront's place in LDS, that nearly do and that do
    not, runs of rows of one nonzero, and blocks with few rows, whose steps have lanes without a row."""
    import torch
    rows = lambda *parts: np.concatenate([np.full(n, v) for n, v in parts] + [np.zeros(64 - sum(n for n, _ in parts), int)])
    pattern = [rows((64, 1)), rows((64, 1)), rows((64, 3)), rows((64, 1)), rows((3, 2)), rows((64, 4)), rows((5, 1)), rows((63, 1), (1, 70)),
               rows((17, 2)), rows((36, 7)), rows((1, 1)), rows((32, 9)), rows((40, 1), (1, 2))]
    m = _matrix_of_lengths(np.concatenate(pattern * 90), 4000, seed=threads)
    ptr, cols, val, x = to_dev(m)
    of_row = np.repeat(np.arange(m.n_rows), np.diff(m.ptr))
    rare = np.argsort(np.bincount(m.col, minlength=m.n_cols), kind="stable")[:3]
    h = H.hbp_build(ptr, cols, val, m.n_rows, m.n_cols, rows_per_block=64, cols_per_block=4096, rounds_per_batch=4,
                    threads_per_worker=threads, num_workers=1, heavy_group_rounds=heavy)
    try:
        assert H.hbp_get_info(h).groups >= 1024
        for bad in ({int(rare[0]): float("inf")}, {int(rare[1]): float("nan"), int(rare[2]): float("-inf")}, {0: float("inf")}, {0: float("nan")}):
            xb = x.clone()
            for c, v in bad.items():
                xb[c] = v
            y = torch.zeros(m.n_rows, device="cuda", dtype=x.dtype)
            H.hbp_spmv(h, xb, y)
            hit = np.unique(of_row[np.isin(m.col, list(bad))])
            assert np.array_equal(np.flatnonzero(~np.isfinite(y.cpu().numpy())), hit), bad
    finally:
        H.hbp_free(h)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("rounds,threads", [(4, 256), (8, 512)])
@pytest.mark.parametrize("workers,W,lens", [
    (2, 1, [2] * 1990 + [60] * 40),                       # more long groups in a range than its list holds
    (1, 2, [2] * 2000 + [1, 9, 70, 3] * 40 + [1] * 700),  # many groups per worker: the lists come last
    (3, 2, [2] * 2000 + [1, 9, 70, 3] * 40 + [1] * 700),  # few: the lists come first
    (2, 64, [3] * 32 + [8] * 31 + [196] + [3] * 63 + [196, 99] + [4] * 62),  # rests of 192 elements and around (96 in fp64)
])
def test_long_groups_before_and_after_the_others(H, oracle, workers, W, lens, rounds, threads, f64):
    from workloads import CsrMatrix, widen_to_f64
    rng = np.random.default_rng(workers + W)
    n_cols = 400
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    m = CsrMatrix("lists", len(lens), n_cols, np.r_[0, np.cumsum(lens)].astype(np.int32), col,
                  rng.standard_normal(len(col)).astype(np.float32), rng.uniform(-1, 1, n_cols).astype(np.float32))
    if f64:
        m = widen_to_f64(m)
    for q8, heavy in ((256, 64), (100, 16), (0, 2048)):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=4096, cols_per_block=n_cols, group_width=W,
                             rounds_per_batch=rounds, threads_per_worker=threads, num_workers=workers, fixed_fraction_q8=q8,
                             heavy_group_rounds=heavy, slot_weight=0, group_weight=0, round_weight=0, column_weight=0)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("lens", [
    [60] * 700,                                   # all of one length: none is long, whatever that length
    [60] * 700 + [200, 300] * 5,                  # and where a few are longer
    [32] * 640 + [33, 96, 97] * 20,               # around a 64th of 2048 and around three times the mean
    [300] * 256 + [380, 2047, 2048, 2049] * 3,    # a quarter more than the mean, heavy ones
])
def test_long_groups_beside_the_average(H, oracle, lens, f64):
    from workloads import CsrMatrix, widen_to_f64
    rng = np.random.default_rng(len(lens))
    n_cols = 3000
    lens = rng.permutation(np.asarray(lens))
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    m = CsrMatrix("beside", len(lens), n_cols, np.r_[0, np.cumsum(lens)].astype(np.int32), col,
                  rng.standard_normal(len(col)).astype(np.float32), rng.uniform(-1, 1, n_cols).astype(np.float32))
    if f64:
        m = widen_to_f64(m)
    for workers, q8, rounds in ((1, 256, 8), (3, 100, 4)):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=512, cols_per_block=n_cols, num_workers=workers,
                             fixed_fraction_q8=q8, rounds_per_batch=rounds)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("threads", [0, 256, 512, 1024])
@pytest.mark.parametrize("slice_bytes", [400, 32000, 48000, 63800, 65536, 72000, 81920, 100000, 131072])
def test_planned_workers_fit_the_device(H, slice_bytes, threads, f64):
    """The workers that the library plans are on the device at once: their slices of x and the kernel's own arrays (bytes
    as the compiler reports them for the variant with lists) fit the 160 KB of a CU, their wavefronts its 16 of 128
    registers per lane; and where two workers of 512 threads fit a CU there are two, else one of 1024."""
    import torch
    own = {256: 10736, 512: 17936, 1024: 32336}
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    vb = 8 if f64 else 4
    n = 16 * cus + 100                        # a group per row: no fewer groups than wavefronts
    ptr = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    col = torch.zeros(n, dtype=torch.int32, device="cuda")
    val = torch.ones(n, dtype=torch.float64 if f64 else torch.float32, device="cuda")
    build = H.hbp_build_f64 if f64 else H.hbp_build
    h = build(ptr, col, val, n, 10**6, group_width=1, cols_per_block=slice_bytes // vb, threads_per_worker=threads)
    try:
        info = H.hbp_get_info(h)
        T, per_cu = info.threads_per_worker, info.num_workers // cus
        assert info.num_workers == per_cu * cus and per_cu >= 1
        assert per_cu * (slice_bytes + own[T]) <= 160 * 1024 and per_cu * T <= 1024
        if threads == 0:
            assert (T, per_cu) == ((512, 2) if 2 * (slice_bytes + own[512]) <= 160 * 1024 else (1024, 1))
    finally:
        H.hbp_free(h)


def test_rebuilds_reuse_memory_of_freed_handles(H, oracle):
    """A build after a free may get the freed handle's memory; the layouts and products are those of fresh memory,
    with handles of other sizes and of the other value type in between, and after the memory was given back."""
    from workloads import widen_to_f64
    a, b = random_csr(3000, 2000, 0.01, 81, empty_row_frac=0.1), random_csr(900, 5000, 0.02, 82)
    for m in (a, b, a, widen_to_f64(a), b, a):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=256, cols_per_block=512, num_workers=9)
    H.hbp_release_workspace()
    check_against_oracle(H, oracle, a, check_add_sign=False, rows_per_block=256, cols_per_block=512, num_workers=9)


@pytest.mark.parametrize("lens,n_cols,R,C", [
    ([4095], 5000, 16, 4096), ([4096], 5000, 16, 5000), ([4096, 1], 5000, 16, 5000), ([1] * 4095 + [2], 3, 4096, 3),
    ([8192, 8192], 8192, 1, 8192),                                     # segments longer than a tile, cut at its ends
    ([20000, 3, 0, 0, 9000], 20000, 8, 20000),
    ([2] * 2000 + [0] * 5000 + [3] * 40 + [0] * 30000 + [1] * 700, 600, 512, 128),   # gaps of empty rows inside a tile
    ([0] * 3000 + [1, 0, 0, 0] * 1200 + [0] * 3000, 5000, 7, 100),     # few rows that start in a tile, many blocks
    # rows looked for from the nonzeros (32768 rows and more between a tile's first and its last): all tiles, the last one
    # for the empty rows behind it, around the limit, a row and a segment across tiles in between
    (([1] + [0] * 20) * 5000, 300, 512, 64), ([3] * 3000 + [0] * 40000, 300, 512, 64),
    ([4096] + [2] * 100 + [0] * 32567 + [1] * 3995, 5000, 512, 5000), ([4096] + [2] * 100 + [0] * 32568 + [1] * 3995, 5000, 512, 5000),
    ([0] * 50000 + [2] * 1000 + [0] * 20000 + [9000] + [0] * 35000 + [1, 0] * 1500 + [0] * 7, 10000, 2048, 700),
])
def test_segments_at_the_ends_of_tiles(H, oracle, lens, n_cols, R, C):
    """The build finds the segments in tiles of 4096 nonzeros: sizes around one, rows and segments across several,
    and rows without a nonzero between the rows of a tile."""
    from workloads import CsrMatrix
    rng = np.random.default_rng(len(lens))
    lens = np.asarray(lens)
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    m = CsrMatrix("tiles", len(lens), n_cols, np.r_[0, np.cumsum(lens)].astype(np.int32), col,
                  rng.standard_normal(len(col)).astype(np.float32), rng.uniform(-1, 1, n_cols).astype(np.float32))
    check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C)
    check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C, hash_shift=5)   # bands narrower than 2^a


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("long,W", [
    ([512], 64), ([513], 64),                                  # the longest row with its group filled as a whole, the shortest with it cut
    ([127, 128, 129, 255, 256, 257, 513, 640, 641], 64),       # ends of rows at the cuts, after 128 rounds each
    ([640] * 70 + [641] * 3, 64), ([3000, 1, 700] * 5, 5),     # whole groups that go on together, narrow groups
    ([9000], 1),
])
def test_groups_cut_where_rows_are_much_longer(H, oracle, long, W, f64):
    """A row of more than 512 nonzeros among short ones: several wavefronts fill a group, 128 rounds each."""
    from workloads import CsrMatrix, widen_to_f64
    rng = np.random.default_rng(len(long) + W)
    n_cols = 10000
    lens = rng.permutation(np.r_[rng.integers(0, 4, 4000), long])
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    m = CsrMatrix("cut", len(lens), n_cols, np.r_[0, np.cumsum(lens)].astype(np.int32), col,
                  rng.standard_normal(len(col)).astype(np.float32), rng.uniform(-1, 1, n_cols).astype(np.float32))
    if f64:
        m = widen_to_f64(m)
    check_against_oracle(H, oracle, m, rows_per_block=1024, cols_per_block=10000, group_width=W)
    check_against_oracle(H, oracle, m, rows_per_block=2048, cols_per_block=1700, group_width=W)


@pytest.mark.parametrize("f64,units,R,share", [
    (True, 512, 2048, 0.3), (True, 513, 2048, 0.3), (True, 768, 2048, 0.3), (True, 769, 2048, 0.3), (False, 1025, 2048, 0.3), (False, 1536, 2048, 0.3),
    (False, 1024, 2048, 0.3), (False, 1537, 2048, 0.3), (True, 1025, 1037, 0.3), (False, 2305, 1025, 0.3), (False, 2304, 1200, 0.3),
    (True, 513, 2048, 0.1), (True, 769, 2048, 0.1), (False, 1025, 2048, 0.1), (False, 2560, 1025, 0.1),   # blocks of fewer than 128 slots
])
def test_combine_with_three_wavefronts(H, oracle, units, f64, R, share):
    """The numbers of combine units around those that three wavefronts each, but not four, have on the device at once (which of them
    runs: test_wavefronts_of_the_combine_part), with blocks of many and of few slots."""
    from workloads import CsrMatrix, widen_to_f64
    rng = np.random.default_rng(units)
    n_rows, n_cols = R * units - 7, 40000
    lens = np.where(rng.random(n_rows) < share, rng.integers(1, 3, n_rows), 0)
    first = rng.integers(0, n_cols // 2, n_rows)                  # at most two nonzeros, half of the columns apart
    ptr = np.r_[0, np.cumsum(lens)].astype(np.int32)
    col = np.empty(ptr[-1], np.int32)
    col[ptr[:-1][lens > 0]] = first[lens > 0]
    col[ptr[:-1][lens > 1] + 1] = first[lens > 1] + n_cols // 2
    m = CsrMatrix("units", n_rows, n_cols, ptr, col, rng.standard_normal(len(col)).astype(np.float32), rng.uniform(-1, 1, n_cols).astype(np.float32))
    if f64:
        m = widen_to_f64(m)
    info = check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=10000 if R > 1500 or share < 0.3 else 16000)
    assert info.combine_units == units
    assert (info.slots < 128 * info.blocks) == (share < 0.3)


@pytest.mark.parametrize("blocks", [8191, 8192, 8193, 16384, 16385])
@pytest.mark.parametrize("empty", [0, 3])
def test_scans_at_the_ends_of_a_workgroups_turns(H, oracle, blocks, empty):
    """A row per block: the scans over the block table, the row blocks and the groups have as many entries, 8192 to a turn of the
    workgroup that scans alone, and 16385 are for the two kernels; with empty rows the last two have fewer."""
    from workloads import CsrMatrix
    rng = np.random.default_rng(blocks)
    lens = rng.integers(1, 4, blocks + empty)
    lens[rng.choice(blocks + empty, empty, replace=False)] = 0
    n_cols = 60
    col = np.concatenate([np.sort(rng.choice(n_cols, n, replace=False)) for n in lens]).astype(np.int32)
    m = CsrMatrix("scans", len(lens), n_cols, np.r_[0, np.cumsum(lens)].astype(np.int32), col,
                  rng.standard_normal(len(col)).astype(np.float32), rng.uniform(-1, 1, n_cols).astype(np.float32))
    info = check_against_oracle(H, oracle, m, rows_per_block=1, cols_per_block=n_cols, group_width=2)
    assert (info.blocks, info.groups) == (blocks, blocks)
