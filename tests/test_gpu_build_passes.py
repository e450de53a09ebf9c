"""The build's passes over the segments at the sizes where they go other ways: layouts bit for bit and products against the oracle."""
import numpy as np
import pytest

from test_gpu_parity import H, check_against_oracle  # noqa: F401  (H is a fixture)
from workloads.generators import CsrMatrix

pytestmark = pytest.mark.gpu


def matrix(lens, n_cols, seed=1, f64=False, run=0):
    """Rows of the given lengths; columns at random, or `run` neighbouring ones at a time."""
    rng = np.random.default_rng(seed)
    lens = np.minimum(np.asarray(lens, dtype=np.int64), n_cols)
    ptr = np.r_[0, np.cumsum(lens)]
    cols = []
    for n in lens:
        if run:
            starts = rng.choice(max(1, n_cols // run), size=(int(n) + run - 1) // run, replace=False)
            c = (np.sort(starts)[:, None] * run + np.arange(run)).ravel()[:n]
        else:
            c = np.sort(rng.choice(n_cols, size=int(n), replace=False))
        cols.append(c)
    col = np.concatenate(cols) if cols else np.zeros(0)
    val = rng.standard_normal(col.size)
    x = rng.uniform(-1, 1, n_cols)
    dt = np.float64 if f64 else np.float32
    return CsrMatrix("passes", lens.size, n_cols, ptr.astype(np.int32), col.astype(np.int32), val.astype(dt), x.astype(dt))


# A segment's entry in the list: 12 bits for its place in the tile, the row's, the block column's; in all 32, and 33 (no list).
@pytest.mark.parametrize("n_cols", [128 * 64, 128 * 64 + 1])
@pytest.mark.parametrize("f64", [False, True])
def test_lists_of_segments_that_do_and_do_not_fit(H, oracle, n_cols, f64):
    R = 4096 if f64 else 8192
    lens = np.random.default_rng(2).integers(0, 9, 9000)
    check_against_oracle(H, oracle, matrix(lens, n_cols, f64=f64), rows_per_block=R, cols_per_block=64 if not f64 else 32)


# Segments per tile, of which there are as many as block columns change: 138 to 1200 in these.
@pytest.mark.parametrize("run", [17, 16, 15, 8, 7, 4, 3, 1])
@pytest.mark.parametrize("R,C", [(512, 1000), (700, 1024), (64, 128)])
def test_wavefronts_to_a_tile(H, oracle, run, R, C):
    m = matrix(np.full(700, 51), 51 * 40, run=run)
    check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C)


# Block columns as wide as the runs, so that each of these is a segment: 1, 2, 4 and 8 wavefronts to a tile in k_place (which of them: test_build_routes.py); the
# last tile is short.
RUNS = {17: 1, 16: 2, 15: 2, 8: 4, 7: 4, 4: 4, 3: 8, 1: 8}


def runs(run, f64):
    return matrix(np.full(700, 51), 51 * 20, run=run, f64=f64)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("run", RUNS)
@pytest.mark.parametrize("R", [512, 700, 64])
def test_wavefronts_to_a_tile_of_runs(H, oracle, run, R, f64):
    check_against_oracle(H, oracle, runs(run, f64), rows_per_block=R, cols_per_block=run)


# Tiles over one, two, and many row blocks, most of them empty: a segment's row block is looked for.
@pytest.mark.parametrize("every", [1, 3, 50, 700])
@pytest.mark.parametrize("R,C", [(1, 300), (7, 300), (16, 64), (512, 300)])
def test_tiles_over_many_row_blocks(H, oracle, every, R, C):
    lens = np.zeros(3000 * every, dtype=np.int64)[:400_000]
    lens[::every] = np.random.default_rng(3).integers(1, 6, lens[::every].size)
    check_against_oracle(H, oracle, matrix(lens, 300), rows_per_block=R, cols_per_block=C)


def quick(lens, n_cols, seed, f64, long=()):
    """Like `matrix`, for many rows: columns drawn with replacement and merged; `long`: (row, first column, columns) runs of neighbouring
    columns in place of a row's own."""
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens, dtype=np.int64)
    rows = np.repeat(np.arange(lens.size, dtype=np.int64), lens)
    keys = rows * n_cols + rng.integers(0, n_cols, rows.size)
    keys = keys[~np.isin(rows, [r for r, _, _ in long])]
    keys = np.unique(np.concatenate([keys] + [r * n_cols + np.arange(c0, c0 + n) for r, c0, n in long]))
    ptr = np.searchsorted(keys, np.arange(lens.size + 1) * n_cols).astype(np.int32)
    dt = np.float64 if f64 else np.float32
    return CsrMatrix("row blocks", lens.size, n_cols, ptr, (keys % n_cols).astype(np.int32), rng.standard_normal(keys.size).astype(dt),
                     rng.uniform(-1, 1, n_cols).astype(dt))


def totals(m, R, C):
    """Segments, groups, blocks, row blocks that hold something, and the most segments and nonzeros of one; the longest row, where it has more than 512 nonzeros, and
    whether three words of 64 nonzeros in a row are without a segment's begin in one tile of 4096."""
    NBR, NBC = -(-m.n_rows // R), -(-m.n_cols // C)
    row, bn = np.repeat(np.arange(m.n_rows), np.diff(m.ptr)), m.col // C
    start = np.r_[True, (row[1:] != row[:-1]) | (bn[1:] != bn[:-1])]
    slots = np.bincount(row[start] // R * NBC + bn[start], minlength=NBR * NBC)
    nonzeros, longest = np.bincount(row // R, minlength=NBR), int(np.diff(m.ptr).max())
    without = np.zeros((-(-m.nnz // 4096), 64), dtype=bool)
    without.ravel()[:m.nnz // 64] = start[:m.nnz // 64 * 64].reshape(-1, 64).sum(1) == 0
    return dict(S=int(start.sum()), G=int((-(-slots // 64)).sum()), B=int((slots > 0).sum()), row_blocks=int((nonzeros > 0).sum()),
                most_slots=int(slots.reshape(NBR, NBC).sum(1).max()), most_nonzeros=int(nonzeros.max()), longest=longest if longest > 512 else 0,
                long=int((without[:, :-2] & without[:, 1:-1] & without[:, 2:]).any()))


def behind_empty_row_blocks(m, R, C):
    """The matrix with as many empty row blocks in front as make row blocks as a whole worth while in fp32, and so in fp64 (the fewer of all row blocks hold something,
    the less they have to hold): small matrices would all go the other way.  128 row blocks at least."""
    t = totals(m, R, C)
    turns = -(-t["row_blocks"] // 256)
    NBR = max(128, int((4.5 * turns - 1) * 1e6 * t["row_blocks"] / (t["S"] + m.nnz)) + 1)
    more = max(0, NBR - -(-m.n_rows // R)) * R
    return CsrMatrix(m.name, m.n_rows + more, m.n_cols, np.r_[np.zeros(more, np.int32), m.ptr], m.col, m.val, m.x)


def by_type(make):
    """make(f64) for either type from one matrix in fp64."""
    def of(f64):
        m, params, whole = make()
        return (m if f64 else CsrMatrix(m.name, m.n_rows, m.n_cols, m.ptr, m.col, m.val.astype(np.float32), m.x.astype(np.float32))), params, whole
    return of


# What test_build_routes.py holds against the library's rule, too: matrices, parameters and whether they go by row blocks as a whole.
WHOLE = {}


# Row blocks as a whole: 128 and more of them, rows short in every block column, blocks of 256 slots on average.  One to 64 block columns, block
# sizes that are no powers of two, ragged last blocks, row blocks without a nonzero and tiles over several row blocks, every shift that fits and one that does
# not; bits that fit the LDS at one shift and not at the next (16 block columns at R = 2048, a = 1 and 2), and at a = 1 where there are 64 block columns (R = 512).
ROW_BLOCKS = [
    (512, 512 * 127 + 1, 900, 900, 3, -1), (512, 512 * 127, 900, 900, 3, -1),
    (512, 66_000, 300, 599, 6, 0), (700, 90_001, 500, 2_500, 9, 1), (512, 66_000, 64, 4_096, 62, 0), (512, 66_000, 64, 4_096, 62, 1),
    (1000, 130_000, 333, 1_000, 6, 2), (2048, 270_000, 700, 4_000, 9, 3), (2048, 270_000, 700, 4_000, 9, -1), (2047, 262_016, 32, 64, 5, 6),
    (2048, 40_000, 256, 4_096, 30, 1), (2048, 40_000, 256, 4_096, 30, 2),
]
REFUSED = [(2048, 270_000, 700, 4_000, 9, 3), (2047, 262_016, 32, 64, 5, 6), (2048, 40_000, 256, 4_096, 30, 2)]


def row_blocks(R, n_rows, C, n_cols, mean, shift):
    rng = np.random.default_rng(R + n_cols)
    lens = rng.poisson(mean, n_rows)
    lens[R * 5:R * 7] = 0
    lens[R * 20 + 3:R * 20 + 40] = 0
    m = behind_empty_row_blocks(quick(lens, n_cols, 5, True), R, C)
    return m, dict(rows_per_block=R, cols_per_block=C, hash_shift=shift), (R, n_rows, C, n_cols, mean, shift) not in REFUSED


for _p in ROW_BLOCKS:
    WHOLE["rows of %d in %d x %d of %d x %d, shift %d" % (_p[4], _p[0], _p[2], _p[1], _p[3], _p[5])] = by_type(lambda p=_p: row_blocks(*p))


# Every row block in use, each in one share: no lists.  (An fp32 share holds 27,306 nonzeros, an fp64 one 16,384.)
def all_row_blocks(mean, n):
    lens = np.random.default_rng(mean).poisson(mean, 1024 * n - 5)
    return quick(lens, 3_000, 6, True), dict(rows_per_block=1024, cols_per_block=300), True


WHOLE["all row blocks, one fp64 share"] = by_type(lambda: all_row_blocks(15, 160))
WHOLE["all row blocks, one fp32 share"] = by_type(lambda: all_row_blocks(20, 129))

# Row blocks in one and several shares, groups that lie in two of them, rows of up to a block's width, alone and 70 in a row, with tails of one and several pieces
# of 64 rounds; more nonzeros than a row block may have (those of the last list, by themselves).  A group's rows of fewer than 8 * 2^a nonzeros are in order of
# their lengths and the others come behind: at every shift that fits.
LONG = {
    "lengths at edges": [(9, 0, 63), (70, 5, 64), (90, 600, 65), (2100, 0, 96), (2200, 0, 97), (4200, 7, 576), (5000, 7, 577)],
    "70 in a row": [(r, 10 * (r % 50), 500) for r in range(100, 170)],
    "full rows": [(300, 0, 3000), (301, 0, 3000), (302, 0, 2999), (303, 1, 1)],
    "50 of 700": [(r, 0, 700) for r in range(600, 650)],
    "too many": [(r, 0, 1500) for r in range(600, 645)],
}


def shares(long, mean, R, shift):
    lens = np.random.default_rng(mean).poisson(mean, 262_145)
    m = behind_empty_row_blocks(quick(lens, 3_000, 6, True, LONG[long]), R, 600)
    return m, dict(rows_per_block=R, cols_per_block=600, hash_shift=shift), long != "too many"


for _long in LONG:
    for _mean, _R, _shift in ((6, 2048, -1), (6, 1024, -1), (13, 2048, -1), (13, 1024, -1)) + ((6, 2048, 1), (13, 1024, 2), (6, 1024, 2)) * (_long in ("lengths at edges", "70 in a row", "full rows")):
        WHOLE["%s, rows of %d, R = %d, shift %d" % (_long, _mean, _R, _shift)] = by_type(lambda p=(_long, _mean, _R, _shift): shares(*p))


# Five groups of each of five blocks with a row of 600 nonzeros among rows of 15: 14,800 rounds behind the first eight (14,600 behind the first sixteen, 14,200), the list holds 12,288.
def many_tails(shift):
    lens = np.random.default_rng(8).poisson(6, 262_145)
    lens[:300] = 75
    m = behind_empty_row_blocks(quick(lens, 3_000, 9, True, [(r, 0, 3_000) for r in (10, 70, 130, 190, 250)]), 2048, 600)
    return m, dict(rows_per_block=2048, cols_per_block=600, hash_shift=shift), True


for _shift in (0, 1, 2):
    WHOLE["more rounds than the list of tails holds, shift %d" % _shift] = by_type(lambda p=_shift: many_tails(p))


# As many segments as a row block may have, and one more: every row in all of 16 block columns, and one in a 17th.
def full_row_block(one_more):
    lens = np.random.default_rng(13).poisson(12, 2048 * 8)
    lens[2048 * 3:2048 * 4] = 0
    runs = [(2048 * 3 + r, 100 * c + (7 * r + c) % 98, 1 + (r + c) % 3 // 2) for r in range(2048) for c in range(16)] + [(2048 * 3 + 5, 1650, 1)] * one_more
    m = quick(lens, 1_700, 14, True, runs)
    return behind_empty_row_blocks(m, 2048, 100), dict(rows_per_block=2048, cols_per_block=100, hash_shift=0), not one_more


WHOLE["32,768 segments"] = by_type(lambda: full_row_block(0))
WHOLE["32,769 segments"] = by_type(lambda: full_row_block(1))

# Segments longer than a tile of 4096 nonzeros, up to the widest block, that begin at a tile's first nonzero, next to it, and at its last.
def long_segments(C):
    rng = np.random.default_rng(17)
    R, n_cols, lengths = 512, 2 * C, [n for n in (4096, 4097, 5000, 8191, 8192, 12_289, 16_384, 16_385, 32_768) if n <= C]
    lens = rng.poisson(3, 140 * R)
    long = []
    for i, n in enumerate(lengths):       # in different row blocks, behind a row as long as it takes
        m, r = quick(lens, n_cols, 18, True, long), (7 * i + 2) * R + 5
        before = int(m.ptr[r] - m.ptr[r - 1])
        long += [(r - 1, 7, before + ((0, 1, 4095)[i % 3] - int(m.ptr[r])) % 4096), (r, (i % 2) * C + (C - n) // 2, n)]
    m = quick(lens, n_cols, 18, True, long)
    assert [int(m.ptr[r]) % 4096 for r, _, _ in long[1::2]] == [(0, 1, 4095)[i % 3] for i in range(len(lengths))]
    return behind_empty_row_blocks(m, R, C), dict(rows_per_block=R, cols_per_block=C, hash_shift=0), True


WHOLE["segments longer than a tile, up to 16,384"] = by_type(lambda: long_segments(16_384))
WIDE = by_type(lambda: long_segments(32_768))  # (fp32 only)


# Row blocks that hold nothing between others (all of 64 that a wavefront deals out, every second, all but every eighth; the first and the last) and some of two, three
# and four shares among them, in either type: each is taken once, whole.
def lists(some, heavy):
    R, rng = 512, np.random.default_rng(11)
    lens = np.zeros((2200, R), dtype=np.int64)
    lens[some] = rng.poisson(5, lens[some].shape)
    if heavy:
        lens[some.start] = heavy
        lens[some.stop - 1 - (some.stop - 1 - some.start) % (some.step or 1)] = heavy
    return quick(lens.ravel()[:2200 * R - 7], 1_800, 12, True), dict(rows_per_block=R, cols_per_block=600, hash_shift=0), True


for _some in (slice(0, 300), slice(70, 199), slice(0, 300, 2), slice(3, 1100, 8), slice(2063, 2200)):
    for _heavy in (0, 60, 100, 127):
        WHOLE["row blocks %s:%s:%s, rows of %d" % (_some.start, _some.stop, _some.step or 1, _heavy)] = by_type(lambda p=(_some, _heavy): lists(*p))


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("case", WHOLE)
def test_row_blocks_as_a_whole(H, oracle, case, f64):
    m, params, _ = WHOLE[case](f64)
    check_against_oracle(H, oracle, m, check_add_sign=False, rounds_per_batch=4, **params)


def test_segments_as_long_as_a_block_is_wide(H, oracle):
    m, params, _ = WIDE(False)
    check_against_oracle(H, oracle, m, check_add_sign=False, rounds_per_batch=4, **params)


# Block columns up to which the schedule keeps their ranks in LDS, and one more; with row blocks cut into combine units.
@pytest.mark.parametrize("n_cols", [2048, 2049])
@pytest.mark.parametrize("unit_slots", [0, 64])
def test_block_columns_kept_and_not(H, oracle, n_cols, unit_slots):
    lens = np.random.default_rng(4).integers(0, 60, 300)
    check_against_oracle(H, oracle, matrix(lens, n_cols), rows_per_block=128, cols_per_block=1, num_workers=7, column_weight=50,
                         combine_unit_slots=unit_slots)


# Short segments in blocks too small for a workgroup (fewer than 256 slots on average): groups filled row block by row block, with and without groups
# that are cut, in more and fewer workgroups than go to one XCD in a row (128 of four groups, on eight of them); and the same in the layout's order, as the first four
# are too small.
BY_TURNS = [(3_000, 64, 50, 1_000, 4), (3_000, 64, 50, 51, 4), (40_000, 64, 100, 1_500, 4), (66_000, 16, 600, 1_200, 4),
            (6_400, 64, 100, 4_000, 154), (250_000, 64, 100, 1_500, 4), (240_000, 16, 600, 1_200, 4)]


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n_rows,R,C,n_cols,mean", BY_TURNS)
def test_groups_filled_row_block_by_row_block(H, oracle, n_rows, R, C, n_cols, mean, f64):
    lens = np.random.default_rng(n_rows).poisson(mean, n_rows)
    lens[::7] = 0
    for long in ([], [(n_rows // 2, 0, min(n_cols, 700))]):
        check_against_oracle(H, oracle, quick(lens, n_cols, 3, f64, long), check_add_sign=False, rows_per_block=R, cols_per_block=C, rounds_per_batch=4)

