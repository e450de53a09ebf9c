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


# Segments per tile: 4096 nonzeros of segments of `run`, i.e. 1, 2, 4 and 8 wavefronts to a tile in the second pass; the last tile is short.
@pytest.mark.parametrize("run", [17, 16, 15, 8, 7, 4, 3, 1])
@pytest.mark.parametrize("R,C", [(512, 1000), (700, 1024), (64, 128)])
def test_wavefronts_to_a_tile(H, oracle, run, R, C):
    m = matrix(np.full(700, 51), 51 * 40, run=run)
    check_against_oracle(H, oracle, m, rows_per_block=R, cols_per_block=C)


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
    for r, c0, n in long:
        keys = np.concatenate([keys[keys // n_cols != r], r * n_cols + np.arange(c0, c0 + n)])
    keys = np.unique(keys)
    ptr = np.searchsorted(keys, np.arange(lens.size + 1) * n_cols).astype(np.int32)
    dt = np.float64 if f64 else np.float32
    return CsrMatrix("row blocks", lens.size, n_cols, ptr, (keys % n_cols).astype(np.int32), rng.standard_normal(keys.size).astype(dt),
                     rng.uniform(-1, 1, n_cols).astype(dt))


# Row blocks as a whole: 128 and more of them, rows short in every block column, blocks of 256 slots on average.  One to 64 block columns, block
# sizes that are no powers of two, ragged last blocks, row blocks without a nonzero and tiles over several row blocks, every shift that fits and one that does
# not (which goes the other way, like 64 block columns at a = 1).
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("R,n_rows,C,n_cols,mean,shift", [
    (512, 512 * 127 + 1, 900, 900, 3, -1), (512, 512 * 127, 900, 900, 3, -1),
    (512, 66_000, 300, 599, 6, 0), (700, 90_001, 500, 2_500, 9, 1), (512, 66_000, 64, 4_096, 62, 0), (512, 66_000, 64, 4_096, 62, 1),
    (1000, 130_000, 333, 1_000, 6, 2), (2048, 270_000, 700, 4_000, 9, 3), (2048, 270_000, 700, 4_000, 9, -1), (2047, 262_016, 32, 64, 5, 6),
])
def test_row_blocks_as_a_whole(H, oracle, R, n_rows, C, n_cols, mean, shift, f64):
    rng = np.random.default_rng(R + n_cols)
    lens = rng.poisson(mean, n_rows)
    lens[R * 5:R * 7] = 0
    lens[R * 20 + 3:R * 20 + 40] = 0
    m = quick(lens, n_cols, 5, f64)
    check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=R, cols_per_block=C, rounds_per_batch=4, hash_shift=shift)


# Row blocks in one and several shares (an fp32 share holds 27,306 nonzeros, an fp64 one 16,384), groups that lie in two of them, rows
# of up to a block's width, alone and 70 in a row, with tails of one and several pieces of 64 rounds, and more rounds than the list of tails holds.
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("long", [
    [(9, 0, 63), (70, 5, 64), (90, 600, 65), (2100, 0, 96), (2200, 0, 97), (4200, 7, 576), (5000, 7, 577)],
    [(r, 10 * (r % 50), 1500) for r in range(100, 170)], [(300, 0, 3000), (301, 0, 3000), (302, 0, 2999), (303, 1, 1)],
    [(r, 0, 700) for r in range(600, 650)],       # more nonzeros than a row block may have: the other way
])
@pytest.mark.parametrize("mean", [6, 13])
def test_shares_of_row_blocks(H, oracle, long, mean, f64):
    lens = np.random.default_rng(mean).poisson(mean, 262_145)
    m = quick(lens, 3_000, 6, f64, long)
    for R in (2048, 1024):
        check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=R, cols_per_block=600, rounds_per_batch=4)


@pytest.mark.parametrize("f64", [False, True])
def test_more_rounds_than_the_list_of_tails_holds(H, oracle, f64):
    """Five groups of each of five blocks with a row of 600 nonzeros among rows of 15: 14,800 rounds behind the first eight, the list holds 12,288."""
    lens = np.random.default_rng(8).poisson(6, 262_145)
    lens[:300] = 75
    m = quick(lens, 3_000, 9, f64, [(r, 0, 3_000) for r in (10, 70, 130, 190, 250)])
    check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=2048, cols_per_block=600, rounds_per_batch=4, hash_shift=0)


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


# Row blocks that hold nothing between others (all of 64 that a wavefront deals out, every second, all but every eighth; the first and the last) and some of two, three
# and four shares among them, in either type: each is taken once, whole.
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("some", [slice(0, 300), slice(70, 199), slice(0, 300, 2), slice(3, 1100, 8), slice(1163, 1300)])
@pytest.mark.parametrize("heavy", [0, 60, 100, 127])
def test_lists_of_row_blocks(H, oracle, some, heavy, f64):
    R, rng = 512, np.random.default_rng(11)
    lens = np.zeros((1300, R), dtype=np.int64)
    lens[some] = rng.poisson(5, lens[some].shape)
    if heavy:
        lens[some.start] = heavy
        lens[some.stop - 1 - (some.stop - 1 - some.start) % (some.step or 1)] = heavy
    m = quick(lens.ravel()[:1300 * R - 7], 1_800, 12, f64)
    check_against_oracle(H, oracle, m, check_add_sign=False, rows_per_block=R, cols_per_block=600, rounds_per_batch=4, hash_shift=0)
