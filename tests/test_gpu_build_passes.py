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
