"""Which kernels a build takes, and in what grids (the noting runtime of test_launches.py, CPU)."""
import numpy as np
import pytest

from test_gpu_build_passes import BY_TURNS, RUNS, WHOLE, WIDE, quick, runs, totals
from test_launches import run  # noqa: F401  (a fixture)


@pytest.mark.parametrize("f64", [False, True])
def test_few_workgroups_for_row_blocks_and_shares_that_are_not_there(run, f64):  # noqa: F811
    """2000 row blocks (the first cases 20,000, most of them empty; one of 60,000 nonzeros among light ones): a list, 4 bytes an entry, and no workgroup without work, where more than
    an eighth of the workgroups would have none."""
    room, most = 160 * 1024 // (10 if f64 else 6), 4 if f64 else 3
    # row blocks, full ones, most nonzeros, shares, of the XCD with most; entries of the lists, grids of the places' and the fill's kernel
    cases = [(20_000, 600, 60_000, 600 + most - 1, 78), (20_000, 600, 10_000, 600, 76),
             (2000, 2000, room, 2000, 250), (2000, 1750, room, 1750, 219), (2000, 1749, room, 1749, 219),
             (2000, 2000, 2 * room, 4000, 500), (2000, 2000, 2 * room, 3500, 438), (2000, 2000, 2 * room, 3499, 438)]
    want = [(600 + 8 * 78, 600, 8 * 78), (600 + 8 * 76, 600, 8 * 76),
            (0, 2000, 2000), (0, 2000, 2000), (1749 + 8 * 219, 1749, 8 * 219),
            (0, 2000, 4000), (0, 2000, 4000), (8 * 438, 2000, 8 * 438)]
    got = run(f"""
        out = []
        for NBR, there, most, shares, xcd in {cases}:
            h = build({f64}, NBR * 2048, 300_000, 2048, {15_000 if f64 else 30_000}, 30_000_000, 20_000_000, 400_000, 40_000, [0, 0, 30_000, most, there, xcd, shares], 100, a=0)
            seen = grids()
            out.append((noted()[1][3], *(next(grid for name, grid in seen.items() if k in name) for k in ("k_panel_slots", "k_panel_fill"))))
            assert lib.hbp_free(h) == 0 and lib.hbp_release_workspace() == 0
        print(out)
    """)
    none = {2000: got[2][0], 20_000: None}
    for (NBR, *_), (entries, *kernels), (size, *launched) in zip(cases, want, got, strict=True):
        assert launched == kernels
        if none[NBR] is not None:                       # (an eighth more is taken than needed, in steps of 256)
            assert 4 * entries <= size - none[NBR] <= 9 * 4 * entries // 8 + 1024


@pytest.mark.parametrize("f64", [False, True])
def test_groups_row_block_by_row_block_from_six_megabytes_on(run, f64):  # noqa: F811
    """A launch more, and the list of the groups' order, only where the CSR arrays are larger than an XCD's L2."""
    least = -(-(6 << 20) // (12 if f64 else 8))
    got = run(f"""
        out = []
        for nnz in ({least} - 1, {least}):
            h = build({f64}, 100_000, 100_000, 512, 10_000, nnz, nnz // 3, 6_000, 2_000, [0, 0], 100)
            out.append([k for k in ("k_group_turns", "k_fill_flat") if any(k in name for name in noted()[0])])
            assert lib.hbp_free(h) == 0
        print(out)
    """)
    assert got == [["k_fill_flat"], ["k_group_turns", "k_fill_flat"]]


# Row blocks, those that hold something, nonzeros, and the segments from which on they are taken as a whole where rows are short: segments and 8-byte words of the CSR arrays, 3.5
# million for the first turn of 256 row blocks and 4.5 for each other, in proportion to the row blocks that hold something.
@pytest.mark.parametrize("f64,NBR,there,nnz,least", [
    (False, 256, 256, 1_800_000, 1_700_000), (False, 257, 257, 4_200_000, 3_800_000), (False, 600, 600, 7_000_000, 5_500_000), (False, 2000, 2000, 18_000_000, 17_000_000),
    (True, 256, 256, 1_400_000, 1_400_000), (True, 600, 600, 5_000_000, 5_000_000), (False, 2000, 500, 1_450_000, 550_000), (True, 300, 200, 800_000, 1_133_334),
])
def test_work_that_row_blocks_as_a_whole_are_worth(run, f64, NBR, there, nnz, least):  # noqa: F811
    got = run(f"""
        out = []
        for S, longest, shown in (({least} - 1, 0, 0), ({least}, 0, 0), ({nnz} // 3, 1024, 1), ({nnz} // 3, 1025, 1), ({nnz} // 3, 1025, 0)):
            h = build({f64}, {NBR} * 2048, 300_000, 2048, {15_000 if f64 else 30_000}, {nnz}, S, S // 60, S // 300, [longest, shown, 30_000, 60_000, {there}, 99, 700], 100, a=0)
            out.append(any("k_panel" in name for name in noted()[0]))
            assert lib.hbp_free(h) == 0
        print(out)
    """)
    assert got == [False, True, False, True, False]


def test_more_row_blocks_than_a_grid_has_workgroups(run):  # noqa: F811
    """A grid has fewer than 2^32 threads, 4,194,303 workgroups of 1024: beyond, block by block (also where a long row would be waited for)."""
    got = run("""
        rt.set_capacity(1 << 37)
        out = []
        for NBR, most in ((4_194_296, 600), (4_194_304, 600), (2_097_144, 27_307), (2_097_152, 27_307)):
            h = build(False, NBR * 256, 30_000, 256, 30_000, 3 * NBR * 128, NBR * 256, NBR * 4, NBR, [2000, 1, 256, most, NBR, NBR, 8 * NBR], 100, a=0)
            out.append((any("k_panel" in name for name in noted()[0]), max(grid for name, grid in grids().items() if any(k in name for k in ("k_panel", "k_place", "k_fill")))))
            assert lib.hbp_free(h) == 0 and lib.hbp_release_workspace() == 0
        print(out)
    """)
    assert [panel for panel, _ in got] == [True, False, True, False]
    assert all(grid * 1024 < 2**32 for panel, grid in got if panel)


def test_matrices_that_go_by_row_blocks_as_a_whole(run, oracle):  # noqa: F811
    """The matrices of test_gpu_build_passes.py go the way that they are meant to."""
    asked, wanted = [], []
    for name, make in [*WHOLE.items(), ("segments as long as a block is wide", WIDE)]:
        m, params, whole = make(True)
        R, C, shift = params["rows_per_block"], params["cols_per_block"], params["hash_shift"] if "hash_shift" in params else -1
        t = totals(m, R, C)
        a = shift if shift >= 0 else oracle.sample_shift(m.ptr, m.col, m.n_rows, C)
        for f64 in (False, True) if make is not WIDE else (False,):
            asked.append((f64, m.n_rows, m.n_cols, R, C, m.nnz, t["S"], t["G"], t["B"], [t["longest"], t["long"], t["most_slots"], t["most_nonzeros"], t["row_blocks"], 9999], 100, a))
            wanted.append((name, f64, ["k_panel_fill", "k_panel_slots"] if whole else ["k_fill", "k_place"]))
    got = run(f"""
        rt.set_capacity(1 << 36)
        out = []
        for args in {asked}:
            h = build(*args)
            out.append(sorted(k for k in ("k_panel_slots", "k_panel_fill", "k_place", "k_fill", "k_fill_flat") if any(k + "I" in name or k + "E" in name for name in noted()[0])))
            assert lib.hbp_free(h) == 0
        print(out)
    """)
    wrong = [(case, kernels) for case, kernels in zip(wanted, got, strict=True) if case[2] != kernels]
    assert not wrong, wrong


def test_wavefronts_to_a_tile_of_runs(run):  # noqa: F811
    """Those that test_gpu_build_passes.py says: by the grid of k_place, and with all of a workgroup by its template."""
    asked = []
    for length in RUNS:
        m = runs(length, False)
        for R in (512, 700, 64):
            t = totals(m, R, length)
            asked.append((False, m.n_rows, m.n_cols, R, length, m.nnz, t["S"], t["G"], t["B"], [0, 0, t["most_slots"], t["most_nonzeros"]], 100, 4))
    got = run(f"""
        out = []
        for args in {asked}:
            h = build(*args)
            out.append([(name, grid) for name, grid in grids().items() if "k_place" in name])
            assert lib.hbp_free(h) == 0
        print(out)
    """)
    want = [n for n in RUNS.values() for _ in range(3)]
    for n, kernels in zip(want, got, strict=True):
        (name, grid), = kernels
        assert grid == -(-9 * n // 8) and f"k_placeILb{int(n == 8)}E" in name


def test_matrices_whose_groups_go_row_block_by_row_block(run):  # noqa: F811
    asked, want = [], []
    for n_rows, R, C, n_cols, mean in BY_TURNS:
        lens = np.random.default_rng(n_rows).poisson(mean, n_rows)
        lens[::7] = 0
        m = quick(lens, n_cols, 3, True)
        t = totals(m, R, C)
        for f64 in (False, True):
            asked.append((f64, n_rows, n_cols, R, C, m.nnz, t["S"], t["G"], t["B"], [0, 0, t["most_slots"], t["most_nonzeros"]], 100))
            want.append(n_rows in (6_400, 240_000, 250_000))
    got = run(f"""
        out = []
        for args in {asked}:
            h = build(*args)
            out.append(any("k_group_turns" in name for name in noted()[0]))
            assert lib.hbp_free(h) == 0
        print(out)
    """)
    assert got == want
