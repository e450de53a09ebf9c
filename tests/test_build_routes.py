"""Which kernels a build takes, and in what grids (the noting runtime of test_launches.py, CPU)."""
import pytest

from test_launches import run  # noqa: F401  (a fixture)


@pytest.mark.parametrize("f64", [False, True])
def test_no_workgroups_for_row_blocks_and_shares_that_are_not_there(run, f64):  # noqa: F811
    """20,000 row blocks, 600 of which hold something, one of them 60,000 nonzeros: as many workgroups as the device counts row blocks, and as shares for the XCD with most."""
    got = run(f"""
        h = build({f64}, 20_000 * 2048, 300_000, 2048, {15_000 if f64 else 30_000}, 10_000_000, 7_000_000, 120_000, 10_000, [0, 0, 30_000, 60_000, 600, 76], 100, a=0)
        print(sorted((next(k for k in ("k_panel_slots", "k_panel_fill") if k in name), grid) for name, grid in grids().items() if "k_panel" in name))
        assert lib.hbp_free(h) == 0
    """)
    assert got == [("k_panel_fill", 8 * 76), ("k_panel_slots", 600)]


@pytest.mark.parametrize("f64", [False, True])
def test_no_lists_of_all_row_blocks_in_one_share_each(run, f64):  # noqa: F811
    """The lists, 4 bytes a row block, are there where a row block is empty or in two shares."""
    room = 160 * 1024 // (10 if f64 else 6)
    got = run(f"""
        out = []
        for most, there, xcd in (({room}, 2000, 250), ({room}, 1999, 250), ({room} + 1, 2000, 500)):
            h = build({f64}, 2000 * 2048, 300_000, 2048, {15_000 if f64 else 30_000}, 30_000_000, 20_000_000, 400_000, 40_000, [0, 0, 15_000, most, there, xcd], 100, a=0)
            out.append((noted()[1][3], sorted(grid for name, grid in grids().items() if "k_panel" in name)))
            assert lib.hbp_free(h) == 0 and lib.hbp_release_workspace() == 0
        print(out)
    """)
    (none, a), (both, b), (shares, c) = got
    assert (a, b, c) == ([2000, 2000], [1999, 2000], [2000, 4000])
    for more, size in ((4 * 1999 + 32 * 250, both - none), (32 * 500, shares - none)):
        assert more <= size <= 9 * more // 8 + 1024   # (an eighth more is taken than needed, in steps of 256)


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
