"""The scratch memory of a build goes by its segments and blocks, not by its nonzeros (the noting runtime of test_launches.py, CPU)."""
import pytest

from test_launches import run  # noqa: F401  (a fixture)

# rows, columns, R, C, segments, groups, blocks, most slots and nonzeros of a row block, what places the segments and fills the layout
ROUTES = {
    "segments of any length": (1 << 20, 30_000, 512, 30_000, 1 << 20, 1 << 14, 1 << 11, 512, 40_000, ["k_place", "k_fill_flat"]),
    "no list": (1 << 20, 30_000, 2048, 50, 1 << 20, 1 << 18, 1 << 17, 2048, 40_000, ["PassE3", "k_fill_flat"]),
    "short, small blocks": (1 << 20, 600_000, 512, 30_000, 8_000_000, 1_200_000, 40_960, 5_000, 12_000, ["k_place", "k_group_turns", "k_fill_flat"]),
    "short, row blocks": (1 << 20, 300_000, 2048, 30_000, 8_000_000, 130_000, 5_120, 16_000, 40_000, ["k_panel_slots", "k_panel_fill"]),
    "short, no row blocks": (1 << 20, 300_000, 2048, 30_000, 8_000_000, 130_000, 5_120, 40_000, 70_000, ["k_place", "k_fill"]),
}


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("route", ROUTES)
def test_scratch_memory(run, route, f64):  # noqa: F811
    n_rows, n_cols, R, C, S, G, B, most_slots, most_nonzeros, kernels = ROUTES[route]
    C = C // 2 if f64 else C
    short = route.startswith("short")
    sizes = (8_000_000, 31_000_000) if short else (8_000_000, 64_000_000)
    got = run(f"""
        out = []
        for nnz in {sizes}:
            rt.set_capacity(1 << 34)
            h = build({f64}, {n_rows}, {n_cols}, {R}, {C}, nnz, {S}, {G}, {B}, [0, 0, {most_slots}, {most_nonzeros}, 500, 200, 700], 100, a=1)
            out.append(noted())
            assert lib.hbp_free(h) == 0 and lib.hbp_release_workspace() == 0 and rt.live_bytes() == 0
        print(out)
    """)
    NBR, NBC = -(-n_rows // R), -(-n_cols // C)
    D = NBR * NBC
    for nnz, (launched, allocated) in zip(sizes, got):
        wrong = [k for k in kernels if not any(k in name for name in launched)]
        assert not wrong, (wrong, launched)
        assert len(allocated) == 4      # handle, scratch, handle, scratch
        scan = 20 * ((max(D, NBR, nnz // 64 + D) + 1) // 2048 + 2)
        tables = 16 * (D + 1) + 16 * (nnz // 4096 + 1) + 28 * (NBR + 1) + 32 * 200 + 4 * (B + 1) + scan + 16_384
        assert allocated[1] + allocated[3] <= 9 * (tables + 12 * S + 8 * (G + 1)) // 8, (allocated, tables)


def test_room_for_the_starts_of_segments(run):  # noqa: F811
    """They lie where the layout's columns come to be, ten bytes for 64 nonzeros and whole tiles of 4096: no row blocks as a whole below 320 nonzeros."""
    got = run("""
        out = []
        for nnz in (319, 320, 4096, 4097):
            h = build(False, 1 << 18, 300, 2048, 300, nnz, nnz, 1, 1, [0, 0, nnz, nnz], 100, a=0)
            out.append(any("PassE2" in k for k in noted()[0]))
            assert lib.hbp_free(h) == 0
        print(out)
    """)
    assert got == [False, True, True, True]
