"""A build whose scratch memory does not hold the list of segments goes without it (the noting runtime of test_launches.py, CPU)."""
import pytest

from test_launches import run  # noqa: F401  (a fixture)


@pytest.mark.parametrize("n_rows,n_cols,R,C,nnz,S,G,B", [
    (1 << 20, 30_000, 512, 30_000, 64_000_000, 1 << 20, 1 << 14, 1 << 11),       # long segments
    (1 << 20, 300_000, 2048, 30_000, 16_000_000, 8_000_000, 130_000, 5_120),     # short ones
])
def test_builds_without_the_list_where_memory_is_short(run, n_rows, n_cols, R, C, nnz, S, G, B):  # noqa: F811
    got = run(f"""
        def first_passes():
            return [k for k in noted()[0] if "k_segments" in k or "k_place" in k or "k_panel" in k]
        rt.live_bytes.restype = ctypes.c_size_t
        args = (False, {n_rows}, {n_cols}, {R}, {C}, {nnz}, {S}, {G}, {B}, [0] * 2, 100)
        rt.set_capacity(1 << 34)
        h = build(*args)
        with_list, most = first_passes(), rt.live_bytes()
        assert lib.hbp_free(h) == 0 and lib.hbp_release_workspace() == 0 and rt.live_bytes() == 0
        rt.set_capacity(most - 1)
        for wait, words in enumerate([[0, {nnz}], [{S}, {G}, {B}, 0, 4, 0, 0], [0, {nnz}], [100, 0, 0, 0], [100, 0, 0, 0], [100, 0, 0, 0]]):
            for i, w in enumerate(words):
                rt.set_word(wait, i, w)
        # (the build waits for nnz, for the totals, once more when it starts again, and for the totals again)
        p = H.hbp_params_t()
        assert lib.hbp_default_params(ctypes.byref(p)) == 0
        p.rows_per_block, p.cols_per_block, p.rounds_per_batch, p.hash_shift = {R}, {C}, 4, 4
        rt.set_word(3, 0, {S}); rt.set_word(3, 1, {G}); rt.set_word(3, 2, {B}); rt.set_word(3, 3, 0); rt.set_word(3, 4, 4)
        rt.begin()
        h = ctypes.c_void_p()
        rc = lib.hbp_build(word, word, word, {n_rows}, {n_cols}, ctypes.byref(p), None, ctypes.byref(h))
        without, live = first_passes(), rt.live_bytes()
        if rc == 0:
            assert lib.hbp_free(h) == 0
        assert lib.hbp_release_workspace() == 0
        print((rc, with_list, without, most - live, rt.live_bytes()))
    """)
    rc, with_list, without, saved, left = got
    assert rc == 0 and left == 0
    assert saved >= 4 * nnz
    assert any("PassE1" in k or "PassE2" in k for k in with_list) and any("k_place" in k or "k_panel" in k for k in with_list)
    tail = without[-2:]  # what the second attempt ran
    assert "PassE0" in tail[0] and "PassE3" in tail[1]
