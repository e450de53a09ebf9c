"""Which kernels a build and a product launch, and how much memory they take, for sizes that no matrix has to be made for:
the library on the CPU with the HIP runtime of test_memory_of_freed_handles.py in front of the real one, which here also
notes kernels by name and hands the build scripted totals where it reads them back from the device."""
import ast
import os
import subprocess
import sys
import textwrap

import pytest

from test_memory_of_freed_handles import ROOT, RUNTIME

NOTES = r"""
#undef hipMalloc
#undef hipHostMalloc
#undef hipStreamSynchronize
#undef hipLaunchKernel
static struct { const void *f; const char *name; } kernels[kMax];
static int n_kernels, n_launched, n_allocated, n_waits;
static const char *launched[kMax];
static unsigned pushed, grids[kMax];
static size_t allocated[kMax];
static unsigned *readback, script[8][16];
void __hipRegisterFunction(void **module, const void *f, char *device_f, const char *name, unsigned limit, void *a, void *b, void *c, void *d, int *e)
{
    (void)module; (void)device_f; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (n_kernels == kMax) abort();
    kernels[n_kernels].f = f;
    kernels[n_kernels++].name = name;
}
unsigned __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t lds, void *s) { (void)b; (void)lds; (void)s; pushed = g.x; return 0; }
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *lds, void **s) { *g = *b = (dim3_){1, 1, 1}; g->x = pushed; *lds = 0; *s = 0; return 0; }
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **args, size_t lds, void *s)
{
    (void)b; (void)args; (void)lds; (void)s;
    int i = 0;
    while (i < n_kernels && kernels[i].f != f) i++;
    if (i == n_kernels || n_launched == kMax) abort();
    grids[n_launched] = g.x;
    launched[n_launched++] = kernels[i].name;
    return 0;
}
int hipMalloc(void **out, size_t bytes)
{
    if (n_allocated == kMax) abort();
    allocated[n_allocated++] = bytes;
    return quiet_hipMalloc(out, bytes);
}
int hipHostMalloc(void **out, size_t bytes, unsigned flags)
{
    const int rc = quiet_hipHostMalloc(out, bytes, flags);
    readback = *out;
    return rc;
}
int hipStreamSynchronize(void *s)
{
    (void)s;
    if (readback && n_waits < 8) memcpy(readback, script[n_waits], sizeof script[0]);
    n_waits++;
    return 0;
}
void begin(void) { n_launched = n_allocated = n_waits = 0; }
void set_word(int wait, int i, unsigned value) { script[wait][i] = value; }
int launches(void) { return n_launched; }
const char *launch(int i) { return launched[i]; }
unsigned grid(int i) { return grids[i]; }
int allocations(void) { return n_allocated; }
size_t allocation(int i) { return allocated[i]; }
"""

PROGRAM = r"""
import ctypes, json, sys
import paper_2504_08860_amd as H
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # in front of the real runtime for what it defines
lib = ctypes.CDLL(sys.argv[2])
rt.launch.restype = ctypes.c_char_p
rt.allocation.restype = ctypes.c_size_t
rt.set_capacity.argtypes = [ctypes.c_size_t]
for f in (lib.hbp_build, lib.hbp_build_f64):
    f.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int64] * 2 + [ctypes.c_void_p] * 3
for f in (lib.hbp_spmv, lib.hbp_spmv_f64):
    f.argtypes = [ctypes.c_void_p] * 4
lib.hbp_free.argtypes = [ctypes.c_void_p]
word = ctypes.create_string_buffer(64)

def noted():
    return [rt.launch(i).decode() for i in range(rt.launches())], [rt.allocation(i) for i in range(rt.allocations())]

def grids():
    return {rt.launch(i).decode(): rt.grid(i) for i in range(rt.launches())}

def build(f64, n_rows, n_cols, R, C, nnz, S, G, B, counts, U, a=4):
    # (given block parameters: no sampling pass; a given shift: no sampled one; given rounds: workers)
    p = H.hbp_params_t()
    assert lib.hbp_default_params(ctypes.byref(p)) == 0
    p.rows_per_block, p.cols_per_block, p.rounds_per_batch, p.hash_shift = R, C, 4, a
    for wait, words in enumerate([[0, nnz], [S, G, B, 0, a, *counts], [U, 0, 0, 0]]):
        for i, w in enumerate(words):
            rt.set_word(wait, i, w)
    rt.begin()
    h = ctypes.c_void_p()
    rc = (lib.hbp_build_f64 if f64 else lib.hbp_build)(word, word, word, n_rows, n_cols, ctypes.byref(p), None, ctypes.byref(h))
    assert rc == 0, rc
    return h

def product(f64, h):
    rt.begin()
    rc = (lib.hbp_spmv_f64 if f64 else lib.hbp_spmv)(h, word, word, None)
    assert rc == 0, rc
    return noted()[0]
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    """Runs a program against the noting runtime; returns the value that it prints."""
    import paper_2504_08860_amd as H
    if not os.path.exists(H.LIB_PATH):
        from paper_2504_08860_amd.build import build_library
        build_library()
    at = tmp_path_factory.mktemp("launches")
    source, runtime = at / "runtime.c", at / "runtime.so"
    source.write_text("".join(f"#define {f} quiet_{f}\n" for f in ("hipMalloc", "hipHostMalloc", "hipStreamSynchronize", "hipLaunchKernel"))
                      + RUNTIME + NOTES)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", str(source), "-o", str(runtime)])

    def program(body):
        text = at / "program.py"
        text.write_text(PROGRAM + textwrap.dedent(body))
        res = subprocess.run([sys.executable, str(text), str(runtime), H.LIB_PATH], capture_output=True, text=True, cwd=ROOT, timeout=120,
                             env=dict(os.environ, PYTHONPATH=ROOT))
        assert res.returncode == 0, res.stdout + res.stderr
        return ast.literal_eval(res.stdout)
    return program


# rows per block, units and the combine part's wavefronts per unit: on a compute unit fit as many units as their copies of the
# slice and 1024 bytes, in steps of 1280, let into 160 KB, and as their wavefronts let into 32 (in comments: of four and of three wavefronts)
COMBINE = {
    False: [(2048, [(256, 16), (257, 8), (512, 8), (513, 4), (1024, 4), (1025, 3), (1536, 3), (1537, 4)]),   # 4 and 6 units
            (1025, [(2048, 4), (2049, 4), (2304, 4), (2305, 3), (2560, 3), (2561, 4)]),                      # 8 (LDS: 9) and 10 (LDS: 11)
            (1200, [(2048, 4), (2049, 3), (2304, 3), (2305, 4)]),                                            # 8 and 9
            (8192, [(256, 4), (257, 4)])],                                                                   # 1 and 1
    True: [(2048, [(256, 8), (257, 4), (512, 4), (513, 3), (768, 3), (769, 4)]),                             # 2 and 3
           (1037, [(1024, 4), (1025, 3), (1536, 3), (1537, 4)]),                                             # 4 and 6
           (4096, [(256, 4), (257, 4)])],                                                                    # 1 and 1
}


@pytest.mark.parametrize("f64", [False, True])
def test_wavefronts_of_the_combine_part(run, f64):
    got = run(f"""
        out = []
        for R, units in {[(R, [u for u, _ in units]) for R, units in COMBINE[f64]]}:
            for U in units:
                for slots in (127, 128):                  # on average, per block: short chunks below 128, longer ones from there on
                    h = build({f64}, R * U, 1000, R, 1000, 1000 * U, slots * U, 3 * U, U, [0] * 2, U)
                    out.append((R, U, slots, [k for k in product({f64}, h) if "k_combine" in k]))
                    assert lib.hbp_free(h) == 0
                    assert lib.hbp_release_workspace() == 0
        print(out)
    """)
    want = []
    for R, units in COMBINE[f64]:
        for U, wavefronts in units:
            for slots in (127, 128):
                want.append((R, U, slots, "k_combineILi%dE%sLi%dELi%dE" % (64 * wavefronts, "d" if f64 else "f", *((8, 2) if slots == 127 else (4, 4)))))
    assert len(got) == len(want)
    wrong = [(g, w) for g, w in zip(got, want) if g[:3] != w[:3] or len(g[3]) != 1 or w[3] not in g[3][0]]
    assert not wrong, wrong


# rows, nonzeros, longest row, whether a tile showed a long segment, whether groups are cut
CUT = [
    (1 << 20, 16_000_000, 513, True, True),          # rows from 513 nonzeros on
    (1 << 20, 16_000_000, 512, True, False),
    (1 << 20, 16_000_000, 5000, True, True),
    (1 << 20, 16_000_000, 5000, False, False),       # long rows in short segments
    (10_000, 6_000_000, 4800, True, False),          # more than eight times the average
    (10_000, 6_000_000, 4801, True, True),
    (1, 9000, 9000, True, False),
]


def test_groups_cut_where_segments_are_long(run):
    got = run(f"""
        out = []
        for n_rows, nnz, longest, segments, _ in {CUT}:
            h = build(False, n_rows, 30000, 512, 30000, nnz, n_rows, (n_rows + 63) // 64, (n_rows + 511) // 512, [longest, int(segments)], 100)
            out.append([k for k in noted()[0] if "k_fill" in k or "k_list_rest" in k])
            assert lib.hbp_free(h) == 0
            assert lib.hbp_release_workspace() == 0
        print(out)
    """)
    for case, kernels in zip(CUT, got, strict=True):
        want = ["k_fill_flatILb1Ef", "k_list_rest", "k_fill_restIf"] if case[4] else ["k_fill_flatILb0Ef"]
        assert len(kernels) == len(want) and all(w in k for w, k in zip(want, kernels)), (case, kernels)


def test_scratch_memory_for_groups_that_are_cut(run):
    """The list of their parts, 8 bytes per 128 nonzeros, is in the fourth allocation of builds that cut, and of no others."""
    got = run("""
        out = []
        for nnz, longest in ((16_000_000, 512), (64_000_000, 512), (16_000_000, 513), (64_000_000, 513)):
            rt.set_capacity(1 << 32)
            h = build(False, 1 << 20, 30000, 512, 30000, nnz, 1 << 20, 1 << 14, 1 << 11, [longest, 1], 100)
            out.append(noted()[1])
            assert lib.hbp_free(h) == 0
            assert lib.hbp_release_workspace() == 0
        print(out)
    """)
    assert [len(sizes) for sizes in got] == [4] * 4
    small, large, small_cut, large_cut = (sizes[3] for sizes in got)
    assert small == large
    for size, nnz in ((small_cut, 16_000_000), (large_cut, 64_000_000)):
        assert 0 <= size - small - nnz // 16 <= nnz // 16 // 8 + 1024   # (an eighth more is taken than needed, in steps of 256)


def test_what_tiles_show_of_long_segments(tmp_path):
    """A segment of 513 nonzeros shows in a tile wherever it begins and its matrix ends; segments of up to 192 never do."""
    source, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    source.write_text(r"""
#include <cstdio>
#include <vector>
#include "hbp_internal.h"
static bool shown(const std::vector<char> &starts)   // starts[j]: a segment starts at nonzero j
{
    const size_t n = starts.size();
    for (size_t j0 = 0; j0 < n; j0 += 4096) {
        uint64_t words = 0;
        for (size_t j = j0; j < n && j < j0 + 4096; j++) words |= (uint64_t)(starts[j] != 0) << ((j - j0) / 64);
        if (hbp::shows_long_segment(words, (int32_t)(n - j0 < 4096 ? n - j0 : 4096))) return true;
    }
    return false;
}
int main()
{
    for (size_t at = 0; at < 4200; at++)
        for (size_t behind : {0, 1, 63, 700}) {
            std::vector<char> starts(at + 513 + behind, 1);
            for (size_t j = at + 1; j < at + 513; j++) starts[j] = 0;
            if (!shown(starts)) { std::printf("513 from %zu, %zu behind\n", at, behind); return 1; }
        }
    for (size_t length : {1, 64, 191, 192})
        for (size_t at = 0; at < length; at++)
            for (size_t n : {size_t(100), size_t(4096), size_t(8192), size_t(9001)}) {
                std::vector<char> starts(n, 0);
                for (size_t j = at; j < n; j += length) starts[j] = 1;
                starts[0] = 1;
                if (shown(starts)) { std::printf("%zu from %zu of %zu\n", length, at, n); return 1; }
            }
    return 0;
}
""")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2504_08860_amd", "csrc"), str(source), "-o", str(exe)])
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
