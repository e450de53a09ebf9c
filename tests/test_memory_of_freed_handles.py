"""What becomes of a handle's device memory, with a HIP runtime of the test's own in front of the real one: device
memory is host memory of a stated capacity, kernels do nothing (so every matrix is an empty one) and a wait can be
made to fail.  Runs on the CPU, in a process of its own."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stdlib.h>
#include <string.h>
#include <stddef.h>
enum { kMax = 4096 };
static void *at[kMax];
static size_t size_of[kMax], live, capacity = (size_t)1 << 30;
static int frees, refuse_waits;
void set_capacity(size_t bytes) { capacity = bytes; }
void set_refuse_waits(int yes) { refuse_waits = yes; }
size_t live_bytes(void) { return live; }
int free_calls(void) { return frees; }
int hipMalloc(void **out, size_t bytes)
{
    if (live + bytes > capacity) return 2;  /* hipErrorOutOfMemory */
    for (int i = 0; i < kMax; i++)
        if (!at[i]) {
            at[i] = *out = calloc(1, bytes);
            size_of[i] = bytes;
            live += bytes;
            return 0;
        }
    abort();
}
int hipFree(void *p)
{
    for (int i = 0; i < kMax; i++)
        if (p && at[i] == p) {
            live -= size_of[i];
            free(p);
            at[i] = 0;
            frees++;
            return 0;
        }
    return 1;
}
int hipHostMalloc(void **out, size_t bytes, unsigned flags) { (void)flags; *out = calloc(1, bytes); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)s; memset(p, v, n); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipDeviceSynchronize(void) { return refuse_waits ? 900 : 0; }  /* hipErrorStreamCaptureUnsupported */
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
typedef struct { unsigned x, y, z; } dim3_;
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **args, size_t lds, void *s)
{
    (void)f; (void)g; (void)b; (void)args; (void)lds; (void)s;
    return 0;
}
"""

PROGRAM = r"""
import ctypes, sys
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # in front of the real runtime for what it defines
lib = ctypes.CDLL(sys.argv[2])
rt.live_bytes.restype = ctypes.c_size_t
rt.set_capacity.argtypes = [ctypes.c_size_t]
lib.hbp_build.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int64] * 2 + [ctypes.c_void_p] * 3
lib.hbp_free.argtypes = [ctypes.c_void_p]
word = ctypes.create_string_buffer(64)
def build(n_rows, params=None):
    h = ctypes.c_void_p()
    rc = lib.hbp_build(word, word, word, n_rows, 100, params, None, ctypes.byref(h))
    return rc, h
"""


def run(tmp_path, body):
    import paper_2504_08860_amd as H
    if not os.path.exists(H.LIB_PATH):
        from paper_2504_08860_amd.build import build_library
        build_library()
    source, runtime = tmp_path / "runtime.c", tmp_path / "runtime.so"
    source.write_text(RUNTIME)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", str(source), "-o", str(runtime)])
    program = tmp_path / "program.py"
    program.write_text(PROGRAM + textwrap.dedent(body))
    res = subprocess.run([sys.executable, str(program), str(runtime), H.LIB_PATH], capture_output=True, text=True, cwd=ROOT, timeout=120,
                         env=dict(os.environ, PYTHONPATH=ROOT))
    assert res.returncode == 0, res.stdout + res.stderr


def test_memory_is_kept_after_a_wait_and_given_back(tmp_path):
    run(tmp_path, """
        rc, h = build(10**6)
        assert rc == 0
        held = rt.live_bytes()
        assert lib.hbp_free(h) == 0
        assert rt.live_bytes() == held and rt.free_calls() == 0        # kept
        rc, h = build(10**6)
        assert rc == 0 and rt.live_bytes() == held                     # and taken again
        assert lib.hbp_free(h) == 0
        assert lib.hbp_release_workspace() == 0 and rt.live_bytes() == 0
    """)


def test_memory_whose_wait_failed_is_not_handed_out_again(tmp_path):
    run(tmp_path, """
        rc, h = build(10**6)
        assert rc == 0
        before = rt.live_bytes()
        rt.set_refuse_waits(1)
        assert lib.hbp_free(h) == 0
        rt.set_refuse_waits(0)
        assert rt.free_calls() == 2                                    # both of the handle's allocations
        after = rt.live_bytes()
        rc, h = build(10**6)                                           # allocates anew
        assert rc == 0 and rt.live_bytes() == before and after < before
        assert lib.hbp_free(h) == 0
    """)


def test_kept_memory_is_given_up_where_a_build_is_short_of_it(tmp_path):
    run(tmp_path, """
        import paper_2504_08860_amd as H
        given = H.hbp_params_t(512, 64, 64, 0, -1, 0, 0, 0, 8, -1, -1, 0, -1, 0, 1, -1)   # no sampling pass, no scratch memory
        rc, h = build(10**6, ctypes.byref(given))
        assert rc == 0 and lib.hbp_free(h) == 0
        held = rt.live_bytes()
        assert held > 0
        rt.set_capacity(held + 100)                                    # the scratch memory of a build does not fit beside it
        rc, h = build(1000)
        assert rc == 0 and rt.free_calls() == 2
        assert lib.hbp_free(h) == 0
        # nor do a larger handle's own arrays
        assert lib.hbp_release_workspace() == 0
        rt.set_capacity(1 << 30)
        rc, h = build(2 * 10**6, ctypes.byref(given))
        assert rc == 0
        needs = rt.live_bytes()
        assert lib.hbp_free(h) == 0 and lib.hbp_release_workspace() == 0 and rt.live_bytes() == 0
        rt.set_capacity(needs)
        rc, h = build(10**6, ctypes.byref(given))
        assert rc == 0 and lib.hbp_free(h) == 0
        rc, h = build(2 * 10**6, ctypes.byref(given))
        assert rc == 0 and rt.live_bytes() == needs
        assert lib.hbp_free(h) == 0
    """)


def test_a_handle_takes_no_more_than_it_needs(tmp_path):
    """New memory is of the size that is needed; kept memory is taken by handles of about its size only."""
    run(tmp_path, """
        import paper_2504_08860_amd as H
        given = ctypes.byref(H.hbp_params_t(1, 64, 64, 1, -1, 0, 0, 0, 8, -1, -1, 0, -1, 0, 1, -1))
        n = 10**6 + 77777                                              # one row per block: 4 bytes of four arrays per row
        rt.set_capacity(4 * 4 * n + 8 * 1024)
        rc, h = build(n, given)
        assert rc == 0
        held = rt.live_bytes()
        assert lib.hbp_free(h) == 0 and rt.live_bytes() == held
        rt.set_capacity(1 << 30)
        rc, h = build(n - n // 10, given)                              # in the kept memory
        assert rc == 0 and rt.live_bytes() == held
        rc, other = build(n // 2, given)                               # the rest of it gone, beside it
        assert rc == 0 and held < rt.live_bytes() < 1.51 * held
        assert lib.hbp_free(h) == 0 and lib.hbp_free(other) == 0
        held = rt.live_bytes()
        rc, h = build(3 * n // 4, given)                               # kept: one too large, one too small
        assert rc == 0 and rt.live_bytes() > 1.4 * held
        assert lib.hbp_free(h) == 0
    """)
