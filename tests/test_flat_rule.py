"""Which matrices run without workers (flat_wavefronts): the rule against matrices for which both ways were timed
on an MI355X, as (nonzeros, segments, rows, non-empty rows, block columns, bytes per value, unevenness, faster way)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# unevenness: sum over the rows of length * min(length, 64 mean lengths), over nonzeros times the mean length of a
# non-empty row (lognormal rows 4.2, R-MAT 12 to 14, rows of one length 1)
MEASURED = [
    ("5-point grid 450", 1.01e6, 0.208e6, 202500, 202500, 7, 4, 1.0, "flat"),
    ("5-point grid 1265", 8.0e6, 1.724e6, 1600225, 1600225, 49, 4, 1.0, "flat"),
    ("5-point grid 1410 fp64", 9.93e6, 2.33e6, 1988100, 1988100, 122, 8, 1.0, "flat"),
    ("27-point grid 43", 2.05e6, 0.0872e6, 79507, 79507, 3, 4, 1.0, "flat"),
    ("27-point grid 48", 2.86e6, 0.1246e6, 110592, 110592, 4, 4, 1.0, "flat"),
    ("27-point grid 53", 3.87e6, 0.1717e6, 148877, 148877, 5, 4, 1.0, "flat"),
    ("27-point grid 60 fp64", 5.64e6, 0.310e6, 216000, 216000, 14, 8, 1.0, "workers"),
    ("27-point grid 67", 7.88e6, 0.3827e6, 300763, 300763, 10, 4, 1.0, "workers"),
    ("R-MAT 2^17 fp64", 1.94e6, 0.263e6, 131072, 77000, 8, 8, 12.7, "flat"),
    ("R-MAT 2^18", 3.94e6, 0.5006e6, 262144, 148500, 8, 4, 13.9, "flat"),
    ("R-MAT 2^18 fp64", 3.94e6, 0.691e6, 262144, 148500, 16, 8, 13.9, "flat"),
    ("R-MAT 2^19 fp64", 7.97e6, 1.748e6, 524288, 285000, 32, 8, 14.1, "workers"),
    ("rows of 20, one block column", 3.0e6, 0.15e6, 150000, 150000, 1, 4, 1.0, "flat"),
    ("rows of 20, one block column", 4.0e6, 0.2e6, 200000, 200000, 1, 4, 1.0, "workers"),
    ("rows of 32, two block columns", 2.05e6, 0.128e6, 64000, 64000, 2, 4, 1.0, "flat"),
    ("rows of 32, three block columns", 3.07e6, 0.288e6, 96000, 96000, 3, 4, 1.0, "workers"),
    ("lognormal rows, three block columns", 1.99e6, 0.2133e6, 82000, 80500, 3, 4, 4.2, "flat"),
    ("lognormal rows, two block columns fp64", 2.48e6, 0.1886e6, 102000, 100000, 2, 8, 4.2, "workers"),
    ("lognormal rows, four block columns", 2.48e6, 0.31e6, 102000, 100000, 4, 4, 4.2, "workers"),
    ("lognormal rows, six block columns", 1.51e6, 0.2828e6, 62000, 60800, 6, 4, 4.2, "workers"),
    ("lognormal rows, eight block columns", 2.0e6, 0.4566e6, 82000, 80500, 8, 4, 4.2, "workers"),
    ("lognormal rows, four block columns fp64", 1.51e6, 0.2077e6, 62000, 60800, 4, 8, 4.2, "workers"),
    ("rows of 4", 1.0e6, 0.826e6, 250000, 250000, 8, 4, 1.0, "flat"),
    ("rows of 4", 3.0e6, 2.80e6, 750000, 750000, 23, 4, 1.0, "workers"),
    ("rows of 4 fp64", 2.0e6, 1.905e6, 500000, 500000, 31, 8, 1.0, "workers"),
    # two in three rows are empty: the others are not "in a block column or two"
    ("10 in every third row", 1.0e6, 0.4405e6, 300000, 100000, 5, 4, 1.0, "flat"),
    ("10 in every third row", 2.0e6, 0.881e6, 600000, 200000, 5, 4, 1.0, "flat"),
    ("10 in every third row", 10.0e6, 4.405e6, 3000000, 1000000, 5, 4, 1.0, "workers"),
    ("10 in every third row fp64", 4.0e6, 2.53e6, 1200000, 400000, 10, 8, 1.0, "workers"),
]


def test_measured_matrices_run_the_faster_way(tmp_path):
    lines = ['#include <cstdio>', '#include "hbp_internal.h"', 'static void ask(double nnz, double S, long n_rows, long rows, long NBC, int vb, double uneven) {',
             '  const bool known = hbp::rows_matter((int64_t)nnz, n_rows);',
             '  const hbp::RowStats st{known ? (uint32_t)rows : 0u, known ? (unsigned long long)(uneven * nnz * nnz / rows) : 0ull};',
             '  std::printf("%d\\n", hbp::flat_wavefronts((int64_t)nnz, (int64_t)S, NBC, vb, st)); }', 'int main() {']
    lines += ["  ask(%r, %r, %d, %d, %d, %d, %r);" % m[1:8] for m in MEASURED]
    lines += ["  return 0; }"]
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text("\n".join(lines))
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2504_08860_amd", "csrc"), str(src), "-o", str(exe)])
    got = [int(v) for v in subprocess.check_output([str(exe)]).decode().split()]
    for m, wavefronts in zip(MEASURED, got, strict=True):
        assert (wavefronts > 0) == (m[8] == "flat"), (m, wavefronts)
        if wavefronts:
            assert wavefronts == (1 if m[1] < 8 * m[2] else 4), m
