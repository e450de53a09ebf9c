"""Which way the workers' kernel walks a group: the rules of hbp_internal.h against matrices for which both ways were timed on an
MI355X."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _ask(tmp_path, lines):
    """What the C++ expressions give, one number each."""
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text("\n".join(['#include <cstdio>', '#include "hbp_internal.h"', 'int main() {'] +
                             [f'  std::printf("%lld\\n", (long long)({x}));' for x in lines] + ['  return 0; }']))
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2504_08860_amd", "csrc"), str(src), "-o", str(exe)])
    return [int(v) for v in subprocess.check_output([str(exe)]).decode().split()]


# (nonzeros of a long group, of the range it is in, wavefronts of the worker, whether sharing it was faster)
OUTWEIGHING = [
    ("rows of 150 and 20 in equal parts, 300K", 9600, 100_000, 16, False),
    ("rows of 150 and 20 in equal parts, 1M", 9600, 332_000, 16, False),
    ("rows of 150 and 20, 1 to 9, 3M", 9600, 386_000, 16, False),
    ("rows of 500, 150 and 20, 1 to 20 to 300, 1M", 9600, 116_000, 16, False),
    ("R-MAT 2^20, rows of 1000", 64_000, 65_500, 16, True),
    ("R-MAT 2^20", 20_000, 65_500, 16, True),
]


def test_groups_that_outweigh_the_others(tmp_path):
    got = _ask(tmp_path, [f"hbp::outweighs({e}u, {r}u, {w})" for _, e, r, w, _ in OUTWEIGHING])
    for (name, *_, shared), g in zip(OUTWEIGHING, got, strict=True):
        assert bool(g) == shared, name


def test_outweighing_groups_have_their_places(tmp_path):
    """As many as can be of a range, and the largest counts."""
    for wavefronts in (4, 8, 16):
        most = wavefronts // 2 - 1
        assert _ask(tmp_path, [f"hbp::outweighs({e}u, {r}u, {wavefronts}) && {most} <= hbp::kMaxOutweighing"
                               for e, r in ((1000, 1000 * most), (2**31 // (most + 1), 2**31 - 1))][:1] +
                              [f"hbp::outweighs(1000u, 1000u * {most + 1}u, {wavefronts})"]) == [1, 0]
    assert _ask(tmp_path, ["hbp::outweighs(2147483647u, 2147483647u, 16)", "hbp::outweighs(268435455u, 2147483647u, 16)"]) == [1, 0]


# (nonzeros, groups per worker of 256 workers, whether steps were at least as fast as packs, within 4 %)
STEPS = [
    ("rows of 4", 72_000_000, 1103, False),
    ("rows of 5", 90_000_000, 1103, False),
    ("5-point grid 6300", 198_424_800, 3359, False),
    ("rows of 1 and of 20", 54_539_986, 1223, True),
    ("rows of 1 and of 10", 64_988_516, 1223, True),
    ("rows of 1 and of 4", 50_007_428, 1223, True),
    ("rows of 2", 36_000_000, 1101, True),
    ("rows from templates", 33_554_324, 1336, True),
    ("lognormal 4M x 1M", 98_006_305, 3035, True),
    ("lognormal 4M x 400K", 98_080_849, 1886, True),
    ("R-MAT 2^22", 65_246_593, 1785, True),
    ("lognormal 150001 x 400009", 3_696_267, 71, False),
]


def test_matrices_walked_in_steps(tmp_path):
    lines = [f"hbp::walk_in_steps(4, hbp::walk_long_first({g} * 256, 256), {nnz}, {g} * 256)" for _, nnz, g, _ in STEPS]
    for (name, *_, steps), got in zip(STEPS, _ask(tmp_path, lines), strict=True):
        assert bool(got) == steps, name
    assert _ask(tmp_path, ["hbp::walk_in_steps(2, false, 1, 1)", "hbp::walk_in_steps(8, false, 1, 1)", "hbp::walk_in_steps(4, true, 1, 1)",
                           "hbp::walk_in_steps(4, false, 224000, 1000)", "hbp::walk_in_steps(4, false, 224001, 1000)"]) == [1, 0, 0, 1, 0]
