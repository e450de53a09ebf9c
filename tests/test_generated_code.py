"""What the built library's kernels were compiled to (gfx950 assembly of this repository's own sources)."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of each kernel, by mangled name."""
    import paper_2504_08860_amd as H
    if not os.path.exists(H.LIB_PATH):
        from paper_2504_08860_amd.build import build_library
        build_library()
    at = tmp_path_factory.mktemp("code")
    shutil.copy(H.LIB_PATH, at / "lib.so")
    subprocess.check_call([OBJDUMP, "--offloading", "lib.so"], cwd=at, stdout=subprocess.DEVNULL)  # device code into files of its own
    found = {}
    for f in at.iterdir():
        if "gfx950" not in f.name:
            continue
        name = None
        for line in subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], text=True).splitlines():
            label = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
            if label:
                name = label.group(1)
                found[name] = []
            elif name and line.startswith("\t"):
                found[name].append(line.split("//")[0].strip())
    return found


def test_order_block_takes_its_arrays_for_global_memory(kernels):
    """An address that has been an integer may be LDS, too, for all the compiler knows: flat instructions, which wait with the LDS ones."""
    (code,) = [c for name, c in kernels.items() if "k_order_block" in name]
    assert sum(i.startswith(("global_load", "global_store")) for i in code) >= 10
    assert [i for i in code if i.startswith("flat_")] == []
