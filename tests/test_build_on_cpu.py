"""Control flow of the hierarchy build's kernels on the CPU (tests/hip_on_cpu runs a block's threads as fibers): the
sources of the library, compiled for the host."""
import os
import re
import subprocess

import pytest

from paper_2507_04021_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
CXX = os.path.join(os.path.dirname(os.path.dirname(B.HIPCC)), "llvm", "bin", "clang++")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("hip_on_cpu")
    emu = os.path.join(HERE, "hip_on_cpu")
    for f in ("common.h", "internal.h", "bvh.hip", "sort.hip"):
        with open(os.path.join(B.CSRC, f)) as src:
            text = re.sub(r"^.*__asm__ volatile.*\n", "", src.read(), flags=re.M)  # (orders loads on the GPU)
        (d / f.replace(".hip", ".cpp")).write_text(text)
    out = str(d / "build")
    cmd = [CXX, "-O1", "-std=c++17", "-w", "-ffp-contract=on", "-I" + emu, "-I" + str(d), "-I" + B.INCLUDE, "-include",
           "hip/hip_runtime.h", str(d / "bvh.cpp"), str(d / "sort.cpp"), os.path.join(emu, "fibers.cpp"),
           os.path.join(emu, "build_main.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


def _run(program, *args):
    r = subprocess.run([program] + [str(a) for a in args], capture_output=True, text=True, timeout=100)
    return r.returncode, r.stdout.strip()


@pytest.mark.parametrize("n,width,builder", [(3, 4, 2), (700, 4, 2), (1013, 8, 2), (2025, 4, 2), (700, 8, 1)])
def test_build_puts_every_disk_into_one_leaf(program, n, width, builder):
    rc, out = _run(program, n, width, builder)
    assert rc == 0 and out.startswith("built") and out.endswith("disks %d" % n), (rc, out)


@pytest.mark.parametrize("width,level", [(4, 0), (4, 1), (4, 3), (4, 7), (8, 1)])
@pytest.mark.parametrize("backwards", [0, 1])
def test_a_build_that_gives_up_ends_and_is_refused(program, width, level, backwards):
    """The fail word rises while the wavefronts of a block look at it: the block takes one decision, the later launches
    find no frontier, and the host follows nothing that they left unwritten."""
    rc, out = _run(program, 700, width, 2, level, backwards)
    assert rc == 0 and out.startswith("refused"), (rc, out)
