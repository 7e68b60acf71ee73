"""The sliced adjacency's build kernels (csrc/slice_build.h) run on the CPU
under the address and bounds sanitizers: the row order, the slices' places in
the workspace and every entry against the rows they were built from, at the
edges of the slices, of the shared arrays and of the largest graph of every
width, with regular, random and hub graphs."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_06921_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("slices") / "check")
    proc = subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,bounds", "-fno-sanitize-recover=all",
                           "-Wno-unknown-pragmas", "-I", CSRC, os.path.join(ROOT, "tests", "slice_build_host.cpp"),
                           "-o", exe], capture_output=True, text=True)
    assert proc.returncode == 0, proc.stderr
    return exe


@pytest.mark.parametrize("log2T,rows", [
    (0, (1, 63, 64, 65, 1000, 3000)), (1, (64, 129)), (2, (64, 1000)),
    (4, (1, 15, 16, 17, 1024, 1025)), (4, (1152, 1153, 1229)), (4, (1500, 2047, 2048)),
    (5, (1, 7, 8, 9, 65, 500)), (5, (1023, 1024)), (6, (1, 3, 4, 5, 511, 512))])
def test_slices_hold_the_rows(program, log2T, rows):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0")
    proc = subprocess.run([program, str(log2T)] + [str(n) for n in rows], capture_output=True, text=True, env=env,
                          timeout=300)
    assert proc.returncode == 0 and "0 failure(s)" in proc.stdout, proc.stdout[-2000:] + proc.stderr[-4000:]
