"""What the resident sweep loop takes from the plan and the host, without a
GPU: `resident_check.cpp` links the planner with the host C++ compiler and
repeats the kernels' index arithmetic (shared with them in resident.h)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_02377_amd", "csrc")
SOURCES = ["host_plan.cpp", "host_partition.cpp", "host_csr.cpp", "host_graph.cpp"]


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    if not shutil.which("g++") or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the ROCm headers")
    exe = str(tmp_path_factory.mktemp("resident") / "resident_check")
    cmd = ["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
           "-I" + CSRC, os.path.join(ROOT, "tests", "resident_check.cpp")] + [os.path.join(CSRC, f) for f in SOURCES]
    subprocess.run(cmd + ["-o", exe], check=True, capture_output=True)
    return exe


def run(exe, *args):
    p = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr
    tok = p.stdout.split()
    return {k: int(v) for k, v in zip(tok[::2], tok[1::2])}


@pytest.mark.parametrize("N,mode,P", [(14, 1, 3), (22, 1, 5), (30, 2, 9), (40, 1, 50)])
def test_wide_table_kernels_read_within_the_footprint_and_its_ends(checker, N, mode, P):
    # bands that end in a tile of fewer than eight slices: waves with a
    # second slice that does not exist read too
    r = run(checker, "positions", N, 27, mode, P)
    assert r["wide"] == 1 and r["absent"] > 0


@pytest.mark.parametrize("sweeps", [200, 9973, 65536])
def test_control_words_of_an_old_solve_read_as_not_yet(checker, sweeps):
    # fixed sweeps number on without writing the stop words
    r = run(checker, "numbers", sweeps)
    assert r["clears"] >= 2


@pytest.mark.parametrize("N,points,mode,P,fmt", [(24, 7, 1, 8, 3), (17, 7, 2, 5, 4), (24, 7, 3, 8, 2), (15, 27, 1, 4, 3),
                                                 (22, 27, 2, 4, 4), (15, 27, 3, 4, 2)])
def test_footprints_decode_to_the_columns_of_the_other_loops(checker, N, points, mode, P, fmt):
    r = run(checker, "layout", N, points, mode, P)
    assert r["fmt"] == fmt and r["width"] <= 27
    # columns no entry of the tile has: what tables reach beyond their rows' entries, and the holes of the
    # 22^3 footprints, staged so that its widest slices take the loop's 27 slots
    assert (r["holes"] > 0) == (fmt == 3 or N == 22), r
