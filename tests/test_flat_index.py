"""CPU enumeration of the step's blocks of consecutive cells (no GPU): the
cell of every lane and the window of every block, over edges where the
quotients by nx and ny go from tables of small divisors to 0 or 1 (1024), a
block spans several planes, and the last block is partial."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("flat") / "flat_index_check")
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                    os.path.join(HERE, "flat_index_check.cpp"), "-o", exe], check=True,
                   stderr=subprocess.DEVNULL)
    return exe


@pytest.mark.parametrize("shape", [(4, 4, 4), (5, 4, 7), (91, 13, 4), (4, 700, 5), (63, 65, 6),
                                   (1023, 5, 4), (1024, 4, 4), (1025, 4, 5), (6, 1023, 4),
                                   (4, 1025, 4), (2100, 4, 4)])
@pytest.mark.parametrize("qt,vb", [(7, 4), (15, 2), (7, 8)])
def test_blocks_of_consecutive_cells(checker, shape, qt, vb):
    for threads in (64, 256, 1024):
        r = subprocess.run([checker, *map(str, (*shape, qt, vb, threads))], capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0 and r.stdout == "ok\n", (threads, r.stdout + r.stderr)
