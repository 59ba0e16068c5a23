"""CPU enumeration of the weight gradient's copies and LDS reads (no GPU):
tests/wgrad_index_check.cpp compiles the functions k_wgrad_tr runs for the host
and replays whole launches, over ranges of bricks that end inside a column, in
the last one and after one brick, inputs of 8 and 16 channels, inputs with a
coarser second tensor, and one or two output groups."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("wgrad") / "wgrad_index_check")
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                    os.path.join(HERE, "wgrad_index_check.cpp"), "-o", exe], check=True,
                   stderr=subprocess.DEVNULL)
    return exe


@pytest.mark.parametrize("c1s,c2,ys", [(8, 0, 16), (16, 0, 16), (16, 32, 16), (16, 0, 32), (32, 64, 32),
                                       (32, 0, 64), (16, 0, 24)])
@pytest.mark.parametrize("grid,samples,per", [(16, 2, 1), (16, 2, 3), (16, 3, 16), (32, 1, 7), (32, 1, 21),
                                              (64, 1, 63)])
def test_copies_and_reads(checker, grid, samples, per, c1s, c2, ys):
    if grid == 64 and c2:
        pytest.skip("long")
    groups = 1 if ys == 16 else 2
    r = subprocess.run([checker, *map(str, (groups, grid, samples, per, c1s, c2, ys))],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
