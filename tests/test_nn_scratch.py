"""The network's scratch serves every call of up to `batch` samples (no GPU):
the launch plans of a smaller call can take more blocks, and so more partial
sums, than those of the full batch."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("scratch") / "nn_scratch_check")
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(HERE, "nn_scratch_check.cpp"), "-o",
                    exe], check=True)
    return exe


@pytest.mark.parametrize("grid", [8, 16, 32, 64, 128, 256])
def test_every_smaller_call_fits(checker, grid):
    for one, two in ((256, 256), (512, 512), (304, 152), (32, 32), (1, 1)):
        r = subprocess.run([checker, str(grid), str(one), str(two)], capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0 and r.stdout.startswith("ok"), (one, two, r.stdout + r.stderr)


@pytest.mark.parametrize("grid", [8, 16, 32, 64, 128, 256])
def test_workspace_grows_with_the_batch(grid):
    """Room for one sample more is never less room."""
    from paper_1710_04751_amd import capi
    sizes = [capi.lbm_nn_workspace_bytes(capi.nn_config(grid, n)) for n in range(1, 65)]
    assert all(a < b for a, b in zip(sizes, sizes[1:])), [
        n + 1 for n in range(63) if sizes[n] >= sizes[n + 1]]
