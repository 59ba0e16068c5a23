"""CPU check of how many of 16 blocks keep their results in the memory-side
cache (no GPU): all while everything fits, then about 170 MB of the states, and
in FP16 none where only one of 16 would."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shares(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("policy") / "cache_policy_check")
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                    os.path.join(HERE, "cache_policy_check.cpp"), "-o", exe], check=True,
                   stderr=subprocess.DEVNULL)

    def run(value_bytes, *mb):
        r = subprocess.run([exe, str(value_bytes), *map(str, mb)], capture_output=True, text=True,
                           check=True, timeout=60)
        return [int(v) for v in r.stdout.split()]
    return run


@pytest.mark.parametrize("value_bytes", [2, 4, 8])
def test_share_falls_with_the_states(shares, value_bytes):
    mb = [1, 100, 240, 241, 400, 800, 1300, 1361, 1920, 2700, 2721, 10000, 500000]
    got = shares(value_bytes, *mb)
    assert got[:3] == [16, 16, 16] and got[-3:] == [0, 0, 0]
    assert all(a >= b for a, b in zip(got, got[1:]))
    for m, s in list(zip(mb, got))[3:7]:
        assert s * m <= 16 * 170 < (s + 1) * m


def test_the_last_sixteenth(shares):
    """1.36 to 2.7 GB: one of 16 blocks keeps, except in FP16."""
    assert shares(4, 1361, 1920, 2700) == shares(8, 1361, 1920, 2700) == [1, 1, 1]
    assert shares(2, 1361, 1920, 2700) == [0, 0, 0]
