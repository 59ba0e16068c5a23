"""CPU check of which small boxes go three steps a launch (no GPU): the rule
follows the device's compute units, and only updates that were measured faster
with two blocks on a unit take two."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
FP64, FP32, FP16 = 0, 1, 2


@pytest.fixture(scope="module")
def threes(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("threes") / "threes_rule_check")
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                    os.path.join(HERE, "threes_rule_check.cpp"), "-o", exe], check=True,
                   stderr=subprocess.DEVNULL)

    def run(precision, q, box, source=0, stochastic=0, specular=0, units=256):
        r = subprocess.run([exe, *map(str, (units, precision, q, source, stochastic, specular,
                                           *box))],
                           capture_output=True, text=True, check=True, timeout=60)
        return r.stdout == "1\n"
    return run


@pytest.mark.parametrize("precision", [FP64, FP32, FP16])
@pytest.mark.parametrize("q", [7, 15])
@pytest.mark.parametrize("units", [256, 64, 32])
def test_one_block_a_unit_always(threes, precision, q, units):
    edge = {256: 24, 64: 16, 32: 12}[units]
    assert threes(precision, q, (edge, edge, edge), source=1, units=units)
    assert not threes(precision, q, (edge + 24, edge + 24, edge + 24), units=units)


def test_two_blocks_a_unit(threes):
    cube, odd, long = (32, 32, 32), (30, 30, 30), (64, 16, 32)
    assert not threes(FP64, 7, (28, 28, 28))
    for box in (cube, odd, long):
        assert threes(FP32, 7, box) and threes(FP32, 7, box, source=1) and threes(FP16, 7, box)
        assert not threes(FP32, 7, box, units=128)
    for kind in (dict(precision=FP32, q=15), dict(precision=FP16, q=7, stochastic=1),
                 dict(precision=FP16, q=15), dict(precision=FP16, q=15, source=1)):
        assert threes(box=cube, **kind) and threes(box=(40, 28, 28), **kind)
        assert not threes(box=odd, **kind) and not threes(box=long, **kind)
    for kind in (dict(precision=FP32, q=15, source=1), dict(precision=FP16, q=15, stochastic=1)):
        assert not threes(box=cube, **kind) and threes(box=(24, 24, 24), **kind)


def test_rows_that_end_early_in_a_tile(threes):
    ragged = [(13, 13, 13), (5, 17, 53), (14, 24, 24)]
    whole = [(12, 13, 13), (15, 9, 9), (16, 4, 60), (18, 18, 18), (33, 17, 9)]
    for kind in (dict(source=1), dict(specular=1)):
        for precision in (FP64, FP16):
            assert not any(threes(precision, 15, b, **kind) for b in ragged)
            assert all(threes(precision, 15, b, **kind) and threes(precision, 7, b, **kind) for b in whole)
            assert all(threes(precision, 7, b, **kind) for b in ragged)
        assert all(threes(FP32, 15, b, **kind) for b in ragged + whole)
    assert not any(threes(FP16, 15, b, stochastic=1) for b in ragged)
    for precision in (FP64, FP32, FP16):
        assert all(threes(precision, 15, b) for b in ragged + whole)
        assert not threes(precision, 15, (13, 4, 59)) and threes(precision, 7, (13, 4, 59))
