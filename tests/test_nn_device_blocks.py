"""The number of blocks the weight gradient's plans follow is the current
device's (no GPU; the device queries are stubs): an answer the runtime did not
give is not kept, and each device has its own."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1710_04751_amd", "liblbm.so")
CHILD = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before the library: its names win
lib = ctypes.CDLL(sys.argv[2])
class Config(ctypes.Structure):
    _fields_ = [("grid", ctypes.c_int32), ("batch", ctypes.c_int32), ("lr", ctypes.c_float),
                ("beta1", ctypes.c_float), ("beta2", ctypes.c_float), ("eps", ctypes.c_float),
                ("scale", ctypes.c_float * 4)]
lib.lbm_nn_workspace_bytes.restype = ctypes.c_size_t
for word in sys.argv[3:]:
    device, units = map(int, word.split(":"))
    ctypes.c_int.in_dll(stub, "stub_device").value = device
    ctypes.c_int.in_dll(stub, "stub_units").value = units
    print(lib.lbm_nn_workspace_bytes(ctypes.byref(Config(32, 16, 1e-3, 0.9, 0.999, 1e-8))))
"""


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    stub = str(tmp_path_factory.mktemp("stub") / "libstub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", os.path.join(HERE, "device_query_stub.c"), "-o", stub],
                   check=True)

    def run(*devices):
        r = subprocess.run([sys.executable, "-c", CHILD, stub, LIB, *devices], capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [int(v) for v in r.stdout.split()]
    return run


def test_the_stub_reaches_the_plans(sizes):
    assert sizes("0:64")[0] > 0 and sizes("0:64") != sizes("0:512")


def test_a_failed_query_is_not_kept(sizes):
    assert sizes("-1:0", "0:64")[1] == sizes("0:64")[0]


def test_each_device_has_its_own(sizes):
    assert sizes("0:512", "1:64", "0:512") == sizes("0:512") + sizes("1:64") + sizes("0:512")
