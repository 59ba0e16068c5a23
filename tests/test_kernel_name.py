"""CPU check of the names of the step kernels (no GPU): one for each precision,
scalar lattice, collision and number of steps a launch, made without allocating."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1710_04751_amd")


def test_names_without_allocating(tmp_path):
    exe = str(tmp_path / "kernel_name_check")
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                    os.path.join(HERE, "kernel_name_check.cpp"), "-o", exe, "-L", PKG,
                    "-l:liblbm.so", f"-Wl,-rpath,{PKG}"], check=True, stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    want = [f"lbm::kern::k_step{'3' if threes else ''}<{types}, {q}, {general}"
            f"{'' if threes else ', 1'}>"
            for types in ("double, double", "float, float", "float, _Float16")
            for q in (7, 15) for general in ("false", "true") for threes in (False, True)]
    assert r.stdout.splitlines() == want
