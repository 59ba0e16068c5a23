"""What the step kernels compile to (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_1710_04751_amd import build as B


def compiled(source, tmp_path, *flags):
    out = str(tmp_path / "out")
    r = subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "-w", "-x", "hip", "--cuda-device-only", "-S", *flags,
                        os.path.join(B.CSRC, source), "-o", out], check=True, capture_output=True,
                       text=True)
    with open(out) as f:
        return f.read(), r.stderr


def test_steps_of_one_policy_keep_their_registers(tmp_path):
    """A single cavity's kernels spill nothing where all blocks take one cache
    policy (every box below 240 MB or above 2.7 GB)."""
    _, remarks = compiled("lbm_step.hip", tmp_path, "-Rpass-analysis=kernel-resource-usage")
    kernels = re.findall(r"Function Name: (\S*k_step\S*).*?VGPRs Spill: (\d+)", remarks, re.S)
    checked = 0
    for name, spilled in kernels:
        ways = re.search(r"Lb[01]ELi(\d+)EEEv", name)
        if ways and bin(int(ways[1])).count("1") > 1:
            continue
        assert int(spilled) == 0, name
        checked += 1
    assert checked >= 24


def test_batches_load_ordinarily(tmp_path):
    """Non-temporal loads cost a batch; only FP64 D3Q7 members use them."""
    code, _ = compiled("lbm_batch.hip", tmp_path)
    kernels = re.findall(r"^(\S*k_batch_stepI\S*):(.*?)s_endpgm", code, re.S | re.M)
    assert len(kernels) == 12
    for name, body in kernels:
        nt = re.findall(r"buffer_load_\S+ v\S*, v\d+,.* nt$", body, re.M)
        assert bool(nt) == ("IddLi7" in name), name
