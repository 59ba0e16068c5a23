"""The hand-written copies to LDS say what they touch (no GPU): compiled here,
every inline assembly statement that writes m0 declares it, and no copy reads a
buffer descriptor within five wait states of a vector instruction's write to it
(the hardware does not wait for such a write, and the compiler's own checks do
not look into inline assembly)."""
import os
import re
import subprocess

import pytest

from paper_1710_04751_amd import build as B

SOURCE = os.path.join(B.CSRC, "nn_kernels.hip")


def compiled(tmp_path, *flags):
    out = str(tmp_path / "out")
    subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "-w", "-x", "hip", "--cuda-device-only", "-S", *flags,
                    SOURCE, "-o", out], check=True, stderr=subprocess.DEVNULL)
    with open(out) as f:
        return f.read()


def test_m0_is_declared(tmp_path):
    ir = compiled(tmp_path, "-emit-llvm", "-Xclang", "-disable-llvm-passes")
    asm = re.findall(r'asm (?:sideeffect )?"([^"]*)", "([^"]*)"', ir)
    writes = [(text, constraints) for text, constraints in asm if re.search(r"\bm0\b", text)]
    assert writes
    for text, constraints in writes:
        assert "~{m0}" in constraints.split(","), text


def sgprs(token):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", token)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", token)
    return {int(m[1])} if m else set()


def test_descriptors_have_settled(tmp_path):
    code = []
    for line in compiled(tmp_path).splitlines():
        text = line.split(";")[0].strip()
        if text and not text.startswith((".", "#")) and not text.endswith(":"):
            code.append(text.replace(",", " ").split())
    copies = 0
    for i, ins in enumerate(code):
        if ins[0] != "buffer_load_dwordx4" or ins[-1] != "lds":
            continue
        copies += 1
        waited, j = 0, i - 1
        while j >= 0 and waited < 5:
            op = code[j]
            if op[0].startswith("v_"):
                written = set().union(*(sgprs(t) for t in op[1:3]))
                assert not (op[0].startswith(("v_readfirstlane", "v_readlane", "v_cmp", "v_add_co", "v_sub_co",
                                              "v_addc_co", "v_subb_co", "v_div_scale", "v_mad_u64"))
                            and written & sgprs(ins[2])), (op, ins)
            waited += int(op[1], 0) + 1 if op[0] == "s_nop" else 1
            j -= 1
    assert copies > 100
