"""Rows that the combine kernel requests (csrc/combine.hip), counted in the assembly that the compiler makes of it: one 16-byte load
per expert of a token and piece, up to eight experts, and never one more.  No GPU is involved."""
import os
import re
import subprocess

from paper_2605_23911_amd import build


def test_one_load_per_expert(tmp_path):
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    out = tmp_path / "combine.s"
    res = subprocess.run([build.hipcc(), *flags, "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), "--offload-device-only", "-S",
                          os.path.join(build.CSRC, "combine.hip"), "-o", str(out)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    loads = {}
    for m in re.finditer(r"^(\w*combine_kernelILi(\d+)E\w*):(.*?)\.end_amdhsa_kernel", out.read_text(), re.M | re.S):
        loads[int(m[2])] = len(re.findall(r"^\s*global_load_dwordx4 ", m[3], re.M))
    assert loads == {0: 8 + 4 + 2 + 1, **{k: k for k in range(1, 9)}}
