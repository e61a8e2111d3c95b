"""Rows that the combine kernel requests (csrc/combine.hip), counted in the assembly that the compiler makes of it: one 16-byte load
per expert of a token and piece, up to eight experts, and never one more; in the instance for large calls every one of them
non-temporal, in the other none; the store of the result in neither.  No GPU is involved."""
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
    loads, stores, nt = {}, {}, {}
    for m in re.finditer(r"^(\w*combine_kernelILi(\d+)ELb([01])E\w*):(.*?)\.end_amdhsa_kernel", out.read_text(), re.M | re.S):
        key = int(m[2]), m[3] == "1"
        rows = re.findall(r"^\s*global_load_dwordx4 .*", m[4], re.M)
        out_rows = re.findall(r"^\s*global_store_dwordx4 .*", m[4], re.M)
        loads[key], stores[key] = len(rows), len(out_rows)
        nt[key] = {bool(re.search(r"\bnt\b", r)) for r in rows}, {bool(re.search(r"\bnt\b", r)) for r in out_rows}
    per_token = {0: 8 + 4 + 2 + 1, **{k: k for k in range(1, 9)}}
    assert loads == {(k, streamed): n for k, n in per_token.items() for streamed in (False, True)}
    assert set(stores.values()) == {1}
    assert nt == {(k, streamed): ({streamed}, {False}) for k in per_token for streamed in (False, True)}
