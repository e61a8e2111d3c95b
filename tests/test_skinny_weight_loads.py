"""Cache hint of the K-split kernel's weight loads (csrc/ffn_kernels.hpp, skinny_kernel), read from the assembly that the compiler
makes of it.  A load of packed weights consumes whole 128-byte lines once: non-temporal.  A row-major line is consumed by the
four loads of a step, and the hint drops it from the caches between them.  No GPU is involved."""
import os
import re
import subprocess

import pytest

from paper_2605_23911_amd import build


@pytest.mark.parametrize("height", [1, 2])
@pytest.mark.parametrize("packed", [True, False])
def test_non_temporal_only_where_a_load_consumes_whole_lines(tmp_path, packed, height):
    src = tmp_path / "probe.hip"
    src.write_text('#include "ffn_kernels.hpp"\nnamespace moe { namespace {\ntemplate __global__ void skinny_kernel<%d, false, 4, 4, %s>(const GemmArgs);\n} }\n'
                   % (height, str(packed).lower()))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    res = subprocess.run([build.hipcc(), *flags, "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), "--offload-device-only", "-S",
                          str(src), "-o", str(tmp_path / "probe.s")], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    loads = re.findall(r"^\s*global_load_dwordx4 .*$", (tmp_path / "probe.s").read_text(), re.M)
    hinted = [l for l in loads if re.search(r"\bnt\b", l)]
    # per step four weight loads and four loads of each 32-row block of tokens; tokens are re-read by other workgroups: never hinted
    assert len(loads) >= 16
    if packed:
        assert 0 < len(hinted) <= len(loads) / (1 + height)
    else:
        assert not hinted
