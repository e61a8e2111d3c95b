"""Steps that the loads of rows_body (csrc/ffn_kernels.hpp) run ahead, read from the assembly that the compiler makes of it: where
four ring buffers fit, the end of a k step leaves one step's loads outstanding or, if asked, two; where three fit, one.  No other
wait on the vector-memory counter is in the loop: it would empty the ring at every step.  No GPU is involved."""
import os
import re
import subprocess

import pytest

from paper_2605_23911_amd import build

KERNEL = """
#include "ffn_kernels.hpp"
namespace moe { namespace {
__global__ __launch_bounds__(kThreads) void probe(const GemmArgs a, const Tile t, int nt, bool deep) {
    extern __shared__ __attribute__((aligned(1024))) uint16_t xs[];
    rows_body<%d, 1, %s, %s, true>(a, t, nt, deep, xs);
}
} }
"""


@pytest.mark.parametrize("packed", ["true", "false"])
@pytest.mark.parametrize("blocks,gateup,buffers", [(1, "false", 4), (4, "false", 4), (8, "false", 3), (1, "true", 4), (3, "true", 3)])
def test_outstanding_loads(tmp_path, blocks, gateup, buffers, packed):
    src = tmp_path / "probe.hip"
    src.write_text(KERNEL % (blocks, gateup, packed))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    res = subprocess.run([build.hipcc(), *flags, "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), "--offload-device-only", "-S",
                          str(src), "-o", str(tmp_path / "probe.s")], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    loads = blocks + 4 * (2 if gateup == "true" else 1)      # of a wavefront and step
    text = (tmp_path / "probe.s").read_text()
    find = lambda part: {int(n) for n in re.findall(r"s_waitcnt[^\n]*vmcnt\((\d+)\)", part)}
    want = {loads} | ({2 * loads} if buffers == 4 else set())
    assert want <= find(text)
    assert find(text[text.index("v_mfma"):text.rindex("v_mfma")]) <= want
