"""Where a step's loads of rows_body (csrc/ffn_kernels.hpp) read: the start of the k loop comes from tables in memory, whose values the compiler
takes to differ by lane; it is made a scalar once, so that the loop does its addresses on the scalar unit.  Read from the assembly that the
compiler makes of it.  No GPU is involved."""
import os
import re
import subprocess

import pytest

from paper_2605_23911_amd import build

KERNEL = """
#include "ffn_kernels.hpp"
namespace moe { namespace {
__global__ __launch_bounds__(kThreads) void probe(const GemmArgs a, Tile t, const int* by_lane, int nt) {
    extern __shared__ __attribute__((aligned(1024))) uint16_t xs[];
    t.rot_mul = by_lane[threadIdx.x];
    rows_body<%d, 1, %s, false, false>(a, t, nt, false, xs);
}
} }
"""


@pytest.mark.parametrize("blocks,gateup", [(1, "true"), (8, "true"), (8, "false")])
def test_no_lane_values_in_the_loop(tmp_path, blocks, gateup):
    src = tmp_path / "probe.hip"
    src.write_text(KERNEL % (blocks, gateup))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    res = subprocess.run([build.hipcc(), *flags, "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), "--offload-device-only", "-S",
                          str(src), "-o", str(tmp_path / "probe.s")], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    text = (tmp_path / "probe.s").read_text()
    loop = text[text.index("v_mfma"):text.rindex("v_mfma")]
    assert len(re.findall(r"global_load_lds_dwordx4", loop)) > 0
    assert "v_readfirstlane" not in loop
