"""The loads from memory straight into LDS (csrc/lds_dma.hpp) are inline assembly, inside which the compiler places no wait
states.  gfx9 wants five between a vector instruction that writes a scalar register and a vector-memory instruction that reads
it as its address, and one between a scalar write of M0 and the load that goes through it.  Here the helpers are compiled for
gfx950 with operands that come from vector registers, the case in which the compiler itself adds such writes right in front of
the statement, and the assembly is checked.  No GPU is involved."""
import os
import re
import subprocess

import pytest

from paper_2605_23911_amd import build

KERNEL = """
#include "lds_dma.hpp"
extern __shared__ char lds[];
// base and source address differ by lane as far as the compiler can tell
__global__ void probe(const char* const* bases, uint32_t* out) {
    const char* b = bases[threadIdx.x];
    %s;
    moe::wait_vmcnt<0>();
    __syncthreads();
    out[threadIdx.x] = lds[threadIdx.x];
}
"""
CALLS = {"uniform base": "moe::lds_dma16_at<false>(b, threadIdx.x * 16, (uint32_t)(uintptr_t)lds)",
         "uniform base, non-temporal": "moe::lds_dma16_at<true>(b, threadIdx.x * 16, (uint32_t)(uintptr_t)lds)",
         "lane address": "moe::lds_dma16(b, (uint32_t)(uintptr_t)lds)"}

VALU_TO_VMEM = 5
M0_TO_LDS_LOAD = 1


def _scalars(operand):
    """Scalar registers an operand names: s7, s[4:5], m0."""
    if operand == "m0":
        return {"m0"}
    m = re.fullmatch(r"s(\d+)", operand)
    if m:
        return {int(m[1])}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    return set(range(int(m[1]), int(m[2]) + 1)) if m else set()


def hazards(asm):
    """Violations in straight-line gfx9 assembly, and the number of LDS loads looked at."""
    found, loads = [], 0
    states, by_valu, m0_at = 0, {}, -99     # wait states so far; at which of them a register was written
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        if not re.match(r"(s|v|ds|global|buffer|flat|scratch)_", line):
            continue
        op, _, rest = line.partition(" ")
        args = [a.strip() for a in rest.replace(" off", ", off").split(",")]
        args = [w for a in args for w in a.split()]
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            to_lds = "_lds_" in op
            loads += to_lds
            for r in set().union(*map(_scalars, args)):
                if states - by_valu.get(r, -99) < VALU_TO_VMEM:
                    found.append((line, "scalar address written by a vector instruction %d states before" % (states - by_valu[r])))
            if to_lds and states - m0_at < M0_TO_LDS_LOAD:
                found.append((line, "M0 written %d states before" % (states - m0_at)))
        states += int(args[0], 0) + 1 if op == "s_nop" else 1
        written = _scalars(args[0]) if args and not op.startswith(("s_nop", "s_waitcnt", "s_barrier")) else set()
        for r in written:
            if op.startswith("v_"):
                by_valu[r] = states
            elif op.startswith("s_"):
                by_valu.pop(r, None)
                if r == "m0":
                    m0_at = states
    return found, loads


def test_checker_sees_both_hazards():
    bad = "v_readfirstlane_b32 s4, v0\nv_readfirstlane_b32 s5, v1\ns_mov_b32 m0, s6\ns_nop 0\nglobal_load_lds_dwordx4 v2, s[4:5]\n"
    assert len(hazards(bad)[0]) == 2
    assert not hazards(bad.replace("s_nop 0", "s_nop 3"))[0]
    assert not hazards(bad.replace("s_nop 0", "s_mov_b64 s[8:9], s[4:5]").replace("v2, s[4:5]", "v2, s[8:9]"))[0]
    assert hazards("s_mov_b32 m0, s6\nglobal_load_lds_dwordx4 v[2:3], off\n")[0]


@pytest.mark.parametrize("call", list(CALLS))
def test_no_hazard_whatever_the_operands_come_from(tmp_path, call):
    src = tmp_path / "probe.hip"
    src.write_text(KERNEL % CALLS[call])
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    res = subprocess.run([build.hipcc(), *flags, "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), "--offload-device-only", "-S",
                          str(src), "-o", str(tmp_path / "probe.s")], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    found, loads = hazards((tmp_path / "probe.s").read_text())
    assert loads == 1
    assert not found, found
