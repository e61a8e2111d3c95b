"""The token ring of digit_logits_kernel (csrc/route.hip), replayed from the assembly that the compiler makes of it.  The tokens go
from memory straight into LDS, each wavefront brings in a quarter of every operand that the others read, and a step's tile is first
read half a step early.  So between a tile's loads and its first read there has to be a barrier in front of which each wavefront
has waited for its own loads of that tile, and between the last read of a buffer and the next loads into it a barrier too.  No GPU is
involved."""
import os
import re
import subprocess

import pytest

from paper_2605_23911_amd import build


def _kernel(asm, name):
    body, inside = [], False
    for line in asm.splitlines():
        if re.match(r"_ZN\S*%s\S*:" % name, line):
            inside = True
        if inside and line.startswith(".Lfunc_end"):
            return body
        if inside:
            body.append(line.split(";")[0].strip())
    raise AssertionError(f"no kernel {name}")


def split_loop(lines):
    """Instructions in front of the loop over the steps (the one with the matrix instructions), from the block on that holds the first
    load into LDS, and those of one trip."""
    for end, line in enumerate(lines):
        m = re.match(r"s_cbranch_\w+ (\S+)", line)
        if m and lines.index(m[1] + ":") < end:
            start = lines.index(m[1] + ":")
            trip = lines[start + 1: end]
            if any(l.startswith("v_mfma_i32") for l in trip):
                assert not any(re.match(r"s_c?branch|\S+:$", l) for l in trip), "the trip is one straight line"
                first = next(i for i, l in enumerate(lines) if "global_load_lds" in l)
                block = max(i for i, l in enumerate(lines[:first]) if l.endswith(":"))
                return lines[block:start], trip
    raise AssertionError("no loop")


def faults(before, trip, buffers, loads_per_tile=4, reads_per_half=2, trips=7):
    """Tile g is loaded into buffer g % buffers: tiles 0 and 1 in front of the loop, g + 2 in trip g.  Its first half is read in trip
    g - 1 (tile 0: in front of the loop), its second in trip g."""
    found, queue, lds = [], [], []      # memory operations in flight: the tile they bring, or None; LDS reads in flight: their tile
    n_loads = n_reads = 0
    landed, reads = {}, {}              # per tile: loads that this wavefront has awaited, reads that have returned
    visible, over = set(), set()        # tiles whose loads, tiles whose reads every wavefront had behind it at the last barrier
    for line in before + trip * trips:
        if "global_load_lds" in line:
            tile, n_loads = n_loads // loads_per_tile, n_loads + 1
            if tile >= buffers and tile - buffers not in over:
                found.append(f"tile {tile} is loaded over one that may still be read")
            queue.append(tile)
        elif re.match(r"(global|buffer|flat)_", line):
            queue.append(None)
        elif line.startswith("ds_read"):
            tile, n_reads = n_reads // reads_per_half // 2, n_reads + 1
            if tile not in visible:
                found.append(f"tile {tile} is read before a barrier behind which all of it has landed")
            lds.append(tile)
        elif line.startswith("s_waitcnt"):
            for counter, flight, done in (("vmcnt", queue, landed), ("lgkmcnt", lds, reads)):
                m = re.search(r"\b%s\((\d+)\)" % counter, line)
                while m and len(flight) > int(m[1]):
                    tile = flight.pop(0)
                    done[tile] = done.get(tile, 0) + 1
        elif line == "s_barrier":
            visible = {t for t, n in landed.items() if n == loads_per_tile}
            over = {t for t, n in reads.items() if n == 2 * reads_per_half}
    assert n_loads == loads_per_tile * (2 + trips) and n_reads == reads_per_half * (1 + 2 * trips), "the loop as described"
    return found


@pytest.fixture(scope="module")
def kernel(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "route.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    res = subprocess.run([build.hipcc(), *flags, "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), "--offload-device-only", "-S",
                          os.path.join(build.CSRC, "route.hip"), "-o", str(out)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    source = open(os.path.join(build.CSRC, "route.hip")).read()
    return *split_loop(_kernel(out.read_text(), "digit_logits_kernel")), int(re.search(r"\bNB = (\d+)", source)[1])


def test_every_tile_is_awaited_by_all_wavefronts_before_it_is_read(kernel):
    before, trip, buffers = kernel
    assert not faults(before, trip, buffers)
    # the wait in front of the barrier is enough by itself, without those that the compiler places for the experts' digits
    at = trip.index("s_barrier")
    bare = [l for i, l in enumerate(trip) if i == at - 1 or not re.match(r"s_waitcnt vmcnt", l)]
    assert not faults(before, bare, buffers)


def test_the_replay_sees_planted_mistakes(kernel):
    before, trip, buffers = kernel
    trip = [l for i, l in enumerate(trip) if trip[(i + 1) % len(trip)] == "s_barrier" or not re.match(r"s_waitcnt vmcnt", l)]
    at = trip.index("s_barrier")
    assert not faults(before, trip, buffers)
    assert faults(before, trip[:at] + trip[at + 1:], buffers)                                            # no barrier
    assert faults(before, trip[:at - 1] + ["s_waitcnt vmcnt(17)"] + trip[at:], buffers)                  # one load less awaited
    assert faults(before, trip[:at - 1] + trip[at + 1:] + trip[at - 1: at + 1], buffers)                 # both at the end of the trip
    assert faults(before, trip, 1)                                                                       # one buffer only
