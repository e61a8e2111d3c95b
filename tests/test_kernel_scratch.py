"""Scratch memory of the GEMM kernels, from the metadata of the built library: what the epilogue and the other bodies of a kernel derive from the
thread's number is worked out where it is used, not kept in registers through every body's reduction loop (tile_body_dma, rows_body).  Both down
projections with two weight blocks per wavefront have 256 accumulator registers in their tallest body and spill a value or two in its
prologue.  No GPU is involved."""
import re

import paper_2605_23911_amd as moe


def test_no_spills():
    moe.lib()
    blob = open(moe.library_path(), "rb").read()
    scratch = {}
    key = b"\xbb.private_segment_fixed_size"                # a kernel's metadata has its name, then this
    for m in re.finditer(rb"\xa5\.name(?:\xd9.|[\xa0-\xbf])(_Z\w+?)" + re.escape(key) + rb"([\x00-\x7f]|\xcc.|\xcd..)", blob, re.S):
        n = m[2]
        scratch[m[1].decode()] = n[0] if len(n) == 1 else int.from_bytes(n[1:], "big")
    gemms = {k: v for k, v in scratch.items() if re.search(r"tile_kernel|skinny_kernel", k)}
    assert len(gemms) == 15, sorted(gemms)
    wide = {k: v for k, v in gemms.items() if "tile_kernel_mixedILi2E" in k}
    assert len(wide) == 2 and all(v <= 12 for v in wide.values()), wide
    assert all(v == 0 for k, v in gemms.items() if k not in wide), gemms
