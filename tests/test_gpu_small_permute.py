"""Up to 1024 rows of packed weights the gate+up launch of moe_forward permutes by itself: the router's choice, the permutation's tables, h, y_perm and y
bit for bit as with the permutation in a launch of its own, from one row to 1024, two experts to 256, blocks of 32 rows, several
blocks per expert, the build for two workgroups per CU and the combine folded into the down projection."""
import numpy as np
import pytest
import torch

import moe_inputs as mi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,F,E,k,tile_m,skew", [
    (1, 128, 64, 2, 1, 0, 0.0), (1, 256, 192, 8, 8, 0, 0.0), (64, 256, 512, 8, 2, 0, 1.0), (32, 192, 320, 256, 8, 0, 0.0),
    (63, 320, 128, 5, 4, 32, 1.5), (128, 256, 256, 3, 2, 32, 1.0), (256, 128, 128, 2, 1, 32, 2.0), (255, 128, 192, 2, 1, 0, 2.0),
    (64, 2048, 128, 64, 4, 0, 0.5), (31, 4096, 64, 40, 8, 0, 2.0), (128, 64, 64, 2, 2, 64, 0.0), (257, 128, 64, 4, 1, 0, 0.0),
    (512, 256, 192, 8, 2, 0, 1.0), (341, 128, 64, 16, 3, 32, 2.0), (128, 128, 64, 256, 8, 0, 0.3), (1024, 64, 64, 9, 1, 0, 2.0), (100, 2048, 64, 64, 8, 0, 1.0),
    (1025, 64, 64, 9, 1, 0, 0.0)])
def test_permutation_inside_the_gate_up_launch(T, d, F, E, k, tile_m, skew):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as G
    import paper_2605_23911_amd.binding as B
    print(f"[small permute] T={T} d={d} F={F} E={E} k={k} tile_m={tile_m}", flush=True)
    layer = G.Layer(mi.MoEShape("small", T, d, F, E, k, mi.GATE_SOFTMAX_RENORM), seed=T + E, skew=skew)
    for flags in (0, 1):       # 1: MOE_FLAG_FUSE_COMBINE
        try:
            B.test_knob(B.KNOB_SMALL_PERMUTE, 1)
            got = G.run_forward(layer, tile_m=tile_m, flags=flags)
            B.test_knob(B.KNOB_SMALL_PERMUTE, 0)
            want = G.run_forward(layer, tile_m=tile_m, flags=flags)
        finally:
            B.test_knob(B.KNOB_SMALL_PERMUTE, -1)
        for name in want:
            assert np.array_equal(got[name], want[name]), name
        assert (got["y"] != 0).any(axis=1).all()
