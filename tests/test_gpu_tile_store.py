"""The GEMM epilogue stages a tile in LDS and stores whole rows: every row of an expert is written, none behind the last row of the
buffer, no feature behind the last one of a ragged tile (which would land in the next row), through both weight layouts and the
down projections for tiles of 256 rows, with single-block experts and multi-block ones.  Layers this small take cached stores throughout;
test_gpu_streamed_results.py has the non-temporal ones and the builds for two workgroups per CU."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [[1], [31, 1], [33, 255, 64], [256], [257], [600, 0, 7]])
@pytest.mark.parametrize("d,F", [(64, 64), (192, 448)])
def test_rows_and_guards(n, d, F):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    import paper_2605_23911_amd.binding as B
    moe.lib()
    dev, E, R, guard = "cuda:0", len(n), sum(n), 40
    g = torch.Generator().manual_seed(R + d)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).to(torch.bfloat16).to(dev)
    x = rnd(R, d)
    w = rnd(E, F, d, std=d ** -0.5), rnd(E, F, d, std=d ** -0.5), rnd(E, d, F, std=F ** -0.5)
    off = torch.tensor(np.concatenate([[0], np.cumsum(n)]), dtype=torch.int32, device=dev)
    cfg = moe.MoEConfig.of(R, d, F, E, 1)
    packed = torch.empty(moe.packed_weights_size(cfg), dtype=torch.uint8, device=dev)
    moe.moe_pack_weights(cfg, *w, packed)
    ws = torch.empty(moe.ffn_workspace_size(cfg), dtype=torch.uint8, device=dev)
    refh, refy = [], []
    for e in range(E):
        xe = x[sum(n[:e]):sum(n[:e + 1])].double()
        he = torch.nn.functional.silu(xe @ w[0][e].double().t()) * (xe @ w[1][e].double().t())
        refh.append(he)
        refy.append(he @ w[2][e].double().t())
    refh, refy = torch.cat(refh), torch.cat(refy)
    try:
        for p, variant in [(None, 0), (None, 9), (None, 10), (packed, 5), (packed, 6), (packed, 7)]:
            print(f"[tile store] n={n} d={d} F={F} packed={p is not None} down variant {variant}", flush=True)
            B.test_knob(B.KNOB_DOWN_VARIANT, variant)
            h = torch.full((R + guard, F), 7.0, dtype=torch.bfloat16, device=dev)
            y = torch.full((R + guard, d), 7.0, dtype=torch.bfloat16, device=dev)
            moe.moe_grouped_ffn(cfg, x, off, *(w if p is None else (None, None, None)), h[:R], y[:R], ws, W_packed=p)
            torch.cuda.synchronize()
            assert bool((h[R:] == 7.0).all()) and bool((y[R:] == 7.0).all())
            # bf16 results of fp32 sums, y_perm through a bf16 h: the bound that the parity tests state
            assert float((h[:R].double() - refh).abs().max()) <= 1e-2 * float(refh.abs().max())
            assert float((y[:R].double() - refy).abs().max()) <= 1e-2 * float(refy.abs().max())
    finally:
        B.test_knob(B.KNOB_DOWN_VARIANT, -1)
