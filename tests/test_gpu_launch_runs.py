"""Launches that the rule deals to the XCDs in runs with multi-block experts in them (feature-tile counts that are no multiple of 8), both projections:
every row of h and y_perm against float64, for each kernel that has such launches."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("packed,dn,ib", [(True, 5, 1), (True, 6, 2), (True, 7, 2), (False, 0, 1), (False, 10, 2)])
def test_every_row_in_runs_with_multi_block_experts(packed, dn, ib):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    import paper_2605_23911_amd.binding as B
    from tests.test_launch_mapping import _schedule
    moe.lib()
    dev, d, F = "cuda:0", 1792, 1408                       # 14 (7 of 256) and 11 feature tiles
    n = [257, 300, 512, 513, 1030, 64] * 7 + [0, 1, 256]
    E, R, guard = len(n), sum(n), 300
    off, blocks, _, _ = _schedule(np.array(n), 256)
    for gateup, N, K, i, wnt in ((True, F, d, 1, packed), (False, d, F, ib, dn in (5, 6))):
        work = B.map_launch(gateup, i, wnt, N, 256, off, blocks, K=K, packed=packed, runs=True)
        assert {int(r[6]) for r in work if r[0]} == {1}, "the launch is meant to be dealt in runs"
    print(f"[runs] packed={packed} down variant {dn}", flush=True)
    g = torch.Generator(device=dev).manual_seed(dn)
    rnd = lambda *s, std=1.0: torch.empty(s, dtype=torch.bfloat16, device=dev).normal_(generator=g).mul_(std)
    x = rnd(R, d)
    w = rnd(E, F, d, std=d ** -0.5), rnd(E, F, d, std=d ** -0.5), rnd(E, d, F, std=F ** -0.5)
    cfg = moe.MoEConfig.of(R, d, F, E, 1)
    p = None
    if packed:
        p = torch.empty(moe.packed_weights_size(cfg), dtype=torch.uint8, device=dev)
        moe.moe_pack_weights(cfg, *w, p)
    ws = torch.empty(moe.ffn_workspace_size(cfg), dtype=torch.uint8, device=dev)
    h = torch.full((R + guard, F), 7.0, dtype=torch.bfloat16, device=dev)
    y = torch.full((R + guard, d), 7.0, dtype=torch.bfloat16, device=dev)
    try:
        B.test_knob(B.KNOB_DOWN_VARIANT, dn)
        moe.moe_grouped_ffn(cfg, x, torch.from_numpy(off).to(dev), *((None, None, None) if packed else w), h[:R], y[:R], ws, W_packed=p)
        torch.cuda.synchronize()
    finally:
        B.test_knob(B.KNOB_DOWN_VARIANT, -1)
    assert bool((h[R:] == 7.0).all()) and bool((y[R:] == 7.0).all())
    for e in range(E):
        if n[e] == 0:
            continue
        rows = slice(int(off[e]), int(off[e + 1]))
        xe = x[rows].double()
        rh = torch.nn.functional.silu(xe @ w[0][e].double().t()) * (xe @ w[1][e].double().t())
        ry = rh @ w[2][e].double().t()
        # bf16 results of fp32 sums, y_perm through a bf16 h: the bound that the parity tests state
        assert float((h[rows].double() - rh).abs().max()) <= 1e-2 * float(rh.abs().max()), f"h of expert {e}"
        assert float((y[rows].double() - ry).abs().max()) <= 1e-2 * float(ry.abs().max()), f"y_perm of expert {e}"


@pytest.mark.parametrize("packed", [True, False])
def test_no_rows_at_all(packed):
    """Buffers sized for rows of which none came: nothing is written."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    moe.lib()
    dev, E, R, d, F = "cuda:0", 8, 96, 512, 640
    print(f"[no rows] packed={packed}", flush=True)
    w = [torch.ones(s, dtype=torch.bfloat16, device=dev) for s in ((E, F, d), (E, F, d), (E, d, F))]
    cfg = moe.MoEConfig.of(R, d, F, E, 1)
    p = None
    if packed:
        p = torch.empty(moe.packed_weights_size(cfg), dtype=torch.uint8, device=dev)
        moe.moe_pack_weights(cfg, *w, p)
    h = torch.full((R, F), 7.0, dtype=torch.bfloat16, device=dev)
    y = torch.full((R, d), 7.0, dtype=torch.bfloat16, device=dev)
    ws = torch.empty(moe.ffn_workspace_size(cfg), dtype=torch.uint8, device=dev)
    moe.moe_grouped_ffn(cfg, torch.ones((R, d), dtype=torch.bfloat16, device=dev), torch.zeros(E + 1, dtype=torch.int32, device=dev),
                        *((None, None, None) if packed else w), h, y, ws, W_packed=p)
    torch.cuda.synchronize()
    assert bool((h == 7.0).all()) and bool((y == 7.0).all())
