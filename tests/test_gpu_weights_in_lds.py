"""GEMM bodies that stage the weights in LDS (every tile of row-major weights; the single-block tiles
of packed ones): all rows of h and y_perm at the sizes where the body can go wrong - one to eight
32-row blocks and one row past each, two to four ring buffers, one to five k steps, output
widths that leave the last feature tile partly empty - through moe_grouped_ffn, with every
down-projection kernel that holds the body.

Error bounds, per element (u = 2^-24, K the reduction length): an fp32 sum of exact products is off by at
most K u sum|a||b|; SiLU's exp and reciprocal by a few 1e-7 relative; the result is rounded to bf16
once, to eight significant bits: half a unit in the last place is at most 2^-8 of the value.  y_perm is compared with the product of the kernel's own h, so it carries one
rounding only."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))

pytestmark = pytest.mark.gpu

COUNTS = {
    "heights": [1, 32, 33, 64, 96, 128, 129, 160, 161, 192, 224, 225, 256],
    "multi": [257, 0, 300, 31, 520, 160],          # experts of two and three tiles among small ones and an empty one
    "one_row": [0, 1, 0],
    "short_round": [200] * 3,                      # few workgroups: a down projection with a split last round
}


def _run(moe, cfg, x, offsets, w, packed, R):
    dev = x.device
    h = torch.full((R, cfg.F), float("nan"), dtype=torch.bfloat16, device=dev)
    y = torch.full((R, cfg.d), float("nan"), dtype=torch.bfloat16, device=dev)
    ws = torch.empty(moe.ffn_workspace_size(cfg), dtype=torch.uint8, device=dev)
    if packed is None:
        moe.moe_grouped_ffn(cfg, x, offsets, *w, h, y, ws)
    else:
        moe.moe_grouped_ffn(cfg, x, offsets, None, None, None, h, y, ws, W_packed=packed)
    torch.cuda.synchronize()
    return h, y


@pytest.mark.parametrize("counts", list(COUNTS))
@pytest.mark.parametrize("d,F", [(64, 128), (128, 64), (192, 320), (320, 192)])
def test_all_rows(counts, d, F):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    import paper_2605_23911_amd.binding as B
    moe.lib()
    dev = "cuda:0"
    n = COUNTS[counts]
    E, R = len(n), sum(n)
    g = torch.Generator().manual_seed(17 * d + F + R)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).to(torch.bfloat16).to(dev)
    x = rnd(R, d)
    w = rnd(E, F, d, std=d ** -0.5), rnd(E, F, d, std=d ** -0.5), rnd(E, d, F, std=F ** -0.5)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(n)]), dtype=torch.int32, device=dev)
    cfg = moe.MoEConfig.of(R, d, F, E, 1)
    packed = torch.empty(moe.packed_weights_size(cfg), dtype=torch.uint8, device=dev)
    moe.moe_pack_weights(cfg, *w, packed)
    u = 2.0 ** -24
    down = [(None, 0), (None, 9), (None, 10), (packed, 5), (packed, 6), (packed, 7)]
    try:
        for p, variant in down:
            print(f"[weights in LDS] {counts} d={d} F={F} packed={p is not None} down variant {variant}", flush=True)
            B.test_knob(B.KNOB_DOWN_VARIANT, variant)
            h, y = _run(moe, cfg, x, offsets, w, p, R)
            for e in range(E):
                a, b = sum(n[:e]), sum(n[:e + 1])
                if a == b:
                    continue
                xe, he = x[a:b].double(), h[a:b].double()
                wg, wu, wd = (t[e].double() for t in w)
                gate, up = xe @ wg.t(), xe @ wu.t()
                dg, du = d * u * (xe.abs() @ wg.abs().t()), d * u * (xe.abs() @ wu.abs().t())
                s = torch.nn.functional.silu(gate)
                ref = s * up
                bound = 2.0 ** -8 * ref.abs() + 1.1 * up.abs() * dg + s.abs() * du + 1e-6 * ref.abs() + 1e-30
                worst = float(((he - ref).abs() / bound).max())
                assert worst <= 1.0, ("h", e, variant, worst)
                refy = he @ wd.t()
                boundy = 2.0 ** -8 * refy.abs() + F * u * (he.abs() @ wd.abs().t()) + 1e-30
                worst = float(((y[a:b].double() - refy).abs() / boundy).max())
                assert worst <= 1.0, ("y_perm", e, variant, worst)
    finally:
        B.test_knob(B.KNOB_DOWN_VARIANT, -1)


@pytest.mark.parametrize("k", [1, 2])
@pytest.mark.parametrize("layout", ["row-major", "packed"])
def test_rows_through_the_source_map(layout, k):
    """moe_forward reads expert-contiguous row r from token src_of[r] / k: experts of 161 to 256 rows (two and three ring
    buffers) and just beyond one block.  The router's matrix picks features that the tokens carry their experts in, so every
    expert holds the rows asked for; h and y_perm are compared row by row with the bounds above."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    moe.lib()
    print(f"[weights in LDS] source map, {layout}, k={k}", flush=True)
    dev, d, F = "cuda:0", 192, 320
    n = [161, 192, 193, 224, 225, 256, 257, 300]
    E, R = len(n), sum(n)
    T = R // k
    assert T * k == R and max(n) <= T
    g = torch.Generator().manual_seed(91 + k)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).to(torch.bfloat16).to(dev)
    want = torch.repeat_interleave(torch.arange(E), torch.tensor(n)).view(k, T).t()    # [T, k], the experts of a token differ
    want = want[torch.randperm(T, generator=g)]
    x = rnd(T, d)
    x[:, :E] *= 0.125
    for j in range(k):
        x[torch.arange(T, device=dev), want[:, j].to(dev)] = 16.0 - 4.0 * j
    wr = torch.eye(E, d, dtype=torch.bfloat16, device=dev)
    w = rnd(E, F, d, std=d ** -0.5), rnd(E, F, d, std=d ** -0.5), rnd(E, d, F, std=F ** -0.5)
    cfg = moe.MoEConfig.of(T, d, F, E, k, moe.GATE_SOFTMAX_RENORM)
    packed = None
    if layout == "packed":
        packed = torch.empty(moe.packed_weights_size(cfg), dtype=torch.uint8, device=dev)
        moe.moe_pack_weights(cfg, *w, packed)
    lay = moe.forward_workspace_layout(cfg)
    ws = torch.full((lay.total,), 0xFF, dtype=torch.uint8, device=dev)                 # bf16 NaN where nothing is written
    y = torch.empty((T, d), dtype=torch.bfloat16, device=dev)
    moe.moe_forward(cfg, x, wr, None, *(w if packed is None else (None, None, None)), y, ws, W_packed=packed)
    torch.cuda.synchronize()
    src = ws[lay.src_of: lay.src_of + 4 * R].view(torch.int32).long()
    h = ws[lay.h: lay.h + 2 * R * F].view(torch.bfloat16).view(R, F)
    yp = ws[lay.y_perm: lay.y_perm + 2 * R * d].view(torch.bfloat16).view(R, d)
    counts = ws[lay.counts: lay.counts + 4 * E].view(torch.int32).tolist()
    assert counts == n
    u, a = 2.0 ** -24, 0
    for e in range(E):
        b = a + n[e]
        assert bool((want.reshape(-1).to(dev)[src[a:b]] == e).all())
        xe, he = x[src[a:b] // k].double(), h[a:b].double()
        wg, wu, wd = (t[e].double() for t in w)
        gate, up = xe @ wg.t(), xe @ wu.t()
        dg, du = d * u * (xe.abs() @ wg.abs().t()), d * u * (xe.abs() @ wu.abs().t())
        s = torch.nn.functional.silu(gate)
        ref = s * up
        bound = 2.0 ** -8 * ref.abs() + 1.1 * up.abs() * dg + s.abs() * du + 1e-6 * ref.abs() + 1e-30
        assert float(((he - ref).abs() / bound).max()) <= 1.0, ("h", e)
        refy = he @ wd.t()
        boundy = 2.0 ** -8 * refy.abs() + F * u * (he.abs() @ wd.abs().t()) + 1e-30
        assert float(((yp[a:b].double() - refy).abs() / boundy).max()) <= 1.0, ("y_perm", e)
        a = b


# 4096 output features are 32 feature tiles: eight blocks are one whole round of 256 workgroups (loads two steps ahead), seven are
# not (three steps where the ring holds four buffers)
ROUNDS = {"whole_round": [1, 33, 64, 65, 128, 160, 192, 256], "part_round": [1, 33, 65, 128, 160, 192, 193]}


@pytest.mark.parametrize("counts", list(ROUNDS))
@pytest.mark.parametrize("F", [64, 128, 320])
def test_steps_ahead(counts, F):
    COUNTS.update(ROUNDS)
    test_all_rows(counts, 4096, F)
