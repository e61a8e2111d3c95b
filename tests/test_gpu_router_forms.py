"""Router, scan and combine kernels at the edges of their tiles; the router against logits, softmax and top-k in float64 (torch): the int8
form (128 tokens x 64 experts per workgroup, 64 elements of d per step, up to 16 slices of d)
forced on, the all-fp64 form at token counts where the slices of d are chosen by rounds, the one-launch
form for up to eight experts, and the permutation's scan over more chunks than one batch of loads.

Bound on a weight, relative: one rounding to fp32 (2^-24), plus, in the int8 form, twice what a logit may be off (2^-25): 2^-23."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))

pytestmark = pytest.mark.gpu


def _check(moe, T, d, E, k, gating, seed, bias=False):
    dev = "cuda:0"
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(T, d, generator=g).to(torch.bfloat16).to(dev)
    wr = (torch.randn(E, d, generator=g) * d ** -0.5).to(torch.bfloat16).to(dev)
    b = torch.randn(E, generator=g).to(dev) if bias else None
    cfg = moe.MoEConfig.of(T, d, 64, E, k, gating)
    idx = torch.full((T, k), -1, dtype=torch.int32, device=dev)
    w = torch.full((T, k), float("nan"), device=dev)
    ws = torch.empty(moe.route_workspace_size(cfg), dtype=torch.uint8, device=dev)
    moe.moe_route(cfg, x, wr, b, idx, w, ws)
    torch.cuda.synchronize()
    z = x.double() @ wr.double().t()
    if b is not None:
        z += b.double()
    top, want = torch.topk(z, min(k + 1, E), dim=1)
    assert E == 1 or float((top[:, :-1] - top[:, 1:]).min()) > 1e-9    # certifies the order
    top, want = top[:, :k], want[:, :k]
    assert torch.equal(idx.long(), want)
    ref = {0: torch.exp(top - torch.logsumexp(z, 1, keepdim=True)), 1: torch.softmax(top, 1),
           2: torch.sigmoid(top) / torch.sigmoid(top).sum(1, keepdim=True)}[gating]
    assert float(((w.double() - ref).abs() / ref).max()) <= 1.001 * 2.0 ** -23


def _moe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    moe.lib()
    return moe


@pytest.mark.parametrize("T,d,E,k,gating", [(256, 64, 9, 2, 0), (257, 128, 33, 8, 1), (320, 192, 129, 4, 2), (300, 1088, 200, 8, 0),
                                            (383, 576, 256, 8, 1), (513, 2880, 128, 6, 0),
                                            (384, 1024, 65, 4, 0), (385, 960, 64, 4, 1)])
def test_int8_form(T, d, E, k, gating):
    moe = _moe()
    import paper_2605_23911_amd.binding as B
    print(f"[router] int8 form forced, T={T} d={d} E={E} k={k} gating={gating}", flush=True)
    B.test_knob(B.KNOB_ROUTE_EXACT, 0)
    try:
        _check(moe, T, d, E, k, gating, T + E, bias=E % 2 == 0)
    finally:
        B.test_knob(B.KNOB_ROUTE_EXACT, -1)


@pytest.mark.parametrize("T,d,E,k", [(1000, 1088, 256, 8), (1500, 320, 65, 8), (2033, 192, 160, 6), (40, 64, 64, 64)])
def test_all_fp64_slices(T, d, E, k):
    print(f"[router] all fp64, T={T} d={d} E={E} k={k}", flush=True)
    _check(_moe(), T, d, E, k, 0, T + E, bias=True)


@pytest.mark.parametrize("E", range(1, 9))
@pytest.mark.parametrize("d", [64, 2112, 4160])
def test_one_launch_form(E, d):
    print(f"[router] one launch, E={E} d={d}", flush=True)
    _check(_moe(), 13, d, E, min(E, 3), E % 3, 7 * E + d, bias=E % 2 == 1)


@pytest.mark.parametrize("T,E", [(2049, 7), (4097, 256), (8200, 33)])     # x k = 4: 9, 17 and 33 chunks
def test_scan_over_many_chunks(T, E):
    moe = _moe()
    import gpu_util as G
    from oracle import moe_oracle as orc
    print(f"[permute] T={T} E={E}", flush=True)
    rng = np.random.default_rng(T)
    idx = np.stack([rng.choice(E, 4, replace=False) for _ in range(T)]).astype(np.int32)
    c, o, ro, so, _ = G.run_permute(moe.MoEConfig.of(T, 64, 64, E, 4), idx, torch.zeros((T, 64), dtype=torch.bfloat16, device="cuda:0"))
    for got, want in zip((c, o, ro, so), orc.permutation(idx, E)):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 17])
def test_combine_row_batches(k):
    """Every batch width of the combine kernel and its remainders.  An fp32 sum of k products is off by at most
    (k + 1) 2^-24 sum|w y|, and one rounding to bf16 by half a unit in the last place (2^-8)."""
    moe = _moe()
    print(f"[combine] k={k}", flush=True)
    dev, T, d = "cuda:0", 37, 2112
    g = torch.Generator().manual_seed(k)
    yp = torch.randn(T * k, d, generator=g).to(torch.bfloat16).to(dev)
    w = torch.rand(T, k, generator=g).to(dev)
    row_of = torch.randperm(T * k, generator=g).to(torch.int32).to(dev)
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device=dev)
    moe.moe_combine(moe.MoEConfig.of(T, d, 64, 32, k), yp, row_of, w, y)
    torch.cuda.synchronize()
    terms = w.double()[:, :, None] * yp.double()[row_of.long().view(T, k)]
    ref = terms.sum(1)
    bound = 2.0 ** -8 * ref.abs() + (k + 1) * 2.0 ** -24 * terms.abs().sum(1) + 1e-30
    assert float(((y.double() - ref).abs() / bound).max()) <= 1.0


@pytest.mark.parametrize("k", [6, 7, 10, 12, 15, 23, 32])
def test_combine_exact_batches(k):
    """The remaining exact batch widths, and eight-row batches with each remainder; the bound above."""
    test_combine_row_batches(k)
