"""Loads and stores past the caches: the GEMM epilogue at ragged widths, at row counts on both sides of every 32-row body, with guard rows behind
the buffers, in every kernel that stages its tiles; the combine's instances for large calls at every batch width, just on their side of the line
and just below it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TALL = [1, 31, 33, 160, 161, 255, 256, 255]        # none above twice the mean: the rows of h are streamed too
SHORT = [1, 31, 32, 33, 97, 128, 127, 128]         # for the builds for two workgroups per CU, whose tiles hold 128 rows


def _streamed(B, gateup, ib, N, K, n, M, packed, half):
    """Experts whose results the launch stores non-temporally, by the code that the kernel runs."""
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    work = B.map_launch(gateup, ib, True, N, M, off, np.array([(e, 0) for e in range(len(n))], dtype=np.int32), K=K, packed=packed, half=half, runs=True)
    return {int(r[1]) for r in work if r[0] and r[7]}


@pytest.mark.parametrize("n,M,packed,gu,dn,ib,half", [
    (TALL, 0, False, -1, 0, 1, False), (TALL, 0, False, -1, 10, 2, False),
    (TALL, 0, True, 1, 5, 1, False), (TALL, 0, True, 1, 6, 2, False), (TALL, 0, True, 1, 7, 2, False), (SHORT, 128, True, 2, 8, 1, True)])
def test_rows_and_guards_streamed(n, M, packed, gu, dn, ib, half):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    import paper_2605_23911_amd.binding as B
    moe.lib()
    dev, E, R, guard, d, F = "cuda:0", len(n), sum(n), 300, 2880, 4160      # 22.5 and 32.5 tiles of 128 features
    print(f"[streamed tile store] rows {n} packed={packed} variants {gu}, {dn}", flush=True)
    h_streamed = set(range(E)) if packed else {e for e in range(E) if n[e] <= 160}
    assert _streamed(B, True, 1, F, d, n, M or 256, packed, half) == h_streamed
    assert _streamed(B, False, ib, d, F, n, M or 256, packed, half) == set(range(E))
    g = torch.Generator(device=dev).manual_seed(R)
    rnd = lambda *s, std=1.0: torch.empty(s, dtype=torch.bfloat16, device=dev).normal_(generator=g).mul_(std)
    x = rnd(R, d)
    w = rnd(E, F, d, std=d ** -0.5), rnd(E, F, d, std=d ** -0.5), rnd(E, d, F, std=F ** -0.5)
    off = torch.tensor(np.concatenate([[0], np.cumsum(n)]), dtype=torch.int32, device=dev)
    cfg = moe.MoEConfig.of(R, d, F, E, 1, tile_m=M)
    p = None
    if packed:
        p = torch.empty(moe.packed_weights_size(cfg), dtype=torch.uint8, device=dev)
        moe.moe_pack_weights(cfg, *w, p)
    ws = torch.empty(moe.ffn_workspace_size(cfg), dtype=torch.uint8, device=dev)
    h = torch.full((R + guard, F), 7.0, dtype=torch.bfloat16, device=dev)
    y = torch.full((R + guard, d), 7.0, dtype=torch.bfloat16, device=dev)
    try:
        B.test_knob(B.KNOB_GATE_UP_VARIANT, gu)
        B.test_knob(B.KNOB_DOWN_VARIANT, dn)
        moe.moe_grouped_ffn(cfg, x, off, *((None, None, None) if packed else w), h[:R], y[:R], ws, W_packed=p)
        torch.cuda.synchronize()
    finally:
        B.test_knob(B.KNOB_GATE_UP_VARIANT, -1)
        B.test_knob(B.KNOB_DOWN_VARIANT, -1)
    assert bool((h[R:] == 7.0).all()) and bool((y[R:] == 7.0).all())
    for e in range(E):
        rows = slice(sum(n[:e]), sum(n[:e + 1]))
        xe = x[rows].double()
        rh = torch.nn.functional.silu(xe @ w[0][e].double().t()) * (xe @ w[1][e].double().t())
        ry = rh @ w[2][e].double().t()
        # bf16 results of fp32 sums, y_perm through a bf16 h: the bound that the parity tests state
        assert float((h[rows].double() - rh).abs().max()) <= 1e-2 * float(rh.abs().max()), f"h of expert {e}"
        assert float((y[rows].double() - ry).abs().max()) <= 1e-2 * float(ry.abs().max()), f"y_perm of expert {e}"


@pytest.mark.parametrize("below", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15])
def test_combine_on_both_sides_of_its_line(k, below):
    """Rows pass the caches by from T * k * d = 2^26 on.  An fp32 sum of k products is off by at most (k + 1) 2^-24 sum|w y|, and one
    rounding to bf16 by half a unit in the last place (2^-8)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    moe.lib()
    dev, d = "cuda:0", 2112                                # a second pass of the workgroup over 64 features
    T = -(-(1 << 26) // (k * d)) - below
    assert (T * k * d >= 1 << 26) != below
    print(f"[streamed combine] k={k} T={T}", flush=True)
    g = torch.Generator(device=dev).manual_seed(k)
    yp = torch.empty((T * k, d), dtype=torch.bfloat16, device=dev).normal_(generator=g)
    w = torch.rand((T, k), generator=g, device=dev)
    row_of = torch.randperm(T * k, generator=g, device=dev).to(torch.int32)
    y = torch.full((T + 2, d), float("nan"), dtype=torch.bfloat16, device=dev)
    moe.moe_combine(moe.MoEConfig.of(T, d, 64, 32, k), yp, row_of, w, y[:T])
    torch.cuda.synchronize()
    assert bool(y[T:].isnan().all())
    for a in range(0, T, 4096):
        wa = w[a:a + 4096]
        terms = wa.double()[:, :, None] * yp[row_of.long().view(T, k)[a:a + 4096].reshape(-1)].double().view(len(wa), k, d)
        ref = terms.sum(1)
        bound = 2.0 ** -8 * ref.abs() + (k + 1) * 2.0 ** -24 * terms.abs().sum(1) + 1e-30
        assert float(((y[a:a + 4096][:len(wa)].double() - ref).abs() / bound).max()) <= 1.0
