"""What the router costs hangs neither on the data nor on the row length: calls on which the int8 form's digits say less than usual, or logits are equal, against
the same call on normal activations.  The bound is on the ratio of the two (medians of interleaved rounds in one process): a
token whose E logits are all computed again by one wavefront takes 13 times as long as the whole call.  And calls on long rows
against the all-fp64 form of the same call."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T, D, E, K = 1024, 7168, 256, 8


def _zero_tokens(x, wr, bias):
    x[5::200] = 0.0


def _padded_half(x, wr, bias):
    x[T // 2:] = 0.0


def _zero_router(x, wr, bias):
    wr[:] = 0.0


def _few_experts_left(x, wr, bias):
    bias[3:] = -float("inf")      # fewer than k


def _channel_of_thousands(x, wr, bias):
    x[:, 17] *= 1000.0


def _heavy_tails(x, wr, bias):
    x *= torch.exp(1.5 * torch.randn(x.shape, generator=torch.Generator(device=DEV).manual_seed(2), device=DEV))


def _one_large_element(x, wr, bias):
    x[5, 17] = 1000.0


def _large_router_element(x, wr, bias):
    wr[3, 5] = 1000.0


def _infinity_and_nan(x, wr, bias):
    x[700, 3], wr[3, 5] = float("inf"), float("nan")


def _time(moe, cfg, x, wr, bias):
    idx, w = torch.empty((cfg.T, cfg.k), dtype=torch.int32, device=DEV), torch.empty((cfg.T, cfg.k), device=DEV)
    ws = torch.empty(moe.route_workspace_size(cfg), dtype=torch.uint8, device=DEV)

    def once():
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            moe.moe_route(cfg, x, wr, bias, idx, w, ws)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b)

    once()
    return once


def _medians(runs):
    rounds = [[f() for f in runs] for _ in range(9)]
    return [sorted(r[i] for r in rounds)[4] for i in range(len(runs))]


@pytest.mark.parametrize("change,gating,most", [(_zero_tokens, 0, 1.2), (_padded_half, 0, 1.2), (_zero_router, 0, 1.2), (_few_experts_left, 0, 1.2),
                                                (_channel_of_thousands, 0, 2.2), (_channel_of_thousands, 1, 2.2), (_heavy_tails, 0, 2.2), (_heavy_tails, 2, 2.2),
                                                (_one_large_element, 0, 2.2), (_large_router_element, 0, 2.2), (_infinity_and_nan, 1, 2.2)])
def test_cost(change, gating, most):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    moe.lib()
    print(f"[router cost] {change.__name__} gating={gating}", flush=True)
    cfg = moe.MoEConfig.of(T, D, 64, E, K, gating)
    g = torch.Generator(device=DEV).manual_seed(1)
    x, wr, bias = torch.randn(T, D, generator=g, device=DEV), torch.randn(E, D, generator=g, device=DEV) * D ** -0.5, torch.zeros(E, device=DEV)
    x1, wr1, bias1 = x.clone(), wr.clone(), bias.clone()
    change(x1, wr1, bias1)
    runs = [_time(moe, cfg, a.to(torch.bfloat16), b.to(torch.bfloat16), c) for a, b, c in ((x, wr, bias), (x1, wr1, bias1))]
    usual, changed = _medians(runs)
    print(f"  {usual * 200:.1f} us, changed {changed * 200:.1f} us", flush=True)
    assert changed <= most * usual


@pytest.mark.parametrize("T,d,E,k,most", [(8192, 32832, 64, 4, 0.8), (2048, 32832, 256, 8, 0.6), (128, 32768, 256, 8, 1.1), (129, 32768, 160, 4, 1.1)])
def test_long_rows(T, d, E, k, most):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    import paper_2605_23911_amd.binding as B
    moe.lib()
    print(f"[router cost] T={T} d={d} E={E}", flush=True)
    cfg = moe.MoEConfig.of(T, d, 64, E, k, 0)
    g = torch.Generator(device=DEV).manual_seed(1)
    x, wr = ((torch.randn(n, d, generator=g, device=DEV) * std).to(torch.bfloat16) for n, std in ((T, 1.0), (E, d ** -0.5)))
    run = _time(moe, cfg, x, wr, None)

    def in_fp64():
        B.test_knob(B.KNOB_ROUTE_EXACT, 1)
        try:
            return run()
        finally:
            B.test_knob(B.KNOB_ROUTE_EXACT, -1)

    ruled, fp64 = _medians([run, in_fp64])
    print(f"  {ruled * 200:.1f} us, all in fp64 {fp64 * 200:.1f} us", flush=True)
    assert ruled <= most * fp64
