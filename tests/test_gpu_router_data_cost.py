"""What the router costs does not hang on the data: calls on which the int8 form's digits say less than usual, or logits are equal, against
the same call on normal activations.  The bound is on the ratio of the two (medians of interleaved rounds in one process): a
token whose E logits are all computed again by one wavefront takes 13 times as long as the whole call."""
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
    idx, w = torch.empty((T, K), dtype=torch.int32, device=DEV), torch.empty((T, K), device=DEV)
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
    rounds = [[f() for f in runs] for _ in range(9)]
    usual, changed = (sorted(r[i] for r in rounds)[4] for i in (0, 1))
    print(f"  {usual * 200:.1f} us, changed {changed * 200:.1f} us", flush=True)
    assert changed <= most * usual
