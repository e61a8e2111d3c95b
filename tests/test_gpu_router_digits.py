"""The router's int8 form (rows cut into four 8-bit digits, products summed in integers) forced on, against float64 by torch: tiles and
slices with remainders, rows longer than one pass of the digit kernel, ranges at which the fixed point loses elements, logits
that differ by less than the digits resolve, and values that are not finite.  The digits' kernel gives a row a workgroup up to 2200 padded rows and
a wavefront beyond: the cases of 2305 tokens (a padded tile of one token) are there for the second.

Bound on a weight, relative: one rounding to fp32 (2^-24) plus twice the logits' error (the weight's own logit and the sum below it),
which is at most 2^-25 (beyond, they are formed in fp64): 2^-23."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture
def moe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_23911_amd as moe
    import paper_2605_23911_amd.binding as B
    moe.lib()
    B.test_knob(B.KNOB_ROUTE_EXACT, 0)
    yield moe
    B.test_knob(B.KNOB_ROUTE_EXACT, -1)


def _rows(T, d, E, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(T, d, generator=g), torch.randn(E, d, generator=g) * d ** -0.5


def _route(moe, x, wr, k, gating, bias=None):
    T, d = x.shape
    cfg = moe.MoEConfig.of(T, d, 64, wr.shape[0], k, gating)
    idx = torch.full((T, k), -1, dtype=torch.int32, device=DEV)
    w = torch.full((T, k), float("nan"), device=DEV)
    ws = torch.full((moe.route_workspace_size(cfg),), 0xFF, dtype=torch.uint8, device=DEV)
    moe.moe_route(cfg, x, wr, bias, idx, w, ws)
    torch.cuda.synchronize()
    return idx.long(), w.double()


def _parts(v):
    """Per row: the largest magnitude, bounds of the 2-norms of the third and fourth digit's parts and of the sum of the residuals."""
    v = v.to(torch.bfloat16).double()
    a = v.abs().amax(1)
    unit = 2.0 ** (torch.floor(torch.log2(a)) - 29)
    n = torch.trunc(v / unit[:, None])
    count = lambda m: m.sum(1).double()
    return a, 33000 * unit * count(n % 65536 != 0).sqrt(), 128.2 * unit * count(n % 256 != 0).sqrt(), unit * count(n * unit[:, None] != v)


def _check(moe, x, wr, k, gating, gap_min, tol=2.0 ** -23, scale=1.0):
    x, wr = x.to(torch.bfloat16).to(DEV), wr.to(torch.bfloat16).to(DEV)
    idx, w = _route(moe, x, wr, k, gating)
    z = x.double() @ wr.double().t()
    top, want = torch.topk(z, min(k + 1, z.shape[1]), dim=1)
    assert float((top[:, :-1] - top[:, 1:]).min()) > gap_min * scale    # certifies the order in float64
    top, want = top[:, :k], want[:, :k]
    assert torch.equal(idx, want)
    ref = {0: torch.exp(top - torch.logsumexp(z, 1, keepdim=True)), 1: torch.softmax(top, 1),
           2: torch.sigmoid(top) / torch.sigmoid(top).sum(1, keepdim=True)}[gating]
    error = ((w - ref).abs() / ref.clamp_min(1e-37)).max()      # below, fp32 itself has fewer bits
    print(f"  relative error {float(error):.3e}, {tol:.3e} allowed", flush=True)
    assert float(error) <= 1.001 * tol


@pytest.mark.parametrize("T,d,E,k", [(256, 64, 9, 2), (257, 128, 64, 8), (300, 192, 65, 4), (511, 2112, 128, 1), (289, 1088, 129, 8),
                                     (256, 8256, 256, 8), (383, 16448, 40, 3), (256, 32832, 65, 4), (300, 65600, 33, 2),
                                     (2305, 64, 9, 2), (2305, 192, 40, 8), (2305, 8256, 40, 4), (2305, 16448, 129, 2)])
@pytest.mark.parametrize("gating", [0, 1, 2])
def test_remainders(moe, T, d, E, k, gating):
    print(f"[digits] T={T} d={d} E={E} k={k} gating={gating}", flush=True)
    _check(moe, *_rows(T, d, E, T + E), k, gating, 1e-9)


@pytest.mark.parametrize("gating", [0, 1])
@pytest.mark.parametrize("i,j", [(i, j) for i in range(4) for j in range(4)])
@pytest.mark.parametrize("shift", [0, 4])
def test_every_pair_of_digits(moe, i, j, shift, gating):
    """Many elements that consist of one digit, i in the tokens and j in the experts, all of one sign: what a missing or misplaced product would take
    from a logit is far above the tolerance for i + j <= 4 (6.6e-6 for 4).  Of (2, 3) and (3, 2), which are left out, the bound is
    nearly reached: 2.6e-8 is just under 2^-25, with shift 4 4.2e-7 is to be formed in fp64."""
    print(f"[digits] pair {i}, {j} shift={shift} gating={gating}", flush=True)
    T, d, E, k = 300, 2048, 40, 6
    n, c = [(8, 1), (64, 8), (512, 32), (1792, 127), (1792, 127), (1792, 127), (1792, 127)][i + j]
    c0 = [min(c, 64), c, c, c]
    x, wr = torch.zeros(T, d), torch.zeros(E, d)
    x[:, 0], wr[:, 1] = 1.0, 1.0                                           # the largest of each row: units of 2^-29
    x[:, 2], wr[:, 2] = 0.5, 3 * torch.arange(E) / 128.0                   # logits 3/256 apart; the pairs add no multiple of that
    x[:, 128: 128 + n] = c0[i] * 2.0 ** (-5 - 8 * i)
    wr[1::2, 128: 128 + n] = c0[j] * 2.0 ** (-5 - 8 * j)
    _check(moe, x * 2.0 ** shift, wr, k, gating, 1e-9, tol=2.0 ** -24 if i + j < 5 else 2.0 ** -23)


@pytest.mark.parametrize("k", [5, 6])
@pytest.mark.parametrize("ahead", [2.0 ** -26, 2.0 ** -25, 2.0 ** -24])
def test_order_within_and_beyond_the_bound(moe, ahead, k):
    """Pairs of experts of which the second is larger by a sum of left-out products, 2.6e-8, and the first by `ahead`: in the digits'
    sums the first leads, in truth the second where `ahead` is 1.5e-8.  Beyond twice the bound, 5.3e-8, nothing is recomputed; inside the selection and
    across its boundary."""
    print(f"[digits] order, ahead {ahead} k={k}", flush=True)
    T, d, E, n = 300, 2048, 40, 1792
    x, wr = torch.zeros(T, d), torch.zeros(E, d)
    x[:, 0], wr[:, 1] = 1.0, 1.0
    x[:, 2], wr[:, 2] = 0.5, 3 * (torch.arange(E) // 2) / 128.0
    x[:, 3], wr[::2, 3] = 1.0, ahead
    x[:, 128: 128 + n], wr[1::2, 128: 128 + n] = 127 * 2.0 ** -21, 127 * 2.0 ** -29
    _check(moe, x, wr, k, 1, 1e-9)


@pytest.mark.parametrize("gating", [0, 1])
@pytest.mark.parametrize("tokens", [True, False])
@pytest.mark.parametrize("shift", [0, 4])
def test_residuals(moe, tokens, shift, gating):
    """Elements just below the fixed point's unit, of one sign, against the other side's largest: 15 units of 2^-29 are lost, 2.8e-8, and the
    bound is just under 2^-25; with shift 4 it is 4.5e-7, to be formed in fp64."""
    print(f"[digits] residuals of the {'tokens' if tokens else 'experts'} shift={shift} gating={gating}", flush=True)
    T, d, E, k = 300, 256, 40, 6
    x, wr = torch.zeros(T, d), torch.zeros(E, d)
    x[:, 0], wr[:, 1] = 1.0, 1.0
    x[:, 2], wr[:, 2] = 0.5, 3 * torch.arange(E) / 128.0
    small = 255 * 2.0 ** -37
    x[:, 128: 143] = small if tokens else 1.0
    wr[1::2, 128: 143] = 1.0 if tokens else small
    _check(moe, x * 2.0 ** shift, wr, k, gating, 1e-9)


def test_sums_of_long_rows(moe):
    """147456 products of 127 x 127 of one order: more than an int32 holds, a slice of d has to stay below."""
    print("[digits] long rows", flush=True)
    T, d, E, n = 256, 147584, 33, 147456
    x, wr = torch.zeros(T, d, dtype=torch.bfloat16), torch.zeros(E, d, dtype=torch.bfloat16)
    x[:, 0], wr[:, 1] = 1.0, 1.0
    x[:, 2], wr[:, 2] = 0.5, (3 * torch.arange(E) / 128.0).to(torch.bfloat16)
    x[:, 128:] = 127 * 2.0 ** -13
    wr[1::2, 128:] = 127 * 2.0 ** -21
    _check(moe, x, wr, 4, 0, 1e-9, tol=2.0 ** -24)


@pytest.mark.parametrize("outlier", [30.0, 300.0, 3000.0, 1e6])
@pytest.mark.parametrize("gating", [0, 1])
@pytest.mark.parametrize("T,E", [(260, 100), (2305, 100), (2305, 256)])
def test_outliers(moe, outlier, gating, T, E):
    """One element far above the others takes digits away from its row; at the larger ones the softmax has its tiles formed in fp64, the
    renormalised one its candidates.  From 2^19 logits on (the last size) the softmax has its candidates too, and the other experts' logits
    are as exact as the digits: twice their bound comes on top of the tolerance."""
    print(f"[digits] outlier {outlier} T={T} E={E} gating={gating}", flush=True)
    x, wr = _rows(T, 1024, E, 3)
    x[::2, 17] = outlier
    wr[:, 17] *= 1.0 / outlier
    wr[5, 400] = outlier * 1024 ** -0.5
    x[:, 400] *= 1.0 / outlier
    tol = 2.0 ** -23
    if gating == 0 and T * E >= 1 << 19:
        (ax, x2, x3, rx), (aw, w2, w3, rw) = _parts(x), _parts(wr)
        tol += 2 * float((x2[:, None] * w3 + x3[:, None] * w2 + rx[:, None] * aw + ax[:, None] * rw).max())
    _check(moe, x, wr, 6, gating, 1e-10, tol)


@pytest.mark.parametrize("sx,sw", [(2.0 ** -100, 2.0 ** 100), (2.0 ** 90, 2.0 ** -90), (2.0 ** -60, 1.0), (2.0 ** -120, 2.0 ** 118)])
@pytest.mark.parametrize("T", [256, 2305])
def test_range_of_exponents(moe, sx, sw, T):
    print(f"[digits] scales {sx} {sw} T={T}", flush=True)
    x, wr = _rows(T, 512, 70, 7)
    _check(moe, x * sx, wr * sw, 4, 1, 1e-9, scale=sx * sw)


def test_logits_closer_than_the_digits_resolve(moe):
    """Pairs of router rows that differ in one element so small that its last bits lie below the fixed point, in both
    orders, inside the selection and across its boundary."""
    print("[digits] near ties", flush=True)
    x, wr = _rows(400, 256, 40, 11)
    x[:, 9] = x[:, 9].sign() * (x[:, 9].abs() + 0.5)
    wr[:, 9] = 0.0
    for a, b in [(0, 20), (21, 1), (2, 22), (23, 3)]:
        wr[b] = wr[a]
        wr[a, 9] = 2.0 ** -30
        wr[b, 9] = 2.0 ** -30 * (1 + 2.0 ** -7)
    _check(moe, x, wr, 5, 0, 1e-13)


@pytest.mark.parametrize("T", [300, 2305])
def test_infinities_and_nans(moe, T):
    """A NaN logit never wins; tokens and experts without one are as without its neighbours' (whose tile is then formed in fp64:
    on normal rows the digits leave nothing that shows in a weight)."""
    print(f"[digits] infinities and NaN T={T}", flush=True)
    x, wr = _rows(T, 320, 50, 13)
    x, wr = x.to(torch.bfloat16), wr.to(torch.bfloat16)
    bad = x.clone()
    bad[3, 5], bad[4, 6], bad[5] = float("nan"), float("inf"), float("-inf")
    ok = torch.ones(T, dtype=torch.bool)
    ok[3:6] = False
    idx0, w0 = _route(moe, x.to(DEV), wr.to(DEV), 6, 0)
    idx, w = _route(moe, bad.to(DEV), wr.to(DEV), 6, 0)
    assert torch.equal(idx[ok], idx0[ok]) and torch.equal(w[ok], w0[ok])
    assert bool(((idx >= 0) & (idx < 50)).all())
    wbad = wr.clone()
    wbad[7, 3] = float("nan")
    idx, w = _route(moe, x.to(DEV), wbad.to(DEV), 6, 1)
    z = x.double() @ wbad.double().t()
    z[:, 7] = -float("inf")
    assert np.array_equal(idx.cpu().numpy(), torch.topk(z, 6, dim=1)[1].numpy())


def test_masked_experts(moe):
    """A bias of -inf masks experts: they come last, in index order."""
    print("[digits] masked experts", flush=True)
    x, wr = _rows(256, 128, 33, 17)
    x, wr = x.to(torch.bfloat16), wr.to(torch.bfloat16)
    bias = torch.zeros(33)
    bias[5:] = float("-inf")
    idx, w = _route(moe, x.to(DEV), wr.to(DEV), 8, 0, bias.to(DEV))
    z = x.double() @ wr.double().t() + bias.double()
    assert np.array_equal(idx[:, :5].cpu().numpy(), torch.topk(z, 5, dim=1)[1].numpy())
    assert np.array_equal(idx[:, 5:].cpu().numpy(), np.tile([5, 6, 7], (256, 1)))
    assert float((w[:, 5:]).abs().max()) == 0.0
