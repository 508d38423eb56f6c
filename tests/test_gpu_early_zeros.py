"""Long lists whose pass writes the zeros of what it takes for selected: positions, values, u and v bit for bit against the
method's definition in torch, where the guess holds, where it is off on either side, and where the selection falls back."""
import pytest
import torch

pytestmark = pytest.mark.gpu
N, K, NODES, MOMENTUM = 16_000_003, 320_000, 8, 0.9      # 20 selected a row, records of 24; the last row is short


@pytest.fixture(scope="module")
def B():
    from paper_2103_08870_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def top(v, k):
    """Positions of the k largest magnitudes, lowest positions first among equals, ascending."""
    key = v.view(torch.int32) & 0x7FFFFFFF
    bar = key.topk(k).values[-1]
    above, equal = (key > bar).nonzero()[:, 0], (key == bar).nonzero()[:, 0]
    return torch.cat([above, equal[:k - above.numel()]]).sort().values


def gradient(kind, gen):
    g = torch.randn((NODES, N), generator=gen, device="cuda") * 1e-3
    if kind == "ties":            # a handful of magnitudes: the cut falls into thousands of equal ones
        g = torch.round(g * 4e3) / 4e3
    elif kind == "stretches":     # whole rows of large values, which no record holds, among rows of few
        g[:, 1_000_000:1_100_000] *= 50
        g[:, -500:] *= 50
    elif kind == "beyond":        # a few more large values than are selected: T* lies beyond the histogram above the estimate
        for b in range(NODES):
            g[b, torch.randperm(N, generator=gen, device="cuda")[:K + 200]] += 10
    elif kind == "special":
        for i, x in enumerate((float("inf"), -float("inf"), float("nan"), -0.0, 1e-42)):
            g[:, 10 + i::100_003 + i] = x
    return g


# the factor each iteration's gradients are scaled by: steady (carried thresholds), then jumps that put T* far above and below
# the expected one
@pytest.mark.parametrize("kind,factors,falls_back", [("spread", [1] * 9, False), ("spread", [1] * 70 + [1.02, 0.97, 1, 6, 1 / 50, 1], None),
                                                     ("beyond", [1, 1], True), ("ties", [1, 1, 1], None), ("stretches", [1] * 7, False), ("special", [1, 1, 1], None)])
def test_selection_with_zeros_from_the_pass(B, kind, factors, falls_back):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(factors))
    ctx = B.Context(N, K, NODES)
    B.lgc_set_option(ctx, B.LGC_OPT_SELECT_PATH, 2)
    u, v = torch.zeros((NODES, N), device="cuda"), torch.zeros((NODES, N), device="cuda")
    ru, rv = u.clone(), v.clone()
    vals = torch.empty((NODES, K), device="cuda")
    idx = torch.empty((NODES, K), dtype=torch.int32, device="cuda")
    common = gradient(kind, gen)
    for t, f in enumerate(factors):
        g = (common + 0.3 * gradient("spread", gen)) * f if len(factors) > 20 else common * f
        B.lgc_accumulate_topk(ctx, g, u, v, MOMENTUM, K, vals, idx)
        ru.mul_(MOMENTUM).add_(g)
        rv.add_(ru)
        for b in range(NODES):
            want = top(rv[b], K)
            assert torch.equal(idx[b].long(), want), (t, b)
            assert torch.equal(vals[b].view(torch.int32), rv[b][want].view(torch.int32)), (t, b)
            rv[b][want] = 0
            ru[b][want] = 0
            for x, y in ((u, ru), (v, rv)):
                assert torch.equal(x[b].nan_to_num(7.0).view(torch.int32), y[b].nan_to_num(7.0).view(torch.int32)), (t, b)
    fast, fallback, errors = B.lgc_stats(ctx)
    assert errors == 0 and fast + fallback == NODES * len(factors)
    assert falls_back is None or (fallback > 0) == falls_back, (fast, fallback)
    assert len(factors) < 70 or B.lgc_stats_carried(ctx) > 0
