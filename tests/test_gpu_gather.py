"""The list of candidates (flags of the pass -> positions and values in index order) where its parts have edges: groups of 128
rows, groups without candidates, sums per group (from 32 K rows on, and more of them than a block has threads), bitmap lines left out
(flat passes of several launches); flat and by layers.  Against the selection's definition in torch, bit for bit."""
import pytest
import torch

from selection import top

pytestmark = pytest.mark.gpu
GROUP = 128 * 1024       # elements per group of rows


@pytest.fixture(scope="module")
def B():
    from paper_2103_08870_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def vector(layout, n, k, gen):
    v = torch.randn(n, generator=gen, device="cuda") * 1e-3
    if layout == "stretch":       # one stretch holds all that is selected: many pieces of few groups, all other groups empty
        at = 3 * GROUP - k // 3
        v[at:at + k + 77].mul_(1e-1).add_(6e-3)   # (within the histogram's two octaves above the estimate, which lies among the others)
    elif layout == "edges":       # the elements on either side of every group's edge, and the vector's ends
        at = torch.arange(GROUP, n, GROUP, device="cuda")
        v[torch.cat([at, at - 1])] = 5.0
        v[0], v[n - 1] = 6.0, -6.0
    return v


def check(B, v, got_v, vals, idx, want):
    assert torch.equal(idx.long(), want)
    assert torch.equal(vals, v[want])
    v[want] = 0
    assert torch.equal(got_v, v)


@pytest.mark.parametrize("layout", ["spread", "stretch", "edges"])
@pytest.mark.parametrize("n,k,batch", [(2 * GROUP + 1, 6000, 1), (8 * GROUP, 9000, 2), (8 * GROUP - 1, 9001, 3),   # with records
                                       (33_600_001, 33_600, 1), (12_000_001, 40_000, 3),                           # without
                                       (33_600_001, 400_000, 1), (33_600_001, 150_000, 1), (33_600_001, 400_000, 2),   # dense groups as pieces
                                       (257 * GROUP, 30_000, 1), (813 * GROUP + 1, 100_000, 1), (1025 * GROUP - 5, 2_400_000, 1)])
def test_flat_selection(B, layout, n, k, batch):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + k)
    v = torch.stack([vector(layout, n, k, gen) for _ in range(batch)])
    got = v.clone()
    ctx = B.Context(n, k, batch)
    vals = torch.empty((batch, k), device="cuda")
    idx = torch.empty((batch, k), dtype=torch.int32, device="cuda")
    B.lgc_topk(ctx, got, None, k, vals, idx)
    for b in range(batch):
        check(B, v[b], got[b], vals[b], idx[b], top(v[b], k))
    assert B.lgc_stats(ctx) == (batch, 0, 0)


@pytest.mark.parametrize("n,cuts", [(3 * GROUP, [GROUP - 1, GROUP + 1, 2 * GROUP]), (4 * GROUP + 513, [100, GROUP, 2 * GROUP + 1024, 3 * GROUP + 1023]),
                                    (815 * GROUP, [256 * GROUP, 512 * GROUP + 5])])
@pytest.mark.parametrize("layout", ["spread", "stretch", "edges"])
def test_selection_by_layers(B, layout, n, cuts):
    # layers that start on, before and after the edges of groups and rows; rows and groups without candidates between them
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    bounds = [0, *cuts, n]
    ks = [max(1, (hi - lo) // 1000) for lo, hi in zip(bounds, bounds[1:])]
    v = vector(layout, n, sum(ks), gen)
    got = v.clone()
    ctx, seg = B.Context(n, sum(ks), 1), B.Segments(bounds, ks)
    B.lgc_reserve(ctx, None, 0, 0, seg)
    vals = torch.empty((1, sum(ks)), device="cuda")
    idx = torch.empty((1, sum(ks)), dtype=torch.int32, device="cuda")
    B.lgc_topk_segmented(ctx, seg, got[None], None, vals, idx)
    want = torch.cat([lo + top(v[lo:hi], k) for lo, hi, k in zip(bounds, bounds[1:], ks)])
    check(B, v, got, vals[0], idx[0], want)
    assert B.lgc_stats(ctx)[2] == 0
