"""Long lists whose pass may write the zeros of what it takes for selected: positions, values, u and v bit for bit against the
method's definition in torch.

It does so from a node's second selection on, if few rows of the one before held more candidates than a record.  Dense lists (20 selected a row) have
too many such rows: the first test is about rows with and without records side by side, and the change from one to the other.  The tests after it
select 10 a row, which makes zeros pay, and check by the rule that it does: zeros from a sampled and from a carried threshold, where the guess holds,
where it is off on either side, beside ties, infinities and NaN, and where the selection falls back and everything is written back."""
import pytest
import torch

from selection import top

pytestmark = pytest.mark.gpu
N, K, NODES, MOMENTUM = 16_000_003, 320_000, 8, 0.9      # 20 selected a row, records of 24; the last row is short
LONG, RECORD, ROW = 32_000_003, 24, 1024                 # 10 selected a row; the last row is short


@pytest.fixture(scope="module")
def B():
    from paper_2103_08870_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def gradient(kind, gen, n=N):
    g = torch.randn((NODES, n), generator=gen, device="cuda") * 1e-3
    if kind == "ties":            # a handful of magnitudes: the cut falls into thousands of equal ones
        g = torch.round(g * 4e3) / 4e3
    elif kind == "levels":        # more magnitudes, of which the list holds those around the cut
        g = torch.round(g * 4e4) / 4e4
    elif kind == "stretches":     # whole rows of large values, which no record holds, among rows of few
        g[:, 1_000_000:1_100_000] *= 50
        g[:, -500:] *= 50
    elif kind == "beyond":        # a few more large values than are selected: T* lies beyond the histogram above the estimate
        for b in range(NODES):
            g[b, torch.randperm(n, generator=gen, device="cuda")[:K + 200]] += 10
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


class Run:
    """One context's accumulate + top-k beside its definition, on residuals that make zeros from the pass pay."""

    def __init__(self, B):
        self.B, self.ctx = B, B.Context(LONG, K, NODES)
        B.lgc_set_option(self.ctx, B.LGC_OPT_SELECT_PATH, 2)
        self.u, self.v = torch.zeros((NODES, LONG), device="cuda"), torch.zeros((NODES, LONG), device="cuda")
        self.vals = torch.empty((NODES, K), device="cuda")
        self.idx = torch.empty((NODES, K), dtype=torch.int32, device="cuda")
        self.pays = False       # whether the selection before leaves zeros to the next one's pass: it was served, and its rows say so

    def select(self, g):
        """(nodes served, nodes that fell back, of all: carried thresholds)"""
        self.B.lgc_accumulate_topk(self.ctx, g, self.u, self.v, MOMENTUM, K, self.vals, self.idx)
        carried = self.B.lgc_stats_carried(self.ctx)
        fast, fallback, errors = self.B.lgc_stats(self.ctx)
        assert errors == 0 and fast + fallback == NODES
        return fast, fallback, carried

    def step(self, g):
        ru, rv = self.u * MOMENTUM + g, self.v.clone()
        rv.add_(ru)
        outcome = self.select(g)
        self.pays = outcome[1] == 0
        self.bars = []
        for b in range(NODES):
            key = rv[b].view(torch.int32) & 0x7FFFFFFF
            # the rule, at half as many candidates again as are selected (a sample lists a quarter more): 64 candidates in records pay for a crowded row
            rows = torch.nn.functional.pad(key >= key.topk(K + K // 2).values[-1], (0, -LONG % ROW)).view(-1, ROW).sum(dim=1)
            self.pays &= int(rows[rows <= RECORD].sum()) >= 128 * int((rows > RECORD).sum())
            want = top(rv[b], K)
            self.bars.append(float(rv[b][want].abs().min()))
            assert torch.equal(self.idx[b].long(), want), b
            assert torch.equal(self.vals[b].view(torch.int32), rv[b][want].view(torch.int32)), b
            rv[b][want] = 0
            ru[b][want] = 0
            for x, y in ((self.u, ru), (self.v, rv)):
                assert torch.equal(x[b].nan_to_num(7.0).view(torch.int32), y[b].nan_to_num(7.0).view(torch.int32)), b
        return outcome


@pytest.mark.parametrize("kind", ["spread", "levels", "stretches", "special"])
def test_zeros_from_a_sampled_threshold(B, kind):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(kind))
    run, g = Run(B), gradient(kind, gen, LONG)
    for t in range(5):
        outcome = run.step(g)
        assert outcome == (NODES, 0, 0) and run.pays, (t, outcome, run.pays)


@pytest.mark.parametrize("spikes", [K - 3000, K + 200, K + 3000])
def test_what_the_pass_has_zeroed_is_written_back_where_the_selection_falls_back(B, spikes):
    # T* far above the sampled threshold (beyond the histogram), or among many more values far below; the zeros' threshold on either side of the spikes' edge
    gen = torch.Generator(device="cuda")
    gen.manual_seed(spikes)
    run, g = Run(B), gradient("spread", gen, LONG)
    for _ in range(2):
        assert run.step(g) == (NODES, 0, 0) and run.pays
    for b in range(NODES):
        g[b, torch.randperm(LONG, generator=gen, device="cuda")[:spikes]] += 10
    assert run.step(g)[1] == (0 if spikes < K else NODES)
    g = gradient("spread", gen, LONG)
    for _ in range(3):
        run.step(g)


@pytest.mark.parametrize("jump", [0.0, 0.05, -0.6])
def test_zeros_from_a_carried_threshold(B, jump):
    # selections from fixed residuals: T* falls smoothly.  Then the residuals stay, grow by a twentieth (more candidates than the list holds), or shrink by
    # part of what T* falls from one selection to the next (fewer than k above the carried threshold, some of them above the zeros')
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    run = Run(B)
    run.v.normal_(generator=gen).mul_(1e-3)
    still = torch.zeros_like(run.v)
    row = 0
    for _ in range(40):
        row = row + 1 if run.select(still) == (NODES, 0, NODES) else 0
        if row == 3:
            break
    assert row == 3
    for _ in range(2):
        before = getattr(run, "bars", None)
        assert run.step(run.v * 1e-5) == (NODES, 0, NODES) and run.pays
    falls = max(1 - x / y for x, y in zip(run.bars, before))
    g = run.v * (jump if jump >= 0 else jump * falls)
    after = run.u.mul(MOMENTUM).add_(g).add_(run.v).abs_()
    expected = [x * x / y for x, y in zip(run.bars, before)]     # T*, on the line through the last two
    above = [int((after[b] >= expected[b]).sum()) for b in range(NODES)]
    assert min(above) > K // 10 and (jump >= 0 or max(above) < K), above
    outcome = run.step(g)
    assert outcome == ((NODES, 0, NODES) if jump == 0 else (0, NODES, NODES))
    for _ in range(2):
        run.step(run.v * 1e-5)
