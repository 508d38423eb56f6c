"""Candidate thresholds that the pass finds itself (one launch, in a run of carried thresholds) or a launch before it: either side of the
line, nodes that carry a threshold beside nodes that sample, several contexts sampling at the same time.  Bit for bit against the
definition in torch.

A pass samples by itself where a run of carried thresholds ends unseen by the host: the tests make one with one node and then
select another count, or from more nodes."""
import pytest
import torch

pytestmark = pytest.mark.gpu
ONE_LAUNCH = 104 * 1024 * 1024      # elements of all nodes, in rows of 1024


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


class Run:
    """One context's accumulate + top-k beside its definition."""

    def __init__(self, B, n, k, nodes):
        self.B, self.ctx = B, B.Context(n, k + 1, nodes)
        B.lgc_set_option(self.ctx, B.LGC_OPT_SELECT_PATH, 2)
        self.all_u, self.all_v = torch.zeros((nodes, n), device="cuda"), torch.zeros((nodes, n), device="cuda")
        self.all_ru, self.all_rv = self.all_u.clone(), self.all_v.clone()
        self.select(k, nodes)

    def select(self, k, nodes):
        self.k, self.nodes = k, nodes
        self.u, self.v, self.ru, self.rv = (x[:nodes] for x in (self.all_u, self.all_v, self.all_ru, self.all_rv))
        self.vals = torch.empty((nodes, k), device="cuda")
        self.idx = torch.empty((nodes, k), dtype=torch.int32, device="cuda")

    def carry(self, gen):
        """Selections from the first node's fixed residuals, one after the other: T* falls smoothly, thresholds are carried."""
        k, nodes = self.k, self.nodes
        self.select(k, 1)
        self.v.normal_(generator=gen).mul_(1e-3)
        self.rv.copy_(self.v)
        g = torch.zeros_like(self.v)
        for _ in range(26):
            self.step(g)
            self.check(g)
            last = self.B.lgc_stats_carried(self.ctx)
        assert last == 1 and self.B.lgc_stats(self.ctx) == (26, 0, 0)
        self.select(k, nodes)

    def step(self, g):
        self.B.lgc_accumulate_topk(self.ctx, g, self.u, self.v, 0.9, self.k, self.vals, self.idx)

    def check(self, g):
        self.ru.mul_(0.9).add_(g)
        self.rv.add_(self.ru)
        for b in range(self.nodes):
            want = top(self.rv[b], self.k)
            assert torch.equal(self.idx[b].long(), want)
            assert torch.equal(self.vals[b], self.rv[b][want])
            self.rv[b][want] = 0
            self.ru[b][want] = 0
        assert torch.equal(self.u, self.ru) and torch.equal(self.v, self.rv)


def generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


# the shortest vector that is sampled; fewer blocks per node than shares; a short last row; either side of the line
@pytest.mark.parametrize("n,k,nodes", [(1 << 18, 300, 1), ((1 << 18) + 1, 3000, 3), (1_000_001, 20_000, 2), (ONE_LAUNCH, 100_000, 1),
                                       (ONE_LAUNCH + 1, 100_000, 1), (ONE_LAUNCH // 4, 20_000, 4), (ONE_LAUNCH // 4 + 1, 20_000, 4)])
def test_sampled_thresholds(B, n, k, nodes):
    run, gen = Run(B, n, k, nodes), generator(n)
    run.carry(gen)
    run.select(k + 1, nodes)
    for _ in range(2):      # the pass's own sample, and a launch's
        g = torch.randn((nodes, n), generator=gen, device="cuda") * 1e-3
        run.step(g)
        run.check(g)
    assert B.lgc_stats(run.ctx) == (2 * nodes, 0, 0)
    assert B.lgc_stats_carried(run.ctx) == 0


def test_nodes_that_sample_beside_one_that_carries(B):
    n, nodes = 2_000_001, 3
    run, gen = Run(B, n, 2000, nodes), generator(6)
    run.carry(gen)
    g = torch.zeros((nodes, n), device="cuda")
    g[1:].normal_(generator=gen)
    run.step(g)
    run.check(g)
    assert B.lgc_stats_carried(run.ctx) == 1
    assert B.lgc_stats(run.ctx) == (nodes, 0, 0)


def test_a_node_that_samples_beside_nodes_that_carry(B):
    n, nodes = 2_000_001, 3
    run, gen = Run(B, n, 2000, nodes), generator(5)
    common = torch.randn((nodes, n), generator=gen, device="cuda") * 1e-3
    carried = []
    for t in range(60):
        g = common + 3e-4 * torch.randn((nodes, n), generator=gen, device="cuda")
        if t == 50:
            g[1] *= 40.0                         # the threshold that node 1 carries no longer fits
        before = B.lgc_stats_carried(run.ctx)
        run.step(g)
        run.check(g)
        carried.append(B.lgc_stats_carried(run.ctx) - before)
    assert max(carried) == nodes and carried[51] == nodes - 1, carried
    assert B.lgc_stats(run.ctx)[2] == 0


def test_contexts_that_sample_at_the_same_time(B):
    # eight selections on eight streams: every pass's blocks wait for shares that may be with blocks of others' passes in between
    n, k = 8_000_003, 8000
    gens = [generator(s) for s in range(8)]
    runs = [Run(B, n, k, 2) for _ in gens]
    grads = [torch.randn((2, n), generator=gen, device="cuda") * 1e-3 for gen in gens]
    for run, gen in zip(runs, gens):
        run.carry(gen)
        run.select(k + 1, 2)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in runs]
    for _ in range(2):
        for run, g, s in zip(runs, grads, streams):
            with torch.cuda.stream(s):
                run.step(g)
        torch.cuda.synchronize()
        for run, g in zip(runs, grads):
            run.check(g)
        torch.cuda.synchronize()
    assert all(B.lgc_stats(run.ctx) == (4, 0, 0) for run in runs)
