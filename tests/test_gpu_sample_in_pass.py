"""Candidate thresholds that the pass finds itself (one launch, in a run of carried thresholds) or a launch before it: either side of the
line, nodes that carry a threshold beside nodes that sample, several contexts sampling at the same time, and waits that
expire.  Bit for bit against the definition in torch.

A pass samples by itself where a run of carried thresholds ends unseen by the host: the tests carry thresholds through a run longer than
the host asks for, hold the stream up, and queue a selection whose residuals jump and one after it.  That one has no offer and
goes through the pass all the same, as the host knows nothing of the jump.  Every case also runs on the library with a bound on the pass's waits that
expires at once (liblgc_short_wait.so), where the exact path serves the nodes that would sample: that it does shows that the
pass was to sample."""
import copy
import importlib.util
import os

import pytest
import torch

from selection import top

pytestmark = pytest.mark.gpu
ONE_LAUNCH = 104 * 1024 * 1024      # elements of all nodes, in rows of 1024
RUN = 16                            # selections in a row, per node, that must have left carried thresholds


def library(name):
    from paper_2103_08870_amd import binding
    if name == "liblgc.so":
        return binding
    spec = importlib.util.spec_from_file_location("binding_of_" + name.split(".")[0], binding.__file__)
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    b.LIB_PATH = os.path.join(os.path.dirname(binding.LIB_PATH), name)
    return b


@pytest.fixture(scope="module", params=["liblgc.so", "liblgc_short_wait.so"])
def B(request):
    b = library(request.param)
    b.lib()
    b.expires = request.param != "liblgc.so"
    assert torch.cuda.is_available()
    return b


class Run:
    """One context's accumulate + top-k beside its definition."""

    def __init__(self, B, n, k, nodes):
        self.B, self.n, self.k, self.nodes = B, n, k, nodes
        self.ctx = B.Context(n, k + 1, nodes)
        B.lgc_set_option(self.ctx, B.LGC_OPT_SELECT_PATH, 2)
        self.u, self.v = torch.zeros((nodes, n), device="cuda"), torch.zeros((nodes, n), device="cuda")
        self.ru = self.u.clone()
        self.still = torch.zeros_like(self.u)

    def step(self, g):
        vals = torch.empty((self.nodes, self.k), device="cuda")
        idx = torch.empty((self.nodes, self.k), dtype=torch.int32, device="cuda")
        self.B.lgc_accumulate_topk(self.ctx, g, self.u, self.v, 0.9, self.k, vals, idx)
        return vals, idx

    def carry(self, gen):
        """Selections from fixed residuals, one after the other, whose T* falls evenly: thresholds are carried, for more than a run."""
        for b in range(self.nodes):
            at = torch.randperm(self.n, generator=gen, device="cuda").double()
            self.v[b] = torch.exp(at * (-4 / self.n)) * (1 - 2 * (at % 2))
        row = 0
        run = RUN * self.nodes
        for _ in range(run + 64):
            before = self.B.lgc_stats_carried(self.ctx)
            self.step(self.still)
            row = row + 1 if self.B.lgc_stats_carried(self.ctx) - before == self.nodes else 0
            if row == run + 1:
                break
        assert row == run + 1, row
        self.B.lgc_stats(self.ctx)                # (counts anew)
        self.ru.copy_(self.u)
        self.rv = self.v.clone()

    def first(self, nodes):
        """The first nodes of this run, as a run on the same context."""
        part = copy.copy(self)
        part.nodes = nodes
        part.u, part.v, part.ru, part.still = (x[:nodes] for x in (self.u, self.v, self.ru, self.still))
        return part

    def jump(self, nodes):
        """Gradients that put these nodes' residuals a tenth lower: nothing lies above the carried threshold, the exact path serves them and leaves none."""
        self.grads = torch.zeros_like(self.v), self.still
        for b in nodes:
            torch.mul(self.v[b], -0.1, out=self.grads[0][b])

    def unseen(self):
        """Queues the selection that jumps and the next one on a stream held up meanwhile."""
        torch.cuda._sleep(40_000_000)
        held = torch.cuda.Event()
        held.record()
        self.queued = [(g, *self.step(g)) for g in self.grads]
        assert not held.query()

    def check(self):
        for g, vals, idx in self.queued:
            self.ru.mul_(0.9).add_(g)
            self.rv.add_(self.ru)
            for b in range(self.nodes):
                want = top(self.rv[b], self.k)
                assert torch.equal(idx[b].long(), want)
                assert torch.equal(vals[b], self.rv[b][want])
                self.rv[b][want] = 0
                self.ru[b][want] = 0
        assert torch.equal(self.u, self.ru) and torch.equal(self.v, self.rv)


def generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


# the shortest vector that is sampled; fewer blocks per node than shares; a short last row; either side of the line
@pytest.mark.parametrize("n,k,nodes", [(1 << 18, 300, 1), ((1 << 18) + 1, 300, 3), (1_000_001, 1000, 2), (3_333_331, 3333, 3), (ONE_LAUNCH, 100_000, 1),
                                       (ONE_LAUNCH + 1, 100_000, 1), (ONE_LAUNCH // 4, 20_000, 4), (ONE_LAUNCH // 4 + 1, 20_000, 4)])
def test_sampled_thresholds(B, n, k, nodes):
    run = Run(B, n, k, nodes)
    run.carry(generator(n))
    run.jump(range(nodes))
    run.unseen()
    run.check()
    in_pass = n * nodes <= ONE_LAUNCH and B.expires
    assert B.lgc_stats_carried(run.ctx) == nodes
    assert B.lgc_stats(run.ctx) == ((0, 2 * nodes, 0) if in_pass else (nodes, nodes, 0))


@pytest.mark.parametrize("jumps", [[0], [1], [0, 2], [1, 2]])
def test_nodes_that_sample_beside_nodes_that_carry(B, jumps):
    n, k, nodes = 2_000_001, 2000, 3
    run = Run(B, n, k, nodes)
    run.carry(generator(6))
    run.jump(jumps)
    run.unseen()
    run.check()
    expired = len(jumps) if B.expires else 0
    assert B.lgc_stats_carried(run.ctx) == 2 * nodes - len(jumps)
    assert B.lgc_stats(run.ctx) == (2 * nodes - len(jumps) - expired, len(jumps) + expired, 0)


def test_a_graph_recorded_in_a_run_of_carried_thresholds(B):
    # a launch samples in what was recorded, whatever it finds when it is replayed: no wait that could expire
    run = Run(B, 2_000_001, 2000, 2)
    run.carry(generator(8))
    g = torch.zeros_like(run.v)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run.queued = [(g, *run.step(g)) for _ in range(2)]      # two: the scratch's two halves take turns
    for kind, stats in (("still", (4, 0, 0)), ("jump", (2, 2, 0)), ("still", None), ("jump", None), ("still", None)):
        torch.mul(run.v, -0.1 if kind == "jump" else 0.0, out=g)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        run.check()
        got = B.lgc_stats(run.ctx)
        assert got[2] == 0 and stats in (None, got), (kind, got)


@pytest.mark.parametrize("n,k,nodes", [((1 << 18) + 1, 3000, 3), (2_000_001, 2000, 3), (ONE_LAUNCH // 4, 20_000, 4), (ONE_LAUNCH // 4 + 1, 20_000, 4)])
def test_another_number_of_nodes_or_another_count(B, n, k, nodes):
    # right after a run of carried thresholds of the first node; the host knows that no offer is for these, and a launch samples
    run, gen = Run(B, n, k, nodes), generator(n)
    run.first(1).carry(gen)
    run.rv, run.ru = run.v.clone(), run.u.clone()
    for run.k, carried in ((k, 1), (k + 1, 0), (k + 1, 0)):
        g = torch.zeros_like(run.v)
        g[1:].normal_(generator=gen)
        run.queued = [(g, *run.step(g))]
        run.check()
        assert B.lgc_stats_carried(run.ctx) == carried
        assert B.lgc_stats(run.ctx) == (nodes, 0, 0)


def test_a_node_that_samples_beside_nodes_that_carry(B):
    n, nodes = 2_000_001, 3
    run, gen = Run(B, n, 2000, nodes), generator(5)
    run.rv = run.v.clone()
    common = torch.randn((nodes, n), generator=gen, device="cuda") * 1e-3
    carried = []
    for t in range(60):
        g = common + 3e-4 * torch.randn((nodes, n), generator=gen, device="cuda")
        if t == 50:
            g[1] *= 40.0                         # the threshold that node 1 carries no longer fits
        before = B.lgc_stats_carried(run.ctx)
        run.queued = [(g, *run.step(g))]
        run.check()
        carried.append(B.lgc_stats_carried(run.ctx) - before)
    assert max(carried) == nodes and carried[51] == nodes - 1, carried
    assert B.lgc_stats(run.ctx)[2] == 0


def test_contexts_that_sample_at_the_same_time(B):
    # eight selections on eight streams: every pass's blocks wait for shares that may be with blocks of others' passes in between
    n, k = 8_000_003, 8000
    runs, streams = [Run(B, n, k, 2) for _ in range(8)], [torch.cuda.Stream() for _ in range(8)]
    for seed, run in enumerate(runs):
        run.carry(generator(seed))
        run.jump([0, 1])
    torch.cuda.synchronize()
    for run, s in zip(runs, streams):
        with torch.cuda.stream(s):
            run.unseen()
    torch.cuda.synchronize()
    for run in runs:
        run.check()
        assert B.lgc_stats(run.ctx) == ((0, 4, 0) if B.expires else (2, 2, 0))
