"""Exact top-k of short vectors (launches of their own) against the oracle: chunk and bitmap edges, ties through the cut,
more keys sharing the threshold's bin than the LDS list holds, odd row starts, both callers."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2103_08870_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def values(kind, rng, shape):
    if kind == "normal":
        return rng.normal(0, 1e-3, shape).astype(np.float32)
    if kind in ("few", "ties"):   # seven magnitudes, of which three are added up (few) or not (ties: the list overflows on long vectors)
        return (rng.integers(0, 7, shape) * rng.choice([-0.5, 0.5], shape)).astype(np.float32)
    if kind == "narrow":     # all keys share their leading bits, none are equal by design
        return (1.0 + rng.random(shape) * 0.1).astype(np.float32)
    if kind == "edges":      # a few units to either side of a magnitude where the bins' width changes
        at = np.uint32((67, 100, 135, 200)[shape[1] % 4] << 23) + rng.integers(0, 81, shape).astype(np.uint32) - np.uint32(40)
        return (at | (rng.integers(0, 2, shape).astype(np.uint32) << np.uint32(31))).view(np.float32)
    out = rng.normal(0, 1, shape).astype(np.float32)          # "special"
    flat = out.reshape(-1)
    for i, x in enumerate((np.inf, -np.inf, np.nan, 0.0, -0.0, 1e-42)):
        flat[i::11 + i] = x
    return out


def same(t, a):
    h = t.cpu().numpy()
    nan = np.isnan(a)
    return (np.isnan(h) == nan).all() and (h.view(np.uint32)[~nan] == a.view(np.uint32)[~nan]).all()


@pytest.mark.parametrize("kind", ["normal", "few", "narrow", "special", "ties", "edges"])
@pytest.mark.parametrize("n,k,batch,pad", [(1, 1, 1, 0), (3, 2, 3, 2), (4095, 4095 // 3, 2, 1), (4096, 1, 1, 0), (4097, 3072, 3, 0),
                                           (32_767, 300, 2, 2), (32_768, 3072, 1, 0), (32_769, 33, 2, 3), (100_003, 1000, 2, 1),
                                           (262_143, 2621, 1, 0), (262_143, 3073, 2, 1),
                                           # the longest selection of their own, and the first that goes to the radix path
                                           (262_143, 4096, 1, 0), (262_143, 4097, 1, 1), (8193, 4096, 2, 1), (8193, 4097, 1, 0)])
def test_short_vectors(B, oracle, kind, n, k, batch, pad):
    rng = np.random.default_rng(n + k)
    g, u, v = (values(kind, rng, (batch, n + pad)) for _ in range(3))
    if kind in ("ties", "edges"):
        g[:] = 0; u[:] = 0
    ctx = B.Context(n, k, batch)
    with np.errstate(all="ignore"):
        for b in range(batch):
            oracle.accumulate(g[b, :n], un := u[b, :n].copy(), vn := v[b, :n].copy(), 0.9)
            if b == 0:
                eu, ev, ei, eo = [], [], [], []
            key = vn.view(np.uint32) & 0x7fffffff
            listed = int((key >> 18 >= np.sort(key)[n - k] >> 18).sum())      # keys that share the threshold's bin (32 per octave) or lie above
            vals, idx = oracle.topk(vn, un, k)
            # which way the selection goes: 12 288 entries fit the list (lgc_stats does not count short vectors)
            assert n < 200_000 or kind == "special" or (listed > 12_288) == (kind in ("narrow", "ties", "edges")), listed
            eu.append(un); ev.append(vn); ei.append(idx); eo.append(vals)
    for call in ("context", "static", "pair", "radix"):
        dg, du, dv = (torch.from_numpy(a).cuda()[:, :n] for a in (g, u, v))
        ov = torch.zeros((batch, k), device="cuda")
        oi = torch.zeros((batch, k), dtype=torch.int32, device="cuda")
        if call == "static":
            B.lgc_accumulate_topk_static(dg, du, dv, 0.9, k, ov, oi)
        elif call == "pair":
            B.lgc_accumulate(ctx, dg, du, dv, 0.9)
            B.lgc_topk(ctx, dv, du, k, ov, oi)
        else:
            B.lgc_set_option(ctx, B.LGC_OPT_SELECT_PATH, 1 if call == "radix" else 0)
            B.lgc_accumulate_topk(ctx, dg, du, dv, 0.9, k, ov, oi)
        assert (oi.cpu().numpy().astype(np.uint32) == np.stack(ei)).all(), call
        assert same(ov, np.stack(eo)) and same(dv, np.stack(ev)) and same(du, np.stack(eu)), call
    assert B.lgc_stats(ctx)[2] == 0
    ctx.close()


def test_short_vectors_of_a_run_in_progress_take_no_longer_than_the_radix_path(B):
    # the residuals of a run in progress lie close below the threshold: what shares its leading bits has to fit one block's
    # list all the same (with 8 parts per octave it did not: 56 us against 47 for the radix path; now 31)
    n, k = 262_143, 2_621
    gen = torch.Generator(device="cuda"); gen.manual_seed(3)
    grads = [torch.empty(n, device="cuda").exponential_(generator=gen) * (torch.randint(0, 2, (n,), generator=gen, device="cuda") * 2 - 1) * 1e-3
             for _ in range(8)]
    times = {}
    for path in (1, 2):
        ctx = B.Context(n, k, 1)
        B.lgc_set_option(ctx, B.LGC_OPT_SELECT_PATH, path)
        u, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
        ov, oi = torch.zeros(k, device="cuda"), torch.zeros(k, dtype=torch.int32, device="cuda")
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for t in range(192):
            if t == 128:
                torch.cuda._sleep(3_000_000)     # the host runs ahead of what is timed
                start.record()
            B.lgc_accumulate_topk(ctx, grads[t % 8], u, v, 0.9, k, ov, oi)
        stop.record()
        torch.cuda.synchronize()
        times[path] = start.elapsed_time(stop)
        ctx.close()
    assert times[2] < times[1], times


def test_short_and_long_vectors_in_one_graph(B):
    # two selections per replay on alternating scratch, one of them by the short vectors' kernels
    gen = torch.Generator(device="cuda"); gen.manual_seed(3)
    shapes = [(100_003, 100), (400_000, 400)]
    ctx = B.Context(400_000, 400, 1)

    def tensors():
        gen.manual_seed(3)
        return [[torch.randn(n, generator=gen, device="cuda") for _ in range(3)]
                + [torch.zeros(k, device="cuda"), torch.zeros(k, dtype=torch.int32, device="cuda")] for n, k in shapes]

    def step(ts, c):
        for (n, k), (g, u, v, ov, oi) in zip(shapes, ts):
            B.lgc_accumulate_topk(c, g, u, v, 0.9, k, ov, oi)

    recorded, eager = tensors(), tensors()
    other = B.Context(400_000, 400, 1)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(recorded, ctx)
    for _ in range(5):
        graph.replay()
        step(eager, other)
        torch.cuda.synchronize()
        for r, e in zip(recorded, eager):
            assert all(torch.equal(x, y) for x, y in zip(r, e))
    assert B.lgc_stats(ctx)[2] == 0 and B.lgc_stats(other)[2] == 0
    ctx.close(); other.close()


# Records are laid out by the call's rows: several nodes in a context for longer vectors, with few, finishing and dense lists
@pytest.mark.parametrize("n,k,batch,max_n,max_k", [(50_001, 500, 3, 5_000_000, 20_000), (1_100_000, 1100, 3, 5_000_000, 20_000),
                                                   (2_000_003, 12_000, 3, 5_000_000, 20_000), (30_000_001, 900_000, 3, 40_000_000, 1_200_000)])
def test_records_in_a_larger_context(B, n, k, batch, max_n, max_k):
    gen = torch.Generator(device="cuda"); gen.manual_seed(n)
    ctx, own = B.Context(max_n, max_k, batch + 1), B.Context(n, k, batch)
    start = [torch.randn((batch, n), generator=gen, device="cuda") for _ in range(3)]
    results = []
    for c, path in ((ctx, 0), (own, 0), (own, 1)):
        B.lgc_set_option(c, B.LGC_OPT_SELECT_PATH, path)
        g, u, v = (t.clone() for t in start)
        ov, oi = torch.zeros((batch, k), device="cuda"), torch.zeros((batch, k), dtype=torch.int32, device="cuda")
        for _ in range(2):
            B.lgc_accumulate_topk(c, g, u, v, 0.9, k, ov, oi)
        results.append((u, v, ov, oi))
        assert B.lgc_stats(c)[1:] == (0, 0)          # nothing fell back: the records were read
    for other in results[1:]:
        assert all(torch.equal(x, y) for x, y in zip(results[0], other))
    ctx.close(); own.close()


# Rows (1024 elements) whose candidates fill a record exactly, exceed it by one, or fill the row; vectors at the limits of
# the one-launch finish (4096 rows) and a list long enough for the kernels of the dense selections.
@pytest.mark.parametrize("n,k", [(300_001, 1000), (4_194_304, 1000), (4_194_305, 1000), (5_000_003, 50_000), (5_000_003, 200_000)])
def test_rows_at_the_limits_of_a_record(B, oracle, n, k):
    rng = np.random.default_rng(n)
    v = rng.normal(0, 1e-3, (2, n + 1)).astype(np.float32)
    rows = n // 1024
    for b in range(2):
        for i, m in enumerate((1, 31, 32, 33, 40, 64, 1024, 32)):
            r = (i * 37 + b) % rows
            at = r * 1024 + rng.permutation(1024)[:m]
            v[b, at] = rng.choice([-1.0, 1.0], m) * (1.0 + rng.random(m))
    g, u = np.zeros_like(v), rng.normal(0, 1e-4, v.shape).astype(np.float32)
    ctx = B.Context(n, k, 2)
    dg, du, dv = (torch.from_numpy(a).cuda()[:, :n] for a in (g, u, v))
    ov, oi = torch.zeros((2, k), device="cuda"), torch.zeros((2, k), dtype=torch.int32, device="cuda")
    for _ in range(2):
        B.lgc_accumulate_topk(ctx, dg, du, dv, 0.9, k, ov, oi)
        for b in range(2):
            un, vn = u[b, :n].copy(), v[b, :n].copy()
            oracle.accumulate(g[b, :n].copy(), un, vn, 0.9)
            vals, idx = oracle.topk(vn, un, k)
            u[b, :n], v[b, :n] = un, vn
            assert (oi[b].cpu().numpy().astype(np.uint32) == idx).all() and same(ov[b], vals)
        assert same(dv, v[:, :n]) and same(du, u[:, :n])
    assert B.lgc_stats(ctx)[2] == 0
    ctx.close()
