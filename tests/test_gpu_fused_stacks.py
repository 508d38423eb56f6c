"""The stacks of Table I / Table II as one launch each (three-part bf16 products in fp32 precision) against the oracle:
lengths at the edges of a block's run of 15 or 31 latent positions (240, 496 values), inputs the split cannot represent, calls in place."""
import numpy as np
import pytest
import torch

from paper_2103_08870_amd import synth

pytestmark = pytest.mark.gpu

# Every layer rounds its sums to fp32 a few dozen times (2^-24 each, signs at random: about 2^-23 of the output's norm)
# and the stacks have four deep layers.  A product left out of the split would show: m m' alone is 2^-18.
REL_L2 = 4 * 2.0 ** -23


@pytest.fixture(scope="module")
def B():
    from paper_2103_08870_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def stacks(B, change=None):
    enc, dec = synth.paper_ae()
    host = [[t.numpy() for t in xs] for xs in synth.ae_weights(enc, dec, device="cpu")]
    if change is not None:
        host = [[np.ascontiguousarray(change(a, which)) for a in xs] for which, xs in enumerate(host)]
    dev = [[torch.from_numpy(a).cuda() for a in xs] for xs in host]
    return B.Autoencoder(enc, dec, *dev, slope=0.01), enc, dec, host


def both_ways(B, oracle, ae, enc, dec, host, x, latent=None):
    """(gpu latent, oracle's, gpu reconstruction of the oracle's latent, oracle's), per node stacked."""
    batch, k = x.shape
    ctx = B.Context(k, k, batch)
    B.lgc_reserve(ctx, ae, k, batch)
    lat = torch.full((batch, B.lgc_latent_len(ae, k)), 7.0, device="cuda")
    rec = torch.full((batch, k), 7.0, device="cuda")
    B.lgc_encode(ctx, ae, torch.from_numpy(x).cuda(), lat)
    with np.errstate(all="ignore"):
        ol = np.stack([oracle.encode(row, enc, host[0], host[1], slope=0.01) for row in x])
    src = ol if latent is None else latent.reshape(ol.shape)
    B.lgc_decode(ctx, ae, torch.from_numpy(np.ascontiguousarray(src.reshape(batch, -1))).cuda(), rec)
    with np.errstate(all="ignore"):
        orec = np.stack([oracle.decode(np.ascontiguousarray(z), k, enc, dec, host[2], host[3], slope=0.01) for z in src])
    torch.cuda.synchronize()
    ctx.close()
    return lat.cpu().numpy(), ol.reshape(batch, -1), rec.cpu().numpy(), orec


def assert_near(got, want, what):
    assert (np.isnan(got) == np.isnan(want)).all() and (np.isinf(got) == np.isinf(want)).all(), what
    assert (got[np.isinf(want)] == want[np.isinf(want)]).all(), what
    ok = np.isfinite(want)
    err = np.linalg.norm(got[ok].astype(np.float64) - want[ok]) / max(np.linalg.norm(want[ok].astype(np.float64)), 1e-300)
    assert err <= REL_L2, (what, err)


# the last three take 31 positions per block: a last block of 31, of 1 and of 2 positions
@pytest.mark.parametrize("k,batch", [(2, 1), (15, 1), (16, 3), (239, 1), (240, 2), (241, 1), (256, 1), (480, 1), (497, 3),
                                     (496 * 20, 7), (496 * 20 + 1, 7), (496 * 20 + 17, 7)])
def test_lengths_at_the_edges_of_a_block(B, oracle, k, batch):
    ae, enc, dec, host = stacks(B)
    x = np.random.default_rng(k).laplace(0, 0.3, (batch, k)).astype(np.float32)
    lat, ol, rec, orec = both_ways(B, oracle, ae, enc, dec, host, x)
    assert_near(lat, ol, ("latent", k))
    assert_near(rec, orec, ("reconstruction", k))
    ae.close()


# The encoder's runs of 15 positions go to four blocks each (up to 64 runs), to two (up to 128) or to one; what whole rounds of runs of 31 leave over is cut into
# runs of 15 (7 nodes x 1 147 positions: 252 of 31, 21 of 15): a last run of all, of one and of two positions.
@pytest.mark.parametrize("k,batch", [(3840, 4), (3841, 4), (4800, 5), (4801, 5), (4817, 5), (4800, 7), (4801, 7), (18352, 7), (18353, 7)])
def test_lengths_at_the_edges_of_an_encoder_run(B, oracle, k, batch):
    ae, enc, dec, host = stacks(B)
    x = np.random.default_rng(k).laplace(0, 0.3, (batch, k)).astype(np.float32)
    ctx = B.Context(k, k, batch)
    B.lgc_reserve(ctx, ae, k, batch)
    ol = np.stack([oracle.encode(row, enc, host[0], host[1], slope=0.01) for row in x]).reshape(batch, -1)
    for _ in range(3):   # the counts by which blocks meet are as the call before left them
        lat = torch.full((batch, B.lgc_latent_len(ae, k)), 7.0, device="cuda")
        B.lgc_encode(ctx, ae, torch.from_numpy(x).cuda(), lat)
        assert_near(lat.cpu().numpy(), ol, ("latent", k))
    ctx.close(); ae.close()


def test_a_recorded_encode_replays_after_a_larger_reservation(B):
    # 4 and 2 blocks share a run; the activation scratch moves in between, as eager calls of the context need more of it
    ae, _, _, _ = stacks(B)
    small, large = [(1, 1_023), (4, 5_000)], (8, 30_000)
    ctx = B.Context(large[1], large[1], large[0])
    xs = [torch.randn(shape, device="cuda") * 0.3 for shape in small + [large]]
    lats = [torch.empty((x.shape[0], B.lgc_latent_len(ae, x.shape[1])), device="cuda") for x in xs]
    graphs, want = [], []
    for x, lat in zip(xs[:2], lats):
        B.lgc_reserve(ctx, ae, x.shape[1], x.shape[0])
        B.lgc_encode(ctx, ae, x, lat)
        want.append(lat.clone())
        torch.cuda.synchronize()
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            B.lgc_encode(ctx, ae, x, lat)
    B.lgc_reserve(ctx, ae, large[1], large[0])
    other = torch.full((1 << 22,), 5.0, device="cuda")     # what may have taken the old scratch's place
    for _ in range(4):
        for graph, lat, first in zip(graphs, lats, want):
            lat.fill_(7.0)
            graph.replay()
            B.lgc_encode(ctx, ae, xs[2], lats[2])
            torch.cuda.synchronize()
            assert torch.equal(lat, first)
    assert (other == 5.0).all()
    ctx.close(); ae.close()


# The decoder's blocks take 7 latent positions (112 values), 15 (240), or 15 with the weights through the LDS: a last block of all, of one and of two.
@pytest.mark.parametrize("k,batch", [(112, 1), (113, 1), (224, 2), (112 * 3 + 17, 3), (3840, 8), (3841, 8), (3857, 8), (7920, 8), (7921, 8), (7937, 8)])
def test_lengths_at_the_edges_of_a_decoder_block(B, oracle, k, batch):
    ae, enc, dec, host = stacks(B)
    x = np.random.default_rng(k).laplace(0, 0.3, (batch, k)).astype(np.float32)
    _, _, rec, orec = both_ways(B, oracle, ae, enc, dec, host, x)
    assert_near(rec, orec, ("reconstruction", k))
    ae.close()


# The one-launch stacks may not be further from the 64-bit result than one fp32 launch per layer was.  The bounds are what those
# kernels measured for the same weights and values (error of the latent, of the reconstruction, in 1e-8, seeds 0 to 3).
FP32 = {1_023: ((14.31, 3.74), (9.44, 2.28), (11.37, 7.27), (10.05, 3.30)),
        25_600: ((20.24, 3.64), (11.31, 2.19), (12.99, 7.49), (11.45, 3.26))}


@pytest.mark.parametrize("k,batch", [(1_023, 1), (25_600, 4)])
def test_error_against_64_bits(B, k, batch):
    enc, dec = synth.paper_ae()
    slope, errors = 0.01, []
    for seed in range(4):
        w = [[t.cuda() for t in xs] for xs in synth.ae_weights(enc, dec, device="cpu", seed=seed)]
        gen = torch.Generator(device="cuda"); gen.manual_seed(seed)
        x = torch.randn((batch, k), generator=gen, device="cuda") * 0.3
        ae, ctx = B.Autoencoder(enc, dec, *w, slope=slope), B.Context(k, k, batch)
        B.lgc_reserve(ctx, ae, k, batch)
        lat, rec = torch.empty((batch, B.lgc_latent_len(ae, k)), device="cuda"), torch.empty((batch, k), device="cuda")
        B.lgc_encode(ctx, ae, x, lat)
        B.lgc_decode(ctx, ae, lat, rec)
        w = [[t.double().cpu() for t in xs] for xs in w]
        h, lens = x.double().cpu()[:, None], []
        for i, (_, _, ks, st) in enumerate(enc):
            lens.append(h.shape[2])
            h = torch.nn.functional.conv1d(h, w[0][i], w[1][i], stride=st, padding=(ks - 1) // 2)
            h = h if i + 1 == len(enc) else torch.nn.functional.leaky_relu(h, slope)
        got = lat.double().cpu()
        e_lat = ((got - h.flatten(1)).norm() / h.norm()).item()
        h = got.view(h.shape)
        lens = [n for n, (_, _, _, st) in zip(lens, enc) if st == 2]
        for i, (_, _, ks, st) in enumerate(dec):
            n = lens.pop() if st == 2 else h.shape[2]
            pad = (ks - 1) // 2
            h = torch.nn.functional.conv_transpose1d(h, w[2][i], w[3][i], stride=st, padding=pad,
                                                     output_padding=n - ((h.shape[2] - 1) * st + ks - 2 * pad))
            h = h if i + 1 == len(dec) else torch.nn.functional.leaky_relu(h, slope)
        errors.append((e_lat, ((rec.double().cpu() - h[:, 0]).norm() / h.norm()).item()))
        ctx.close(); ae.close()
    for got, bound in zip(errors, FP32[k]):
        assert got[0] < bound[0] * 1e-8 and got[1] < bound[1] * 1e-8, (errors, FP32[k])


# Positive weights: an Inf stays one Inf all the way (weights of both signs would turn it into NaN at once), so the
# values that bf16 parts cannot carry have one right answer.  The largest finite values round to Inf in bf16.  The encoder's runs of
# 15 latent positions with four blocks each (600 values), two (5 nodes x 6 000) and one (7 x 4 802), of 31 (7 x 10 000), and of both (7 x 18 353); the decoder's of 7 and
# of 15.  The values sit inside a block, where two blocks' windows overlap, and at the very end: where a layer's length is even and the next
# one's odd (lengths that leave 2 of 4 values over: conv1; 604: conv2; 600: conv3), that is also the input of a position that
# does not exist, and which the next layer's last output reads as 0.  At 1e-33 the split's low parts, and their products,
# are below the least normal number (the reconstruction, about 3e-38, is just above it); no biases, which would hide it.
@pytest.mark.parametrize("k,batch", [(600, 2), (602, 2), (604, 2), (608, 2), (4_802, 7), (6_000, 5), (10_000, 7), (10_002, 7), (18_353, 7)])
@pytest.mark.parametrize("special", [np.inf, np.nan, 3.4e38, 1e-30, 1e-33, 0.0])
def test_values_that_the_split_cannot_carry(B, oracle, special, k, batch):
    def change(a, which):
        if which % 2:
            return np.zeros_like(a) if special < 1 else np.abs(a)   # biases
        return np.abs(a) * np.float32(0.05)
    ae, enc, dec, host = stacks(B, change)
    rng = np.random.default_rng(5)
    length = -(-k // 16)
    x = np.abs(rng.normal(0, 1, (batch, k))).astype(np.float32)
    z = np.abs(rng.normal(0, 1, (batch, 4, length))).astype(np.float32)
    if special < 1:
        x *= np.float32(special); z *= np.float32(special)
    else:
        x[1, [300, k - 1]] = special
        z[1, 2, [20, length - 1]] = special
        if batch > 2:
            x[3, [16 * 31 * 3 - 8, 16 * 31 * 7]] = special
            z[3, 0, [15 * 4, 15 * 9 - 1]] = special
    lat, ol, rec, orec = both_ways(B, oracle, ae, enc, dec, host, x, z)
    assert_near(lat, ol, ("latent", special))
    assert_near(rec, orec, ("reconstruction", special))
    if not np.isfinite(special):
        assert (~np.isfinite(ol)).any() and np.isfinite(ol[0]).all()   # the case is what it says
    ae.close()


# The sum at the position behind conv1's last one overflows (the last input times the first tap), no sum at a position that exists does.
@pytest.mark.parametrize("k,batch", [(602, 2), (4_802, 7), (6_002, 5), (10_002, 7)])
def test_a_sum_that_overflows_where_there_is_no_position(B, oracle, k, batch):
    def change(a, which):
        if which % 2:
            return np.abs(a)
        a = np.abs(a) * np.float32(0.05)
        if which == 0 and a.shape[1] == 1:
            a[:, 0, 0], a[:, 0, 2] = 3.0, 1e-5
        return a
    ae, enc, dec, host = stacks(B, change)
    x = np.abs(np.random.default_rng(k).normal(0, 1, (batch, k))).astype(np.float32)
    x[batch - 1, k - 1] = 3e38
    lat, ol, _, _ = both_ways(B, oracle, ae, enc, dec, host, x, np.ones((batch, 4 * -(-k // 16)), np.float32))
    assert np.isfinite(ol).all() and ol[-1].max() > 1e30    # the case is what it says
    assert_near(lat, ol, "latent")
    ae.close()


def test_values_that_are_not_finite_cost_no_more_than_fp32(B):
    # the redo runs on the matrix cores (measured: 3 times the ordinary call where every block redoes); position by
    # position on the vector units it took 100 times as long
    k, batch = 25_600, 4
    ae, _, _, _ = stacks(B)
    ctx = B.Context(k, k, batch)
    B.lgc_reserve(ctx, ae, k, batch)
    lat, rec = torch.empty((batch, B.lgc_latent_len(ae, k)), device="cuda"), torch.empty((batch, k), device="cuda")

    def milliseconds(x):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for timed in (False, True):
            if timed:
                start.record()
            for _ in range(20):
                B.lgc_encode(ctx, ae, x, lat)
                B.lgc_decode(ctx, ae, lat, rec)
        stop.record()
        torch.cuda.synchronize()
        return start.elapsed_time(stop)

    usual = milliseconds(torch.full((batch, k), 0.5, device="cuda"))
    nan = milliseconds(torch.full((batch, k), float("nan"), device="cuda"))
    assert torch.isnan(rec).all() and nan < 12 * usual, (nan, usual)
    ctx.close(); ae.close()


@pytest.mark.parametrize("factor", [np.inf, 1e6, 1e-36])
def test_weights_that_the_split_cannot_carry(B, oracle, factor):
    # such a handle keeps to the fp32 kernels: one Inf (NaN where the oracle has a NaN), deep layers so large that what the split
    # loses of small numbers could show, a layer of weights near the least normal number (nothing else may cover what it gives);
    # positive ones, so that sums do not cancel
    def change(a, which):
        a = a.copy() if factor == np.inf else np.abs(a)
        if factor == np.inf:
            if a.shape == (256, 128, 3):
                a[7, 3, 1] = np.inf
        elif factor == 1e-36:
            a *= np.float32(factor if a.shape in ((128, 64, 3), (32, 64, 3)) else 1e3 if a.ndim == 3 else 0)
        elif a.ndim == 3 and min(a.shape[:2]) >= 32:
            a *= np.float32(factor)
        return a
    ae, enc, dec, host = stacks(B, change)
    x = np.random.default_rng(1).uniform(0, 1, (1, 100)).astype(np.float32)
    lat, ol, rec, orec = both_ways(B, oracle, ae, enc, dec, host, x, np.ones((1, 4 * 7), np.float32))
    assert_near(lat, ol, "latent")
    assert_near(rec, orec, "reconstruction")
    ae.close()


@pytest.mark.parametrize("k,batch", [(600, 2), (20_000, 4)])
def test_in_place(B, oracle, k, batch):
    # the output over the input: every value of it is stored after the last read of what it replaces
    ae, enc, dec, host = stacks(B)
    x = np.random.default_rng(k).laplace(0, 0.3, (batch, k)).astype(np.float32)
    ctx = B.Context(k, k, batch)
    B.lgc_reserve(ctx, ae, k, batch)
    length = B.lgc_latent_len(ae, k)
    buf = torch.from_numpy(x).cuda()
    lat = buf.view(-1)[:batch * length].view(batch, length)
    B.lgc_encode(ctx, ae, buf, lat)
    ol = np.stack([oracle.encode(row, enc, host[0], host[1], slope=0.01) for row in x])
    assert_near(lat.cpu().numpy(), ol.reshape(batch, -1), "latent")
    B.lgc_decode(ctx, ae, lat, buf)
    orec = np.stack([oracle.decode(z, k, enc, dec, host[2], host[3], slope=0.01) for z in ol])
    assert_near(buf.cpu().numpy(), orec, "reconstruction")
    ctx.close(); ae.close()
