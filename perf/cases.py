"""Cases that stand for what a program uses this library for, each timed as one pass through the public entry
points (`paper_2103_08870_amd.binding`).

A worker's iteration is accumulate + top-k, encode, decode, scatter; the library also serves the per-layer selection
with the innovation component (parameter server), the ring-allreduce pattern, the selection on its own, the
call that needs no context, and the autoencoder of the paper's Tables I and II on its own.  Sizes are those of the
five benchmark workloads and ragged ones between and below them.

A pass of a `step` case is one iteration of a run in progress: the residuals u, v are those of a run (a plain-torch
imitation of forty iterations brings them there) and every pass takes the next of several resident gradients.
"""
import math
import random

import torch

from paper_2103_08870_amd import binding as B

MOMENTUM = 0.9
LEARNING_RATE = 0.1
WARM_ITERATIONS = 40
SLOPE = 0.01            # of the paper's leaky-ReLU; the two-layer autoencoders use 0

# layers are (c_in, c_out, kernel, stride)
PAPER_ENC = [(1, 64, 3, 2), (64, 128, 3, 2), (128, 256, 3, 2), (256, 64, 3, 2), (64, 4, 1, 1)]
PAPER_DEC = [(4, 4, 3, 1), (4, 32, 3, 2), (32, 64, 3, 2), (64, 128, 3, 2), (128, 32, 3, 2), (32, 1, 1, 1)]


def listed():
    return [
        # one small model on one node: seven dependent small kernels, latency and launches
        dict(name="step_tiny", kind="step", nodes=1, n=1 << 20, k=1024, layers=0, ties=False, hidden=8),
        # the headline workload: ResNet50-sized, four nodes, 0.1 %
        dict(name="step_resnet50", kind="step", nodes=4, n=25_600_000, k=25_600, layers=161, ties=False, hidden=8),
        # ResNet101-sized, eight nodes
        dict(name="step_resnet101", kind="step", nodes=8, n=44_500_000, k=44_500, layers=314, ties=False, hidden=16),
        # the largest vector and the densest selection, with many equal magnitudes
        dict(name="step_stress_1pct", kind="step", nodes=1, n=1 << 28, k=2_684_354, layers=0, ties=True, hidden=16),
        # Alg. 1 in full: per-layer selection, innovation component, decoder with the innovation channel
        dict(name="innovation_resnet50", kind="innovation", nodes=4, n=25_600_000, layers=161, ratio=0.001, hidden=8),
        # Alg. 2: one node selects, the others take the values at its positions, the latents are averaged
        dict(name="ring_resnet50", kind="ring", nodes=4, n=25_600_000, k=25_600, layers=161, hidden=8),
        # accumulation and selection as two calls (a program that looks at v in between), rows that no vector load
        # is aligned to
        dict(name="pair_ragged", kind="pair", nodes=3, n=3_333_331, k=3_333, layers=40),
        # one layer's tensor, compressed by a caller that holds no context
        dict(name="static_small", kind="static", nodes=1, n=100_003, k=1_000, layers=0),
        # Table I and Table II at the headline workload's size, each direction on its own
        dict(name="encode_paper_resnet50", kind="encode", nodes=4, k=25_600),
        dict(name="decode_paper_resnet50", kind="decode", nodes=4, k=25_600),
        # both directions for a short ragged vector (few tiles: latency) and for the longest one (PSPNet-sized)
        dict(name="autoencode_paper_small", kind="autoencode", nodes=1, k=1_023),
        dict(name="autoencode_paper_pspnet", kind="autoencode", nodes=8, k=67_000),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "innovation", "ring", "pair", "static", "encode", "decode", "autoencode"])
    if kind in ("encode", "decode", "autoencode"):
        return dict(kind=kind, nodes=rng.randint(1, 8), k=_log_uniform(rng, 500, 67_000))
    if kind == "static":
        nodes, n = rng.randint(1, 4), _log_uniform(rng, 20_000, 4_000_000)
        return dict(kind=kind, nodes=nodes, n=n, k=max(1, n // rng.choice([100, 1000])), layers=rng.randint(1, 20))
    if kind == "pair":
        nodes, n = rng.randint(1, 8), _log_uniform(rng, 30_000, 20_000_000)
        return dict(kind=kind, nodes=nodes, n=n, k=max(1, n // rng.choice([100, 1000, 10_000])), layers=rng.randint(1, 100))
    nodes = rng.randint(2, 8) if kind == "ring" else rng.randint(1, 8)
    n = _log_uniform(rng, 300_000, min(60_000_000, 240_000_000 // nodes))
    if kind == "innovation":
        return dict(kind=kind, nodes=nodes, n=n, layers=rng.randint(10, 400), ratio=rng.choice([0.001, 0.01]),
                    hidden=rng.choice([8, 16]))
    case = dict(kind=kind, nodes=nodes, n=n, k=max(64, n // rng.choice([100, 1000, 1000, 10_000])),
                layers=rng.randint(1, 400), hidden=rng.choice([8, 16]))
    if kind == "step":
        case["ties"] = rng.random() < 0.2
    return case


# ---------------------------------------------------------------------------------------- inputs

def _layout(n, layers):
    """Layer boundaries [0, .., n] (sizes spread over three decades) and the layers' gradient scales."""
    if layers == 0:
        return [0, n], [1e-3]
    rng = random.Random(1000 * layers + n)
    weights = [math.exp(rng.uniform(math.log(1e3), math.log(2.4e6))) for _ in range(layers)]
    total, room = sum(weights), n - 64 * layers
    sizes = [64 + int(room * w / total) for w in weights]
    sizes[-1] += n - sum(sizes)
    scales = [math.exp(rng.uniform(math.log(1e-5), math.log(1e-2))) for _ in range(layers)]
    bounds = [0]
    for s in sizes:
        bounds.append(bounds[-1] + s)
    return bounds, scales


def _layer_ks(bounds, ratio):
    return [max(1, int(ratio * (bounds[i + 1] - bounds[i]))) for i in range(len(bounds) - 1)]


def _total_k(case):
    return case["k"] if "k" in case else sum(_layer_ks(_layout(case["n"], case["layers"])[0], case["ratio"]))


def _laplace(shape, gen):
    x = torch.rand(shape, generator=gen, device="cuda").sub_(0.5)
    size = x.abs().mul_(-2.0).clamp_(min=-0.9999999).log1p_().neg_()
    return size.copysign_(x)


def _gradients(case, gen):
    """One iteration's gradients [nodes][n]: a common part plus 0.3 of a part of the node's own, scaled per layer."""
    nodes, n = case["nodes"], case["n"]
    out = torch.empty((nodes, n), device="cuda")
    if case.get("ties"):
        # 0.1 % large entries, a quarter of all entries snapped to 4096 magnitudes
        for b in range(nodes):
            g = torch.randn(n, generator=gen, device="cuda")
            g *= torch.where(torch.rand(n, generator=gen, device="cuda") < 0.001, 1e-1, 1e-4)
            level = torch.round(torch.log10(g.abs().clamp_(1e-5, 1.0)).add_(5.0).mul_(4095.0 / 5.0))
            snapped = torch.pow(10.0, level.mul_(5.0 / 4095.0).sub_(5.0)).copysign_(g)
            out[b] = torch.where(torch.rand(n, generator=gen, device="cuda") < 0.25, snapped, g)
        return out
    bounds, scales = _layout(n, case["layers"])
    sizes = torch.tensor([bounds[i + 1] - bounds[i] for i in range(len(scales))], device="cuda")
    scale = torch.repeat_interleave(torch.tensor(scales, device="cuda"), sizes, output_size=n)
    common = _laplace((n,), gen)
    for b in range(nodes):
        torch.add(common, _laplace((n,), gen), alpha=0.3, out=out[b])
        out[b] *= scale
    return out


def _sets(case):
    return 8 if case["nodes"] * case["n"] <= 20_000_000 else 4


def _residuals(case, grads):
    """u, v of a run in progress: the iteration with a sampled threshold in the place of the exact selection."""
    nodes, n = case["nodes"], case["n"]
    u, v = torch.zeros((nodes, n), device="cuda"), torch.zeros((nodes, n), device="cuda")
    share = _total_k(case) / n
    bounds = _layout(n, case["layers"])[0] if case["kind"] == "innovation" else [0, n]
    spans = []
    for lo, hi in zip(bounds, bounds[1:]):
        step = max(1, (hi - lo) // (65_536 if len(bounds) == 2 else 8_192))
        count = -(-(hi - lo) // step)
        spans.append((lo, hi, step, max(1, min(count, round(share * count)))))
    for t in range(WARM_ITERATIONS):
        u.mul_(MOMENTUM).add_(grads[t % len(grads)])
        v.add_(u)
        for lo, hi, step, rank in (spans if len(spans) == 1 or t % 4 == 3 else ()):
            part = v[:, lo:hi]
            bar = part[:, ::step].abs().topk(rank, dim=1).values[:, -1:]
            sent = part.abs() > bar
            part.masked_fill_(sent, 0.0)
            u[:, lo:hi].masked_fill_(sent, 0.0)
    return u, v


def _selected_values(case, gen):
    """[nodes][k] values like those a selection sends: magnitudes above a threshold, layers of different spread."""
    shape = (case["nodes"], case["k"])
    spread = torch.repeat_interleave(torch.rand((shape[0], -(-shape[1] // 256)), generator=gen, device="cuda"), 256, dim=1)
    tail = -torch.log1p(-torch.rand(shape, generator=gen, device="cuda"))
    sign = torch.where(torch.rand(shape, generator=gen, device="cuda") < 0.5, -1.0, 1.0)
    return (sign * (0.2 + (0.02 + 0.2 * spread[:, :shape[1]]) * tail)).contiguous()


def _stacks(case):
    """(encoder layers, decoder layers, slope)"""
    if "hidden" not in case:
        return PAPER_ENC, PAPER_DEC, SLOPE
    h = case["hidden"]
    enc = [(1, h, 3, 2), (h, h // 2, 3, 2)]
    if case["kind"] == "innovation":
        return enc, [(h // 2, h, 3, 2), (h, h // 2, 3, 2), (h // 2 + 1, 1, 1, 1)], 0.0
    return enc, [(h // 2, h, 3, 2), (h, 1, 3, 2)], 0.0


def _weights(case, gen):
    """(enc_w, enc_b, dec_w, dec_b): uniform within 1 / sqrt(fan in)."""
    enc, dec, _ = _stacks(case)

    def uniform(shape, bound):
        return torch.rand(shape, generator=gen, device="cuda").mul_(2.0).sub_(1.0).mul_(bound)

    out = [[], [], [], []]
    for at, layers in ((0, enc), (2, dec)):
        for ci, co, ks, _ in layers:
            bound = 1.0 / math.sqrt(ks * ci)
            out[at].append(uniform((co, ci, ks) if at == 0 else (ci, co, ks), bound))
            out[at + 1].append(uniform((co,), bound))
    return out


def _inputs(case, seed):
    """What the seed decides, as plain tensors."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind in ("encode", "decode", "autoencode"):
        got = dict(weights=_weights(case, gen), vals=_selected_values(case, gen))
        if kind == "decode":
            enc, _, slope = _stacks(case)
            got["latent"] = _encode64(got["vals"].double(), enc, got["weights"], slope).float().flatten(1).contiguous()
        return got
    grads = [_gradients(case, gen) for _ in range(_sets(case))]
    u, v = _residuals(case, grads)
    got = dict(grads=grads, u=u, v=v)
    if kind not in ("pair", "static"):
        got["weights"] = _weights(case, gen)
        got["params"] = torch.randn(case["n"], generator=gen, device="cuda").mul_(0.02)
    return got


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"], s["t"] = case, 0
    kind, nodes, k = case["kind"], case["nodes"], _total_k(case)
    s["k"] = k
    if kind != "static":
        s["ctx"] = B.Context(case.get("n", k), k, nodes)
    if "weights" in s:
        enc, dec, slope = _stacks(case)
        s["ae"] = B.Autoencoder(enc, dec, *s["weights"], slope=slope)
        if kind == "innovation":
            bounds = _layout(case["n"], case["layers"])[0]
            ks = _layer_ks(bounds, case["ratio"])
            starts = [0]
            for kl in ks:
                starts.append(starts[-1] + kl)
            s["seg"] = B.Segments(bounds, ks)
            s["inv_seg"] = B.Segments(starts, [max(1, kl // 10) for kl in ks])
            s["innov"] = torch.empty((nodes, k), device="cuda")
        B.lgc_reserve(s["ctx"], s["ae"], k, nodes, s.get("seg"))
        lat = B.lgc_latent_len(s["ae"], k)
        if "latent" not in s:
            s["latent"] = torch.empty((nodes, lat), device="cuda")
        s["avg"] = torch.empty((1, lat), device="cuda")
        s["rec"] = torch.empty((1 if kind == "ring" else nodes, k), device="cuda")
    if kind not in ("encode", "decode", "autoencode"):
        s["vals"] = torch.empty((nodes, k), device="cuda")
        s["idx"] = torch.empty((1 if kind == "ring" else nodes, k), device="cuda", dtype=torch.int32)
    return s


# ---------------------------------------------------------------------------------------- one pass

def run(s):
    case, t = s["case"], s["t"]
    s["t"] = t + 1
    kind, nodes = case["kind"], case["nodes"]
    if kind in ("encode", "autoencode"):
        B.lgc_encode(s["ctx"], s["ae"], s["vals"], s["latent"])
        if kind == "encode":
            return {"latent": s["latent"]}
    if kind in ("decode", "autoencode"):
        B.lgc_decode(s["ctx"], s["ae"], s["latent"], s["rec"])
        return {"rec": s["rec"]} if kind == "decode" else {"latent": s["latent"], "rec": s["rec"]}
    g, u, v = s["grads"][t % len(s["grads"])], s["u"], s["v"]
    out = {"vals": s["vals"], "idx": s["idx"], "u": u, "v": v}
    if kind == "pair":
        B.lgc_accumulate(s["ctx"], g, u, v, MOMENTUM)
        B.lgc_topk(s["ctx"], v, u, s["k"], s["vals"], s["idx"])
        return out
    if kind == "static":
        B.lgc_accumulate_topk_static(g, u, v, MOMENTUM, s["k"], s["vals"], s["idx"])
        return out
    out.update(latent=s["latent"], rec=s["rec"], params=s["params"])
    ctx, ae = s["ctx"], s["ae"]
    if kind == "ring":
        lead = t % nodes
        B.lgc_accumulate_topk(ctx, g[lead], u[lead], v[lead], MOMENTUM, s["k"], s["vals"][lead], s["idx"][0])
        for lo, hi in ((0, lead), (lead + 1, nodes)):
            if hi > lo:
                B.lgc_accumulate_gather(ctx, g[lo:hi], u[lo:hi], v[lo:hi], MOMENTUM, s["idx"][0], s["vals"][lo:hi])
        B.lgc_encode(ctx, ae, s["vals"], s["latent"])
        B.lgc_average(ctx, s["latent"], 1.0 / nodes, s["avg"][0])
        B.lgc_decode(ctx, ae, s["avg"], s["rec"])
        B.lgc_scatter(ctx, s["rec"], s["idx"], -LEARNING_RATE, s["params"])
        return out
    if kind == "innovation":
        B.lgc_accumulate_topk_segmented(ctx, s["seg"], g, u, v, MOMENTUM, s["vals"], s["idx"])
        B.lgc_innovation(ctx, s["inv_seg"], s["vals"], s["innov"])
        B.lgc_encode(ctx, ae, s["vals"], s["latent"])
        B.lgc_decode_innovation(ctx, ae, s["latent"], s["innov"], s["rec"])
        out["innov"] = s["innov"]
    else:
        B.lgc_accumulate_topk(ctx, g, u, v, MOMENTUM, s["k"], s["vals"], s["idx"])
        B.lgc_encode(ctx, ae, s["vals"], s["latent"])
        B.lgc_decode(ctx, ae, s["latent"], s["rec"])
    B.lgc_scatter(ctx, s["rec"], s["idx"], -LEARNING_RATE / nodes, s["params"])
    return out


# ---------------------------------------------------------------------------------------- what a pass needs

def _lengths(case):
    """Output lengths of the encoder's and the decoder's layers."""
    enc, dec, _ = _stacks(case)
    lens, strided = [_total_k(case)], []
    for _, _, _, st in enc:
        if st == 2:
            strided.append(lens[-1])
        lens.append((lens[-1] + st - 1) // st)
    out = []
    for _, _, _, st in dec:
        out.append(strided.pop() if st == 2 else (out[-1] if out else lens[-1]))
    return lens[1:], out


def work(case):
    kind, nodes, k = case["kind"], case["nodes"], _total_k(case)
    n = case.get("n", 0)
    moved = flops = 0
    if n:
        # g, u, v read and u, v written once; as two calls v is read again and the sent positions of v and u cleared;
        # the selected values and positions written
        moved += nodes * (20 * n + (4 * n + 8 * k if kind == "pair" else 0)) + 8 * nodes * k
        flops += nodes * 3 * n
    if kind not in ("pair", "static"):
        enc, dec, _ = _stacks(case)
        enc_len, dec_len = _lengths(case)
        latent = enc[-1][1] * enc_len[-1]
        dec_nodes = 1 if kind == "ring" else nodes
        if kind != "decode":
            flops += 2 * nodes * sum(ci * co * ks * le for (ci, co, ks, _), le in zip(enc, enc_len))
            moved += 4 * nodes * (k + latent)
        if kind != "encode":
            # every input position of a transposed layer meets every tap once
            ins = [enc_len[-1]] + dec_len[:-1]
            flops += 2 * dec_nodes * sum(ci * co * ks * le for (ci, co, ks, _), le in zip(dec, ins))
            moved += 4 * dec_nodes * (k + latent)
        if kind in ("step", "ring", "innovation"):
            moved += dec_nodes * k * 16          # values and positions read, parameters updated
        if kind == "innovation":
            moved += 8 * nodes * k
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    if case["kind"] in ("pair", "static"):
        return "exact"
    # 32-bit sums of up to 768 products, up to six layers of them: 0.4e-7 to 2.8e-7 off the 64-bit result;
    # positions are the same whatever the rounding
    return {"rel": 1e-6, "max": 2e-5}


# ---------------------------------------------------------------------------------------- the same in 64 bits

def _act(x, slope, last):
    return x if last else torch.where(x > 0, x, slope * x)


def _encode64(x, layers, weights, slope):
    """x [nodes][k] -> [nodes][c][l], in x's precision."""
    x = x[:, None, :]
    for i, (_, _, ks, st) in enumerate(layers):
        w, bias = weights[0][i].to(x.dtype), weights[1][i].to(x.dtype)
        pad = (ks - 1) // 2
        l_out = (x.shape[2] + 2 * pad - ks) // st + 1
        xp = torch.nn.functional.pad(x, (pad, pad))
        y = bias[:, None].expand(x.shape[0], -1, l_out).clone()
        for t in range(ks):
            y += torch.matmul(w[:, :, t].contiguous(), xp[:, :, t:t + st * (l_out - 1) + 1:st].contiguous())
        x = _act(y, slope, i + 1 == len(layers))
    return x


def _decode64(x, layers, weights, slope, out_len, innov=None):
    """x [nodes][c][l] -> [nodes][k]; innov: the extra channel of the last layer."""
    for i, (_, co, ks, st) in enumerate(layers):
        w, bias = weights[2][i].to(x.dtype), weights[3][i].to(x.dtype)
        if innov is not None and i + 1 == len(layers):
            x = torch.cat([x, innov[:, None, :].to(x.dtype)], dim=1)
        pad = (ks - 1) // 2
        full = torch.zeros((x.shape[0], co, (x.shape[2] - 1) * st + ks + 1), dtype=x.dtype, device=x.device)
        for t in range(ks):
            full[:, :, t:t + st * (x.shape[2] - 1) + 1:st] += torch.matmul(w[:, :, t].t().contiguous(), x)
        y = full[:, :, pad:pad + out_len[i]] + bias[:, None]
        x = _act(y, slope, i + 1 == len(layers)).contiguous()
    return x[:, 0, :]


def _top(key, k):
    """Positions of the k largest of an int32 key, lowest positions first among equals, ascending."""
    bar = key.topk(k).values[-1]
    above = (key > bar).nonzero()[:, 0]
    equal = (key == bar).nonzero()[:, 0]
    return torch.cat([above, equal[:k - above.numel()]]).sort().values


def _select64(case, u, v, u64, v64):
    """Selection by the 32-bit values that the method defines; (vals64, idx); the sent positions of u64, v64 cleared."""
    vals, idx = [], []
    for b in range(case["nodes"]):
        key = v[b].view(torch.int32) & 0x7FFFFFFF
        if case["kind"] == "innovation":
            bounds = _layout(case["n"], case["layers"])[0]
            ks = _layer_ks(bounds, case["ratio"])
            at = torch.cat([bounds[i] + _top(key[bounds[i]:bounds[i + 1]], ks[i]) for i in range(len(ks))])
        elif case["kind"] == "ring" and b > 0:
            at = idx[0]
        else:
            at = _top(key, case["k"])
        vals.append(v64[b][at])
        idx.append(at)
        v64[b][at] = 0
        u64[b][at] = 0
    return torch.stack(vals), torch.stack(idx)


def exact(case, seed):
    s = _inputs(case, seed)
    kind, nodes = case["kind"], case["nodes"]
    if kind in ("encode", "decode", "autoencode"):
        enc, dec, slope = _stacks(case)
        if kind == "decode":
            latent = s["latent"].double().view(nodes, enc[-1][1], -1)
        else:
            # a program decodes the latent that the encoder gave it; in 64 bits the two run on without rounding
            latent = _encode64(s["vals"].double(), enc, s["weights"], slope)
        out = {} if kind == "decode" else {"latent": latent.flatten(1)}
        if kind != "encode":
            out["rec"] = _decode64(latent, dec, s["weights"], slope, _lengths(case)[1])
        return out
    g, u, v = s["grads"][0], s["u"], s["v"]
    u64 = u.double().mul_(float(torch.tensor(MOMENTUM))).add_(g)
    v64 = v.double().add_(u64)
    u = u.mul(MOMENTUM).add_(g)     # three operations, each rounded to 32 bits: what decides the selection
    v = v.add(u)
    vals, idx = _select64(case, u, v, u64, v64)
    if kind == "ring":
        idx = idx[:1]
    out = {"vals": vals, "idx": idx.int(), "u": u64, "v": v64}
    if kind in ("pair", "static"):
        return out
    enc, dec, slope = _stacks(case)
    latent = _encode64(vals, enc, s["weights"], slope)
    innov = None
    if kind == "innovation":
        innov = torch.zeros_like(vals)
        start = 0
        sent = torch.stack([v[b][idx[b]] for b in range(nodes)]).view(torch.int32) & 0x7FFFFFFF
        for kl in _layer_ks(_layout(case["n"], case["layers"])[0], case["ratio"]):
            for b in range(nodes):
                at = start + _top(sent[b, start:start + kl], max(1, kl // 10))
                innov[b, at] = vals[b, at]
            start += kl
        out["innov"] = innov
    if kind == "ring":
        lead = latent.mean(dim=0, keepdim=True)
        rec = _decode64(lead, dec, s["weights"], slope, _lengths(case)[1])
        scale = -LEARNING_RATE
    else:
        rec = _decode64(latent, dec, s["weights"], slope, _lengths(case)[1], innov)
        scale = -LEARNING_RATE / nodes
    params = s["params"].double()
    for b in range(rec.shape[0]):
        params[idx[b].long()] += scale * rec[b]
    out.update(latent=latent.flatten(1), rec=rec, params=params)
    return out
