"""What the library's host side launches and allocates for a call, read from a HIP runtime that only records
(recording_hip.cpp): no GPU, no tensor, any size."""
import ctypes as C
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

u64, p = C.c_uint64, C.c_void_p
PAPER = ([(1, 64, 3, 2), (64, 128, 3, 2), (128, 256, 3, 2), (256, 64, 3, 2), (64, 4, 1, 1)],
         [(4, 4, 3, 1), (4, 32, 3, 2), (32, 64, 3, 2), (64, 128, 3, 2), (128, 32, 3, 2), (32, 1, 1, 1)])


class Layer(C.Structure):
    _fields_ = [("c_in", C.c_int32), ("c_out", C.c_int32), ("ksize", C.c_int32), ("stride", C.c_int32)]


class Host:
    """The library over the recording runtime."""

    def __init__(self, fake, library):
        self.fake, self.lib = C.CDLL(fake, mode=C.RTLD_GLOBAL), C.CDLL(library)
        self.fake.recorded.restype = C.c_char_p

    def log(self):
        """[("malloc", bytes) or ("launch", kernel, grid)] since the last call."""
        out = []
        self.raw = self.fake.recorded().decode()
        for line in self.raw.splitlines():
            what, *rest = line.split()
            if what == "malloc":
                out.append((what, int(rest[0])))
            else:   # _ZN3lgc15k_encoder_fusedI...: the name is as long as its number says
                digits = rest[0][rest[0].index("lgc") + 3:]
                n = "".join(c for c in digits[:3] if c.isdigit())
                out.append((what, digits[len(n):len(n) + int(n)], [int(x) for x in rest[1:]]))
        return out

    def kernels(self):
        return [x[1] for x in self.log() if x[0] == "launch"]

    def topk(self, ctx, n, k, batch):
        """The template arguments of the streaming pass of one accumulation and selection."""
        self.log()
        assert self.lib.lgc_accumulate_topk(ctx, p(1 << 40), p(1 << 41), p(1 << 42), u64(n), batch, u64(n), C.c_float(0.9), u64(k), p(1 << 43), p(1 << 43), None) == 0
        names = [line.split()[1] for line in self.raw.splitlines() if "k_candidates" in line] if self.log() else []
        return names

    def ctx(self, max_n, max_k, batch):
        h = p()
        assert self.lib.lgc_create(C.byref(h), 0, u64(max_n), u64(max_k), batch) == 0
        return h

    def autoencoder(self, enc, dec):
        weights = (p * 64)(*[1 << 40] * 64)
        h = p()
        assert self.lib.lgc_ae_create(C.byref(h), 0, len(enc), (Layer * len(enc))(*enc), len(dec), (Layer * len(dec))(*dec), C.c_float(0.01),
                                      weights, weights, weights, weights) == 0
        return h

    def encode(self, ctx, ae, vals, k, batch, latent):
        return self.lib.lgc_encode(ctx, ae, p(vals), u64(k), batch, p(latent), None)

    def decode(self, ctx, ae, latent, k, batch, rec):
        return self.lib.lgc_decode(ctx, ae, p(latent), u64(k), batch, p(rec), None)


def paper_stacks_in_place(h):
    k, batch = 1000, 2
    ctx, ae = h.ctx(k, k, batch), h.autoencoder(*PAPER)
    assert h.lib.lgc_reserve(ctx, ae, u64(k), batch, None) == 0
    latent = 4 * batch * 4 * 63             # bytes: 4 channels of 63 positions
    at = 1 << 30
    out = {}
    h.log()
    for name, offset in (("apart", 4 * k * batch), ("same", 0), ("last", 4 * k * batch - 4), ("before", -latent), ("into", 4 - latent)):
        assert h.encode(ctx, ae, at, k, batch, at + offset) == 0
        out["encode " + name] = h.kernels()
    for name, offset in (("apart", latent), ("same", 0), ("last", latent - 4), ("before", -4 * k * batch), ("into", 4 - 4 * k * batch)):
        assert h.decode(ctx, ae, at, k, batch, at + offset) == 0
        out["decode " + name] = h.kernels()
    return out


RECORDS = [  # elements, kept, nodes; whether the rows keep records: measured sizes on either side of each line of the rule
    (1 << 20, 1024, 1, True), (3_333_331, 3333, 3, True), (16_000_000, 16_000, 1, True), (8_000_000, 8000, 4, True), (8_500_000, 8500, 4, False),
    (25_600_000, 25_600, 4, False), (44_500_000, 44_500, 8, False), (1 << 28, 1_610_612, 1, False), (1 << 28, 1_879_048, 1, False),
    (1 << 28, 2_147_483, 1, True), (1 << 28, 2_684_354, 1, True), (44_500_000, 445_000, 8, True), (67_000_000, 536_000, 1, False)]


def records(h):
    out = []
    for n, k, batch, _ in RECORDS:
        h.log()
        ctx = h.ctx(n, k, batch)
        taken = [x[1] for x in h.log() if x[0] == "malloc"]
        passes = h.topk(ctx, n, k, batch)
        h.lib.lgc_destroy(ctx)
        out.append([taken, sorted(set(passes))])
    big = h.ctx(1 << 28, 2_684_354, 2)      # one context for all: what fits a call does not depend on the context's own rows
    out.append([h.topk(big, n, k, batch) for n, k, batch in ((1 << 28, 2_684_354, 2), (1 << 28, 2_684_354, 1), (16_000_000, 16_000, 2), (16_000_000, 16_000, 1))])
    return out


def fall_backs_of_the_one_launch_finish(h):
    """Kernels of selections on a context, the first of which reports a fall-back; the same with every selection that goes
    through the one-launch finish reporting one."""
    out = {}
    for name, max_n, max_k, every in (("larger", 25_600_000, 25_600, False), ("own", 1 << 20, 1000, False), ("larger, each", 25_600_000, 25_600, True)):
        ctx = h.ctx(max_n, max_k, 1)
        words = C.cast(p.in_dll(h.fake, "pinned"), C.POINTER(C.c_uint32))
        seen, reported, numbered = [], False, 0
        for _ in range(140):
            h.topk(ctx, 1 << 20, 1000, 1)
            kernel = "finish" if "k_finish_or_exact" in h.raw else "many" if "k_output_or_exact" in h.raw else "exact"
            numbered += kernel != "exact"            # selections that take the exact path outright report nothing and have no number
            if kernel == "finish" and (every or not reported):
                words[0], reported = numbered, True
            elif kernel != "exact":
                words[1] = numbered
            seen.append(kernel)
        out[name] = seen
        h.lib.lgc_destroy(ctx)
    return out


GATHERS = [  # elements, kept, nodes; which kernel lists the candidates: measured sizes on either side of each line of the rule
    (25_600_000, 25_600, 4, "k_gatherILb1ELb0E"), (33_000_000, 33_000, 1, "k_gatherILb1ELb0E"), (44_500_000, 44_500, 8, "k_gather_piecesILi512ELb0E"),
    (60_000_000, 600_000, 1, "k_gather_piecesILi1024ELb1E"), (60_000_000, 600_000, 2, "k_gather_piecesILi1024ELb1E"),
    (60_000_000, 600_000, 3, "k_gather_piecesILi512ELb0E"), (40_000_000, 200_000, 1, "k_gather_piecesILi512ELb1E"), (40_000_000, 200_000, 2, "k_gather_piecesILi512ELb0E"), (100_000_000, 100_000, 1, "k_gather_piecesILi512ELb0E"),
    (1 << 28, 2_684_354, 1, "k_gather_piecesILi1024ELb0E"), (30_000_000, 300_000, 8, "k_gather_piecesILi1024ELb0E")]


def gathers(h):
    out = []
    for n, k, batch, _ in GATHERS:
        ctx = h.ctx(n, k, batch)
        h.topk(ctx, n, k, batch)
        out.append([line.split()[1] for line in h.raw.splitlines() if "k_gather" in line])
        h.lib.lgc_destroy(ctx)
    for n in (25_600_000, 44_500_000):       # by layers: two halves
        ctx, seg = h.ctx(n, n // 1000, 4), p()
        assert h.lib.lgc_segments_create(C.byref(seg), 0, u64(n), u64(2), (u64 * 3)(0, n // 2, n), (u64 * 2)(n // 2000, n // 2000)) == 0
        assert h.lib.lgc_reserve(ctx, None, u64(0), 0, seg) == 0
        h.log()
        assert h.lib.lgc_topk_segmented(ctx, seg, p(1 << 42), None, 4, u64(n), p(1 << 43), p(1 << 43), None) == 0
        h.log()
        out.append([line.split()[1] for line in h.raw.splitlines() if "k_gather" in line or "k_group" in line])
    return out


def zeros(h):
    """The kernels with a form for zeros from the pass, of selections with long lists: records, none, records and no carried thresholds."""
    out = []
    for n, k, carry in ((1 << 28, 2_684_354, 1), (67_000_000, 536_000, 1), (1 << 28, 2_684_354, 0)):
        ctx = h.ctx(n, k, 1)
        assert h.lib.lgc_set_option(ctx, 2, C.c_int64(carry)) == 0
        h.topk(ctx, n, k, 1)
        out.append(sorted({line.split()[1] for line in h.raw.splitlines() if any(x in line for x in ("k_sample", "k_emit_scanned", "k_candidates"))}))
        h.lib.lgc_destroy(ctx)
    return out


def who_samples(h):
    """One letter per selection of 2^20 elements: l, a launch samples before the pass; p, the pass takes the carried threshold or samples."""
    ctx = h.ctx(1 << 28, 1 << 18, 4)
    words = C.cast(p.in_dll(h.fake, "pinned"), C.POINTER(C.c_uint32))
    capturing = C.c_int.in_dll(h.fake, "capturing")
    numbered = 0

    def run(outcomes, n=1 << 20, k=1000, batch=1):
        nonlocal numbered
        seen = ""
        for word in outcomes:
            h.topk(ctx, n, k, batch)
            numbered += 1
            if word is not None:
                words[word] = numbered
            seen += "l" if "k_sample" in h.raw else "p"
        return seen

    out = {"served, nothing carried": run([1] * 30), "carried": run([2] * 20), "carried, long vector": run([2], 1 << 28)}
    run([2] * 16)
    out["once not, by one node of two"] = run([1]) + run([2] * 18)
    out["once not seen yet"] = run([None, 2])
    out["a carried one fell back"] = run([3]) + run([2] * 17)
    out["another length"] = run([2] * 18, (1 << 20) + 1)
    out["another count"] = run([2] * 18, (1 << 20) + 1, 1001)
    out["four nodes"] = run([2] * 66, batch=4)
    out["one of them, unseen"] = run([None] * 3)
    out["and four again"] = run([None] * 2 + [2], batch=4)
    run([2] * 16)
    capturing.value = 1
    out["recorded"] = run([2])
    capturing.value = -1
    out["no answer to that"] = run([2])
    capturing.value = 0
    out["not recorded"] = run([2])
    assert h.lib.lgc_set_option(ctx, 0, C.c_int64(1)) == 0      # LGC_OPT_SELECT_PATH: exact, which carries nothing
    h.topk(ctx, 1 << 20, 1000, 1)
    assert h.lib.lgc_set_option(ctx, 0, C.c_int64(0)) == 0
    out["after an exact selection"] = run([2] * 17)
    assert h.lib.lgc_set_option(ctx, 2, C.c_int64(0)) == 0      # LGC_OPT_CARRY_THRESHOLD
    out["option off"] = run([1] * 2)
    h.lib.lgc_destroy(ctx)
    return out


SHARED = [  # values, nodes; blocks per run of 15 positions: on either side of what 256 compute units have room for
    (1_023, 1, 4), (240, 64, 4), (241, 32, 4), (240, 65, 2), (240, 128, 2), (15_360, 2, 2), (15_361, 2, 1)]


def shared_runs(h):
    """Per (values, nodes) of an encode, as one that is recorded in a graph would hold it: blocks per run, and the bytes still allocated where its
    blocks meet (sums, counts) after larger reservations."""
    max_k = 1_000_000
    ctx, ae = h.ctx(max_k, max_k, 128), h.autoencoder(*PAPER)
    shares, allocated = h.fake.encoder_shares, h.fake.allocated_from
    shares.restype, allocated.restype = p, C.c_size_t
    out, held = [], []
    for k, batch, _ in SHARED:
        assert h.lib.lgc_reserve(ctx, ae, u64(k), batch, None) == 0
        h.log()
        assert h.encode(ctx, ae, 1 << 40, k, batch, 1 << 41) == 0
        (_, kernel, grid), = h.log()
        out.append([kernel, grid])
        held.append([shares(0), shares(1)])
    assert h.lib.lgc_reserve(ctx, ae, u64(max_k), 8, None) == 0
    return [x + [allocated(u64(a or 0)) for a in addresses] for x, addresses in zip(out, held)]


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    """Every scenario (a function above, by name), run in one process of its own."""
    from paper_2103_08870_amd import build
    library = build.build(force=False)
    fake = str(tmp_path_factory.mktemp("hip") / "librecording_hip.so")
    r = subprocess.run([build._hipcc(), "-O1", "-std=c++17", "-shared", "-fPIC", "--offload-arch=gfx950", os.path.join(HERE, "recording_hip.cpp"), "-o", fake],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([sys.executable, os.path.abspath(__file__), fake, library], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


def test_paper_stacks_in_place_go_layer_by_layer(answers):
    # a stack in one launch writes outputs while other blocks still read inputs; the last of several launches does not
    for name, kernels in answers["paper_stacks_in_place"].items():
        fused = kernels in (["k_encoder_fused"], ["k_decoder_fused"])
        assert fused == (name.split()[1] in ("apart", "before")), (name, kernels)
        assert fused or len(kernels) >= 3, (name, kernels)


def test_records_are_kept_and_allocated_where_the_rule_asks_for_them(answers):
    *single, shared = answers["records"]
    for (n, k, batch, wanted), (taken, passes) in zip(RECORDS, single):
        assert passes and all(("ELb1EEEv" in x) == wanted for x in passes), (n, k, batch, passes)
        rows, room = -(-n // 1024) * batch, sum(taken[1:]) / 256
        # room for what a call within the context's limits can keep records of: no more than 32 K rows and one per node (2^25
        # elements in all), or 4096 rows per node, unless the lists are dense
        assert room >= rows if wanted else room <= min(rows, max(2 ** 15 + batch, 4096 * batch)), (n, k, batch, taken)
    assert [all("ELb1EEEv" in x for x in passes) for passes in shared] == [True, True, True, True]


def test_fall_backs_of_the_one_launch_finish(answers):
    got = answers["fall_backs_of_the_one_launch_finish"]
    # a context that holds longer lists uses them; one of the selection's own size holds no more and takes the exact path once
    assert got["larger"] == ["finish"] + ["many"] * 64 + ["finish"] * 75
    assert got["own"] == ["finish", "exact"] + ["finish"] * 138
    assert got["larger, each"] == (["finish"] + ["many"] * 64) * 2 + ["finish"] + ["many"] * 9


def test_how_the_candidates_are_listed(answers):
    for (n, k, batch, wanted), got in zip(GATHERS, answers["gathers"]):
        assert len(got) == 1 and wanted in got[0], (n, k, batch, got)
    short, long = answers["gathers"][len(GATHERS):]
    assert len(short) == 1 and "k_gatherILb0ELb0E" in short[0], short
    assert len(long) == 2 and "k_group_counts" in long[0] and "k_gatherILb0ELb1E" in long[1], long


def test_only_selections_with_zeros_from_the_pass_take_the_kernels_that_know_of_them(answers):
    for got, yes in zip(answers["zeros"], (True, False, False)):
        emit, (sample, passes) = [x for x in got if "k_emit" in x], sorted((x for x in got if "k_emit" not in x), key=lambda x: "k_cand" in x)
        assert ["k_emit_scannedILb1E" in x for x in emit] == [yes] and ("k_sampleILb1ELb1E" in sample) == yes and ("ELb1ELb1EEEv" in passes) == yes, got


def test_the_pass_samples_only_in_a_run_of_carried_thresholds(answers):
    # a run is 16 selections of one shape per node
    assert answers["who_samples"] == {
        "served, nothing carried": "l" * 30, "carried": "l" * 16 + "p" * 4, "carried, long vector": "l",
        "once not, by one node of two": "p" + "l" * 16 + "p" * 2, "once not seen yet": "pp", "a carried one fell back": "p" + "l" * 16 + "p",
        "another length": "l" * 16 + "pp", "another count": "l" * 16 + "pp", "four nodes": "l" * 64 + "pp", "one of them, unseen": "lll",
        "and four again": "lll", "recorded": "l", "no answer to that": "l", "not recorded": "p", "after an exact selection": "l" * 16 + "p", "option off": "ll"}


def test_where_an_encoder_s_blocks_meet_outlives_later_reservations(answers):
    for (k, batch, blocks), (kernel, grid, sums, counts) in zip(SHARED, answers["shared_runs"]):
        runs = -(-(-(-k // 16)) // 15)
        assert kernel == "k_encoder_fused" and grid == [runs, batch, blocks], (k, batch, grid)
        # as much room as the blocks write: 64 channels x 16 positions each, a count per run
        assert blocks == 1 or (sums >= 4096 * runs * batch * blocks and counts >= 4 * runs * batch), (k, batch, sums, counts)


if __name__ == "__main__":
    host = Host(sys.argv[1], sys.argv[2])
    print(json.dumps({f.__name__: f(host) for f in (paper_stacks_in_place, records, fall_backs_of_the_one_launch_finish, gathers, zeros, who_samples, shared_runs)}))
