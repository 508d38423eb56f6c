"""The gfx950 assembly of every kernel, as the library's build flags make it: wait states the hardware does not supply,
registers and scratch memory.  And in the sources: no record of a node's selection that gets both atomics and plain stores from one kernel."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2103_08870_amd import build

# gfx940 and later: a vector instruction that reads a scalar register needs two wait states after the vector
# instruction that wrote it.  The compiler inserts them between its own instructions, but not into inline assembly.
WAIT_STATES = 2
TWO_RESULTS = ("v_add_co", "v_addc_co", "v_sub_co", "v_subb_co", "v_subrev_co", "v_subbrev_co", "v_div_scale", "v_mad_u64_u32", "v_mad_i64_i32")


def assembly(source):
    cmd = [build._hipcc()] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", "-"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return r.stdout


def scalar_registers(operand):
    if operand in ("vcc", "vcc_lo", "vcc_hi"):
        return {"vcc": {"vcc_lo", "vcc_hi"}}.get(operand, {operand})
    m = re.fullmatch(r"-?\|?s(\d+)\|?", operand)
    if m:
        return {int(m.group(1))}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    return set(range(int(m.group(1)), int(m.group(2)) + 1)) if m else set()


def short_waits(text):
    """Lines of `text` that read a scalar register too soon after a vector instruction wrote it."""
    found, clock, written = [], 0, {}
    for number, line in enumerate(text.splitlines(), 1):
        words = line.split(";")[0].strip().split(None, 1)
        if not words or words[0].startswith(".") or words[0].endswith(":") or "=" in words[0]:
            continue
        name, operands = words[0], [o.strip() for o in words[1].split(",")] if len(words) > 1 else []
        if name.startswith("v_"):
            results = 2 if name.startswith(TWO_RESULTS) else 1
            for o in operands[results:]:
                if any(clock - written.get(r, -99) < WAIT_STATES + 1 for r in scalar_registers(o)):
                    found.append((number, line.strip()))
        results = operands[:2 if name.startswith(TWO_RESULTS) else 1]
        for o in results:
            for r in scalar_registers(o):
                if name.startswith("v_"):
                    written[r] = clock
                else:
                    written.pop(r, None)
        clock += int(operands[0]) + 1 if name == "s_nop" else 1
    return found


def test_the_check_sees_a_short_wait():
    assert short_waits("v_cmp_ne_u32_e64 s[0:1], 0, v0\nv_writelane_b32 v20, s0, 14\n") == [(2, "v_writelane_b32 v20, s0, 14")]
    assert short_waits("v_cmp_ne_u32_e32 vcc, 0, v0\ns_mov_b32 s4, s5\nv_cndmask_b32_e32 v1, v2, v3, vcc\n")
    assert not short_waits("v_cmp_ne_u32_e64 s[0:1], 0, v0\ns_nop 1\nv_writelane_b32 v20, s1, 14\n")
    assert not short_waits("v_cmp_ne_u32_e64 s[0:1], 0, v0\ns_mov_b32 s0, s5\nv_mov_b32_e32 v20, s0\n")


@pytest.fixture(scope="module")
def listings():
    with ThreadPoolExecutor(max_workers=8) as ex:
        return dict(zip(build.SOURCES, ex.map(assembly, build.SOURCES)))


def resources(text):
    """{kernel: {"vgpr_count": .., ..}} as the listing's metadata has it."""
    found = {}
    for part in text.split("- .agpr_count:")[1:]:
        found[re.search(r"\.name:\s+(\S+)", part)[1]] = {k: int(v) for k, v in re.findall(r"\.(\w+_(?:count|size)):\s+(\d+)", part)}
    return found


def test_no_kernel_keeps_registers_in_memory(listings):
    every = {kernel: r for text in listings.values() for kernel, r in resources(text).items()}
    assert len(every) > 50 and all("vgpr_count" in r for r in every.values())
    # (scalar registers are spilled into the lanes of vector registers, which costs no memory)
    assert {k: r for k, r in every.items() if r["private_segment_fixed_size"] or r["vgpr_spill_count"]} == {}


def test_the_pass_leaves_room_for_seven_wavefronts(listings):
    # 512 vector registers per SIMD, handed out in eights: the flat selection's forms, with and without records or their own sample
    forms = {k: r["vgpr_count"] for k, r in resources(listings["streaming.hip"]).items() if re.search(r"k_candidatesILb[01]ELb0ELb[01]ELb0E", k)}
    assert len(forms) == 8 and max(forms.values()) <= 72, forms


def test_scalar_registers_written_by_vector_instructions_are_waited_for(listings):
    for source, text in listings.items():
        assert source == "api.hip" or text.count("v_cmp") > 0   # (the host side has no kernels)
        assert short_waits(text) == [], source


def functions(text):
    """{name: [body, ..]} of the functions defined at namespace level."""
    text, found, at = re.sub(r"//[^\n]*|__launch_bounds__\([^()]*\)", "", text), {}, 0
    for m in re.finditer(r"^(?!namespace)[\w].*?\b(\w+)\([^;{}]*\)\s*\{", text, re.M):
        if m.start() < at:
            continue
        depth, at = 1, m.end()
        while depth:
            depth += {"{": 1, "}": -1}.get(text[at], 0)
            at += 1
        found.setdefault(m[1], []).append((m[0], text[m.end():at]))
    return found


def test_a_node_s_record_gets_atomics_or_plain_stores_from_a_kernel():
    # Each XCD has an L2 of its own: a line that several of them update by atomics can lose what one of them stores.  `s`, `sel`: a Sel record
    every = {}
    for name in ("device_helpers.h", "carry.h", *build.SOURCES):
        with open(os.path.join(build.CSRC, name)) as f:
            for k, v in functions(f.read()).items():
                every.setdefault(k, []).extend(v)

    def reached(name, seen):
        for _, body in every.get(name, []):
            for other in set(re.findall(r"\b(\w+)(?:<[^;()]*>)?\(", body)) & every.keys() - seen:
                reached(other, seen | {name})
                seen.add(other)
        return seen

    kernels = [k for k, v in every.items() if any("__global__" in head for head, _ in v)]
    assert {"k_gather", "k_gather_pieces", "k_candidates", "k_sample", "k_count_chunks", "k_finish_or_exact"} <= set(kernels)
    record = r"(?:\bs->|\bsel\[[^\]]*\]\.)"
    stored = set()
    for kernel in kernels:
        text = "".join(body for f in {kernel} | reached(kernel, set()) for _, body in every[f])
        atomics, stores = re.findall(r"atomic\w+\(&(?:a\.)?" + record + r"(\w+)", text), re.findall(record + r"(\w+) = ", text)
        assert not (atomics and stores), (kernel, atomics, stores)
        stored |= set(stores) | set(atomics)
    assert {"t_est", "cand_total", "thr", "fast_ok"} <= stored
