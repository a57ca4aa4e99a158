"""Properties of the fused kernel's machine code that cost microseconds when they are lost and
that no functional test notices (CPU only: hipcc cross-compiles gfx950 without a GPU).

The latency-bound builds (one unit per cluster, or one workgroup per unit) must
  - fetch every kernel argument their first loads are addressed with in ONE trip to memory:
    a single wait for scalar loads ahead of the first vector load (scalar registers running
    out at the head of the kernel, or an argument first used behind a branch, brought a second
    and a third trip, 0.1-0.5 us each on every launch), and no trip at all in the builds whose
    leading arguments are in registers when a wave starts;
  - use no scratch memory (a fragment held through a pointer once put 208 bytes per lane
    there: +9 us).
And one that costs nothing but is a race when it is lost: a workgroup counts itself in, which allows
the launch's first workgroup to advance the epoch and the lengths, only behind a barrier that each of its
waves reaches with both words in hand.
"""
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2509_12211_amd import build as tsbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_12211_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# head_dim 64, page size, no loop, append folded in, bf16, clusters: tables of more than 72 groups of
# pages a member
KERNELS = {
    "page 16": "_ZN2ts25query_aware_decode_kernelILi64ELi16ELb0ELb1ELb0ELb0ELb1EEEvNS_11FusedParamsE",
    "page 32": "_ZN2ts25query_aware_decode_kernelILi64ELi32ELb0ELb1ELb0ELb0ELb1EEEvNS_11FusedParamsE",
}
# the builds that look at the lengths first: append folded in and not, clusters and one
# workgroup per unit
SHARES = {
    "shares, append, clusters": "_ZN2ts20shares_decode_kernelILi64ELi16ELb1ELb0ELb1EEEvNS_11FusedParamsE",
    "shares, single": "_ZN2ts20shares_decode_kernelILi64ELi16ELb0ELb0ELb0EEEvNS_11FusedParamsE",
}
# head_dim, page size, append, half, no clusters (shares) and head_dim, page size, no loop, append, int8,
# half, no clusters: one workgroup per unit, 129 to 255 of them
APPEND = ["shares_decode_kernel<64, 16, true, false, false>", "shares_decode_kernel<128, 4, true, false, false>",
          "shares_decode_kernel<64, 32, true, false, false>", "shares_decode_kernel<64, 64, true, false, false>",
          "shares_decode_kernel<128, 32, true, true, false>",
          "query_aware_decode_kernel<128, 16, false, true, false, false, false>",
          "query_aware_decode_kernel<128, 64, false, true, false, false, false>",
          "query_aware_decode_kernel<64, 8, false, true, true, false, false>",
          "query_aware_decode_kernel<64, 32, false, true, true, false, false>",
          "query_aware_decode_kernel<128, 32, false, true, true, false, false>"]
# clusters that take several units in turn, INT8 cache, 128 channels
LOOPING = [f"query_aware_decode_kernel<128, {s}, true, false, true, false, true>" for s in (16, 32, 64)]
# the kernels whose leading arguments are in registers when a wave starts, and their arguments: head_dim,
# page size, append, int8, half, groups of pages a wave; head_dim, page size, half; head_dim, page
# size, int8, half
POINTERS, FIRST = "const uint16_t*, const uint16_t*, const uint16_t*, ", "uint32_t, uint32_t, uint32_t, uint32_t, FusedParams"
PRELOADED = {
    # (the benchmark's shapes run these: the 64-, 16- and 8-sequence ones with up to five groups a wave, the
    # single sequence with one; up to nine are the most there is)
    "one_round_decode_kernel": (POINTERS + "const uint16_t*, const uint16_t*, " + FIRST,
                                ["64, 16, true, false, false, 1", "64, 16, true, false, false, 3",
                                 "64, 16, true, false, false, 5", "64, 16, false, false, false, 5",
                                 "64, 32, true, false, false, 5", "64, 32, true, false, false, 3",
                                 "128, 16, true, false, true, 3", "64, 16, true, true, false, 5",
                                 "64, 16, true, false, false, 9", "64, 16, false, true, false, 9",
                                 "128, 16, true, false, true, 9", "128, 8, true, true, false, 9",
                                 "128, 32, true, true, false, 1", "128, 32, true, true, false, 3",
                                 "128, 64, true, true, false, 5", "128, 32, true, true, false, 9",
                                 "128, 64, true, true, false, 9"]),
    "one_group_dealt_decode_kernel": (POINTERS + "const uint16_t*, const uint16_t*, " + FIRST,
                                      ["64, 16, true, false, false", "128, 16, false, false, true"]),
    "small_units_i8_decode_kernel": (POINTERS + "const int32_t*, const int32_t*, const int32_t*, uint32_t, uint32_t, FusedParams",
                                     ["64, 16", "64, 8", "128, 16", "128, 32"]),
    "small_units_decode_kernel": (POINTERS + "const int32_t*, const int32_t*, const int32_t*, uint32_t, uint32_t, FusedParams",
                                  ["64, 16, false", "128, 16, false", "64, 32, true", "128, 64, false"]),
    "sparse_attention_kernel": ("const uint16_t*, const int32_t*, const int32_t*, const int32_t*, const int32_t*, "
                                "uint32_t, int, int, int, AttendParams, int32_t*, int",
                                ["64, 8, false, false", "128, 16, false, false", "64, 16, true, false"]),
}


def assembly(source):
    """The gfx950 assembly of a .hip file, compiled with the library's own flags."""
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    tmp = tempfile.mkdtemp(prefix="ts_isa_")
    try:
        out = os.path.join(tmp, "kernels.s")
        flags = [f for f in tsbuild.HIPCC_FLAGS if f not in ("-fPIC",)]
        cmd = [HIPCC] + flags + ["-I", CSRC, "--offload-device-only", "-S", source, "-o", out]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout[-2000:]
        with open(out) as f:
            return f.read()
    finally:
        shutil.rmtree(tmp, ignore_errors=True)


@pytest.fixture(scope="module")
def fused_asm():
    return assembly(os.path.join(CSRC, "fmt_bf16_d64.hip"))


@pytest.fixture(scope="module")
def append_asm(tmp_path_factory):
    """The APPEND and LOOPING builds, of several formats, compiled by themselves."""
    src = str(tmp_path_factory.mktemp("isa") / "append.hip")
    with open(src, "w") as f:
        f.write('#include "ts_fused.h"\nnamespace ts {\n' +
                "".join(f"template __global__ void {k}(FusedParams);\n" for k in APPEND + LOOPING) + "}\n")
    return assembly(src)


@pytest.fixture(scope="module")
def preloaded_asm(tmp_path_factory):
    src = str(tmp_path_factory.mktemp("isa") / "preloaded.hip")
    with open(src, "w") as f:
        f.write('#include "ts_fused.h"\nnamespace ts {\n' +
                "".join(f"template __global__ void {k}<{a}>({args});\n"
                        for k, (args, builds) in PRELOADED.items() for a in builds) + "}\n")
    return assembly(src)


def mangled(kernel):
    """The beginning of the symbol of a kernel given as name<integers and truth values>."""
    name, args = kernel[:-1].split("<")
    code = "".join("Lb%dE" % (a == "true") if a in ("true", "false") else "Li%sE" % a for a in args.split(", "))
    return "_ZN2ts%d%sI%sEEv" % (len(name), name, code)


def symbol(asm, kernel):
    m = re.search(r"^(" + re.escape(mangled(kernel)) + r"\w*):", asm, re.M)
    assert m, f"{kernel} not in the assembly"
    return m.group(1)


def kernel_body(asm, symbol):
    m = re.search(r"^" + re.escape(symbol) + r":.*?\n\s*s_endpgm", asm, re.S | re.M)
    assert m, f"{symbol} not in the assembly"
    return [l.strip() for l in m.group(0).split("\n") if l.strip() and not l.strip().startswith(";")]


def descriptor(asm, sym, field):
    m = re.search(r"\.amdhsa_kernel " + re.escape(sym) + r"\n(.*?)\.end_amdhsa_kernel", asm, re.S)
    assert m, "kernel descriptor not found"
    value = re.search(r"\.amdhsa_" + field + r" (\d+)", m.group(1))
    assert value, f"no {field} in the kernel descriptor"
    return int(value.group(1))


def head_of(body):
    """Ahead of the first vector load: trips to memory for kernel arguments that are waited for, scalar
    registers parked in vector lanes, and whether a fetch is still on its way."""
    trips, pending, spills = 0, False, 0
    for line in body:
        if line.startswith(("global_load", "buffer_load", "flat_load")):
            return trips, spills, pending
        if line.startswith("s_load"):
            pending = True
        elif line.startswith("s_waitcnt") and "lgkmcnt" in line and pending:
            trips, pending = trips + 1, False
        elif line.startswith("v_writelane"):
            spills += 1
    pytest.fail("no vector load in the kernel")


@pytest.mark.parametrize("which", sorted(KERNELS))
def test_arguments_arrive_in_one_trip(fused_asm, which):
    trips, spills, pending = head_of(kernel_body(fused_asm, KERNELS[which]))
    assert not pending, "a scalar load ahead of the first vector load is never waited for?"
    assert trips == 1, f"{trips} dependent trips for kernel arguments ahead of the first load"
    assert spills == 0, f"{spills} scalar registers parked in vector lanes ahead of the first load"


@pytest.mark.parametrize("kernel", APPEND)
def test_arguments_of_the_append_builds_arrive_in_one_trip(append_asm, kernel):
    """The builds with the append folded in, whose rare blocks use many arguments late (a parked
    register costs four cycles; it was up to eighteen, and a second trip)."""
    trips, spills, _ = head_of(kernel_body(append_asm, symbol(append_asm, kernel)))
    assert trips == 1, f"{trips} dependent trips for kernel arguments ahead of the first load"
    assert spills <= 2, f"{spills} scalar registers parked in vector lanes ahead of the first load"


@pytest.mark.parametrize("kernel", LOOPING)
def test_looping_int8_builds_use_no_scratch_memory(append_asm, kernel):
    sym = symbol(append_asm, kernel)
    assert descriptor(append_asm, sym, "private_segment_fixed_size") == 0
    assert not any(line.startswith("scratch_") for line in kernel_body(append_asm, sym))


@pytest.mark.parametrize("kernel", [f"{k}<{a}>" for k, (_, builds) in PRELOADED.items() for a in builds])
def test_first_loads_go_out_on_arguments_in_registers(preloaded_asm, kernel):
    """All fourteen words are asked for in the kernel's descriptor, and behind the prologue that hardware
    with that feature skips nothing is waited for ahead of the first vector load."""
    sym = symbol(preloaded_asm, kernel)
    assert descriptor(preloaded_asm, sym, "user_sgpr_kernarg_preload_length") == 14
    body = kernel_body(preloaded_asm, sym)
    entry = next(i for i, line in enumerate(body) if line.split() == [".p2align", "8"])
    trips, spills, _ = head_of(body[entry:])
    assert trips == 0, f"{trips} trips for scalar loads ahead of the first vector load"
    assert spills == 0, f"{spills} scalar registers parked in vector lanes ahead of the first load"
    size = descriptor(preloaded_asm, sym, "private_segment_fixed_size")
    assert size == 0, f"scratch bytes per lane: {size}"


# as in PRELOADED: with and without an append, more than one group of pages a wave in the first five
COUNTED = ["64, 16, true, false, false, 3", "64, 16, true, false, false, 5", "64, 16, false, false, false, 9",
           "128, 16, true, false, true, 9", "64, 16, true, true, false, 5", "64, 16, true, false, false, 1"]
ARRIVALS = "global_atomic_add "   # (the only atomic on memory in these builds)


@pytest.fixture(scope="module")
def counted_asm(tmp_path_factory):
    src = str(tmp_path_factory.mktemp("isa") / "counted.hip")
    args = PRELOADED["one_round_decode_kernel"][0]
    with open(src, "w") as f:
        f.write('#include "ts_fused.h"\nnamespace ts {\n' + "".join(
            f"template __global__ void one_round_decode_kernel<{a}>({args});\n" for a in COUNTED) + "}\n")
    return assembly(src)


def blocks_of(asm, sym):
    """The kernel's basic blocks, as lists of instructions, and the blocks each can go on to."""
    m = re.search(r"^" + re.escape(sym) + r":.*?^\.Lfunc_end", asm, re.S | re.M)
    assert m, f"{sym} not in the assembly"
    blocks, label, name = {}, "entry", {}
    order = ["entry"]
    blocks["entry"] = []
    for line in m.group(0).split("\n")[1:]:
        line = line.split(";")[0].strip()
        if re.match(r"\.LBB\w+:$", line) or (blocks[label] and blocks[label][-1].startswith(("s_cbranch", "s_branch"))):
            label = line[:-1] if line.endswith(":") else "after %d" % len(order)
            blocks[label] = []
            order.append(label)
        if line and not line.startswith("."):
            blocks[label].append(line)
    after = {}
    for i, label in enumerate(order):
        last = blocks[label][-1] if blocks[label] else ""
        target = [last.split()[1]] if last.startswith(("s_cbranch", "s_branch")) else []
        falls = not last.startswith(("s_branch", "s_endpgm", "s_setpc"))
        after[label] = target + ([order[i + 1]] if falls and i + 1 < len(order) else [])
    return blocks, after


@pytest.mark.parametrize("build", COUNTED)
def test_a_workgroup_counts_itself_in_behind_a_barrier(counted_asm, build):
    """On every path to the count a wave has waited for the epoch and the length, which it asks for ahead
    of its metadata (several groups of pages a wave), and has then passed a barrier.  Loads come back
    in order: the two are there once no more are in flight than went out behind the second."""
    blocks, after = blocks_of(counted_asm, symbol(counted_asm, f"one_round_decode_kernel<{build}>"))
    assert sum(line.startswith(ARRIVALS) for b in blocks.values() for line in b) >= 1
    words = set()
    if not build.endswith(" 1"):
        ahead = [line for b in blocks.values() for line in b]      # up to the last group ahead of the sums
        ahead = ahead[:[i for i, line in enumerate(ahead) if line.endswith(" nt")][3]]
        words = {line for line in ahead if line.startswith("global_load_dword ")}
        assert len(words) == 2 and sum("offset:64" in line for line in words) == 1, "the epoch and the length"

    # a path's state, the lower the less is certain: words not yet asked for (one or two), memory
    # operations sent out behind them, both there, a barrier behind that
    ASKED, THERE, BARRIER = 2, 1000, 1001

    def step(s, line):
        if line in words:
            return s + 1
        if line.startswith(("global_", "buffer_", "scratch_", "flat_")) and ASKED <= s < THERE:
            return min(s + 1, THERE - 1)
        if line.startswith("s_waitcnt") and "vmcnt" in line and ASKED <= s < THERE:
            return THERE if int(re.search(r"vmcnt\((\d+)\)", line).group(1)) <= s - ASKED else s
        return BARRIER if line.startswith("s_barrier") and s == THERE else s

    def through(s, label):
        for line in blocks[label]:
            s = step(s, line)
        return s

    state, work = {"entry": ASKED - 2 if words else THERE}, ["entry"]
    while work:
        label = work.pop()
        s = through(state[label], label)
        for nxt in after[label]:
            if s < state.get(nxt, BARRIER + 1):
                state[nxt] = s
                work.append(nxt)
    for label, s in state.items():
        for line in blocks[label]:
            if line.startswith(ARRIVALS):
                assert s == BARRIER, "counted in with no barrier behind the epoch and the length"
            s = step(s, line)


def test_small_clusters_do_not_carry_the_merge_by_slices(tmp_path):
    """One group of pages a wave: clusters of up to eight members, whose last one merges, run a build without the
    merge that larger ones deal out to their members (up to 2 % of the shortest launches); the two barriers
    between the waves that divide a slice's partials are in the other build alone."""
    args = PRELOADED["one_round_decode_kernel"][0]
    kernels = ["one_round_decode_kernel<64, 16, true, false, false, 1>",
               "one_group_dealt_decode_kernel<64, 16, true, false, false>"]
    src = tmp_path / "merges.hip"
    src.write_text('#include "ts_fused.h"\nnamespace ts {\n' +
                   "".join(f"template __global__ void {k}({args});\n" for k in kernels) + "}\n")
    asm = assembly(str(src))
    barriers = [sum(line == "s_barrier" for b in blocks_of(asm, symbol(asm, k))[0].values() for line in b) for k in kernels]
    assert barriers[1] - barriers[0] == 2, barriers


@pytest.mark.parametrize("which", sorted(KERNELS) + sorted(SHARES))
def test_no_scratch_memory(fused_asm, which):
    sym = KERNELS.get(which) or SHARES[which]
    size = descriptor(fused_asm, sym, "private_segment_fixed_size")
    assert size == 0, f"scratch bytes per lane: {size}"
    assert not any(l.startswith("scratch_") for l in kernel_body(fused_asm, sym))
