"""The arithmetic by which ragged batches are dealt out to workgroups (csrc/ts_shares.h), on the
CPU: the header is compiled into a small library of its own and the dealing done in Python."""
import ctypes
import math
import os
import subprocess

import pytest

from paper_2509_12211_amd import workloads as wl

from helpers import goes_by_shares

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_12211_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SRC = """
#include <hip/hip_runtime.h>
#include "ts_shares.h"
extern "C" float even(int P, int Kb, int chunk, int S, int g) { return ts::even_rows(P, Kb, chunk, S, 1.f / g); }
extern "C" int rounds(int total, int longest, int B, int units) { return ts::rounds_of(total, longest, B, units); }
extern "C" int cluster(int units, int most, int P, int K, int S, int d) { return ts::cluster_members(units, most, P, K, S, d); }
extern "C" float cluster_us(int units, int g, int P, int K, int S, int d) {
  const int chunk = ts::chunk_of(K, g, S);
  return ts::cluster_us(units, (K + chunk - 1) / chunk, chunk, P, S, d).all;
}
extern "C" int chunk(int K, int g, int S) { return ts::chunk_of(K, g, S); }
extern "C" float members(int P, int Kb, int Kmax, int S, int exchange, float t) {
  const ts::SeqWork w = ts::seq_work(P, Kb, Kmax, S, exchange != 0);
  return ts::members_of(w, t > w.whole ? 1.f / (t - w.whole) : INFINITY);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    tmp = tmp_path_factory.mktemp("shares")
    src, so = str(tmp / "shares.hip"), str(tmp / "shares.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-shared", "-fPIC",
                    "-Wno-unknown-warning-option", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", CSRC, src, "-o", so], check=True, capture_output=True)
    L = ctypes.CDLL(so)
    L.even.argtypes = [ctypes.c_int] * 5
    L.even.restype = ctypes.c_float
    L.cluster_us.restype = ctypes.c_float
    L.members.argtypes = [ctypes.c_int] * 5 + [ctypes.c_float]
    L.members.restype = ctypes.c_float
    return L


def deal(lib, seqs, n, S, exchange=1, kmax=None):
    """Members of each (pages, kept) sequence: the smallest share with which they fit into n."""
    kmax = kmax or max(k for _, k in seqs)
    lo, hi = 1.0, float(max(p + k * S for p, k in seqs))
    for _ in range(40):
        t = 0.5 * (lo + hi)
        fits = sum(lib.members(p, k, kmax, S, exchange, t) for p, k in seqs) <= n
        lo, hi = (lo, t) if fits else (t, hi)
    return [int(lib.members(p, k, kmax, S, exchange, hi)) for p, k in seqs]


def test_a_long_sequence_with_a_small_budget_is_scored_by_many(lib):
    """8000 pages of which 4 are kept: the scoring is the work, and it is divided."""
    got = deal(lib, [(8000, 4)] + [(100, 100)] * 5, 32, 16)
    assert got[0] >= 10 and sum(got) <= 32 and min(got) >= 1


def test_no_more_members_than_the_longest_list_has_pages_for(lib):
    assert lib.members(8000, 4, 4, 16, 1, 100.0) == 1       # four pages at most: one page per wave
    assert lib.members(8000, 4, 40, 16, 1, 100.0) == 10
    assert lib.members(8000, 4, 4000, 16, 1, 100.0) == 32   # (a limit of its own)
    assert lib.members(0, 0, 40, 16, 1, 100.0) == 1         # an empty sequence has its workgroup


def test_members_that_each_score_everything_divide_only_the_pages_kept(lib):
    assert lib.members(8000, 4, 4000, 16, 0, 100.0) == 1      # nothing to attend for a second one
    assert lib.members(500, 100, 4000, 16, 0, 900.0) == 4     # 1600 rows of tokens, 400 a member
    assert lib.members(500, 100, 4000, 16, 0, 400.0) == 25    # (less than the scoring: the limit)
    assert lib.members(0, 0, 4000, 16, 0, 100.0) == 1
    got = deal(lib, [(512, 128)] * 4 + [(64, 16)] * 12, 32, 16, exchange=0)
    assert got == [5] * 4 + [1] * 12 and sum(got) <= 32       # 512 + 2048 / 5 rows each


@pytest.mark.parametrize("B,Hkv,d,S,L,topk,frac", [(5, 4, 64, 16, 30000, 0, .4), (13, 8, 128, 32, 3500, 0, .3),
                                                    (33, 2, 64, 4, 9000, 0, .3), (24, 8, 128, 16, 8192, 0, .25),
                                                    (7, 8, 128, 32, 50001, 0, .1), (12, 8, 128, 16, 32000, 64, 0)])
def test_model_of_the_rule_deals_like_the_header(lib, B, Hkv, d, S, L, topk, frac):
    """helpers.goes_by_shares, which the GPU tests ask which way a case goes, against the header."""
    spec = wl.WorkloadSpec("m", B, Hkv, Hkv, d, S, L, topk)
    P_max = -(-L // S)
    lens = [1 + (L - 1) * i // (B - 1) for i in range(B)]
    K_max = topk if topk else math.ceil(frac * P_max) + 1
    budgets = topk if topk else [max(1, math.ceil(frac * -(-n // S))) for n in lens]
    went, members = goes_by_shares(spec, P_max, K_max, lens, budgets)
    assert went
    g = max(1, min(256 // (B * Hkv), (K_max + 3) // 4))
    seqs = [(-(-n // S), min(k, -(-n // S))) for n, k in zip(lens, budgets if frac else [topk] * B)]
    want = deal(lib, seqs, 256 // Hkv, S, 1 if g > 1 else 0, K_max)
    assert members == want and sum(members) <= 256 // Hkv
    # alike lengths, whatever the table has room for: nothing to deal out
    same = [L // 2] * B
    assert not goes_by_shares(spec, P_max, K_max, same, topk if topk else [K_max // 2] * B)[0]


def test_rows_of_an_even_cluster(lib):
    assert lib.even(1024, 128, 32, 16, 4) == 256 + 512      # a quarter of the scoring, 32 pages
    assert lib.even(1024, 4, 32, 16, 4) == 256 + 64         # fewer kept than a member's piece
    assert lib.even(512, 128, 128, 16, 1) == 512 + 2048


def test_one_budget_for_all_needs_metadata_to_gain_by():
    """The same kept pages everywhere: only the metadata differ, and short tables have little."""
    spec = wl.WorkloadSpec("m", 16, 32, 4, 64, 16, 16384, 128)
    lens = [1000 + 1000 * i for i in range(16)]
    assert goes_by_shares(spec, 1026, 128, lens, 128) == (False, None)            # not even asked
    assert goes_by_shares(spec, 1026, 128, lens, [128] * 16)[1] is not None


WHOLE, HALVES, FEW_LONG = 0, 1, 2


@pytest.mark.parametrize("pages,Hkv,want", [
    ([256] * 64, 8, WHOLE),                      # even, two full rounds
    ([125] * 68, 8, HALVES),                     # even, a last round of 32
    ([125] * 75, 9, WHOLE),                      # even, a last round of 163
    ([10 * i + 100 for i in range(68)], 8, WHOLE),   # ragged: the rounds do not end together anyway
    ([1000] * 3 + [50] * 61, 8, FEW_LONG),
    ([0] * 64, 8, WHOLE),                        # nothing cached at all
])
def test_rounds_of_whole_or_divided_units_go_by_the_lengths(lib, pages, Hkv, want):
    """The full-cache path over two rounds of units and more; the pool and the table's width have
    no say (a pool of B full tables let a few long sequences decide the finish time)."""
    assert lib.rounds(sum(pages), max(pages), len(pages), len(pages) * Hkv) == want


@pytest.mark.parametrize("S", [4, 8, 16, 32, 64])
def test_members_of_clusters_of_one_size(lib, S):
    """No more members than the plan has room for, never one, every kept page in somebody's chunk; a
    short list leaves compute units alone, a long one over long rows takes all of them."""
    for units in (1, 4, 16, 32, 64, 128):
        for P in (1, 7, 250, 1000, 16384):
            for K in (5, 48, 250, 2000):
                most = min(256 // units, (K + 3) // 4, 64)
                if most < 2:
                    continue
                for d in (64, 128):
                    g = lib.cluster(units, most, P, K, S, d)
                    chunk = lib.chunk(K, g, S)
                    assert 2 <= g <= most and chunk * g >= K and (S >= 16 or chunk % 4 == 0)
    assert lib.cluster(4, 63, 1000, 250, S, 64) < 40
    assert lib.cluster(64, 4, 4000, 1000, S, 128) == 4


@pytest.mark.parametrize("units", [1, 3, 4, 16, 40, 85])
def test_search_for_the_cluster_size_ends_early_at_the_best(lib, units):
    """Sizes that are passed over divide the list like one that was looked at, or are no better."""
    for S in (4, 8, 16, 64):
        for d in (64, 128):
            for P in (1, 60, 257, 1000, 4098, 16384):
                for K in (9, 33, 48, 250, 1500, 9345):
                    most = min(256 // units, (K + 3) // 4, 64)
                    if most < 2:
                        continue
                    us = [lib.cluster_us(units, g, P, K, S, d) for g in range(2, most + 1)]
                    assert lib.cluster_us(units, lib.cluster(units, most, P, K, S, d), P, K, S, d) == min(us)
