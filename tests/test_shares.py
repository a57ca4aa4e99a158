"""The arithmetic by which ragged batches are dealt out to workgroups (csrc/ts_shares.h), on the
CPU: the header is compiled into a small library of its own and the dealing done in Python."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_12211_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SRC = """
#include <hip/hip_runtime.h>
#include "ts_shares.h"
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
    L.members.argtypes = [ctypes.c_int] * 5 + [ctypes.c_float]
    L.members.restype = ctypes.c_float
    return L


def deal(lib, seqs, n, S, exchange=1):
    """Members of each (pages, kept) sequence: the smallest share with which they fit into n."""
    kmax = max(k for _, k in seqs)
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
