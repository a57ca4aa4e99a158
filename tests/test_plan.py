"""The work plan of the fused calls (csrc/tinyserve.hip), on the CPU: the entry-point file is
compiled with stand-ins for the kernels' files and asked what it would launch."""
import ctypes
import os
import subprocess

import pytest

from paper_2509_12211_amd import tinyserve as ts

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_12211_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LDS = 160 << 10   # of a compute unit

# uniform: all sequences have the same budget.  out: members, kept pages of each and LDS bytes, of the
# plan and of what is launched with room for `resident` workgroups; by shares or not
SRC = """
#include "tinyserve.hip"
extern "C" void plan(const ts_layout* L, int max_topk, int uniform, int resident, int* out) {
  ts::Plan pl = ts::make_plan(L, max_topk);
  if (uniform) pl.shares = pl.shares_uniform;
  out[0] = pl.g, out[1] = pl.chunk, out[2] = (int)pl.lds_fused, out[6] = pl.shares;
  ts::fit_clusters(L, max_topk, resident, pl);
  out[3] = pl.g, out[4] = pl.chunk, out[5] = (int)pl.lds_fused;
}
extern "C" int through(const ts_layout* L) { return ts::boxes_through(L); }
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    tmp = tmp_path_factory.mktemp("plan")
    src, so = str(tmp / "plan.hip"), str(tmp / "plan.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-shared", "-fPIC",
                    "-Wno-unknown-warning-option", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", CSRC, src,
                    os.path.join(ROOT, "tests", "sanitize", "format_stubs.hip"), "-o", so],
                   check=True, capture_output=True)
    lib = ctypes.CDLL(so)
    fn = lib.plan

    def ask(B, Hkv, d, S, pages, topk, uniform=True, resident=256, G=1):
        lay = ts.TsLayout(B, Hkv * G, Hkv, d, S, pages, 1)
        out = (ctypes.c_int * 7)()
        fn(ctypes.byref(lay), topk, int(uniform), resident, out)
        return dict(zip(("g", "chunk", "lds", "g_run", "chunk_run", "lds_run", "shares"), out))
    ask.through = lambda B, Hkv, d, S, pages, phys: lib.through(
        ctypes.byref(ts.TsLayout(B, Hkv, Hkv, d, S, pages, phys)))
    return ask


@pytest.mark.parametrize("B,Hkv", [(1, 1), (2, 1), (1, 4), (3, 8), (4, 16)])
def test_what_is_launched_fits_where_its_plan_does(plan, B, Hkv):
    """A call whose plan fits the LDS of a compute unit is not turned away for what is launched in
    its place: clusters of fewer members hold longer lists each."""
    fits = 0
    for S in (4, 16, 64):
        for d in (64, 128):
            for pages in list(range(11003, 16385, 310)) + [14255, 16142, 16384]:
                for topk in {pages // 8, pages // 2, 9345, pages - 1, pages}:
                    for uniform in (True, False):
                        p = plan(B, Hkv, d, S, pages, topk, uniform)
                        if p["lds"] > LDS:
                            continue
                        fits += 1
                        assert p["lds_run"] <= LDS, (B, Hkv, d, S, pages, topk, uniform, p)
                        assert p["g_run"] <= p["g"] and p["chunk_run"] * p["g_run"] >= topk
    assert fits > 100


@pytest.mark.parametrize("S", [8, 16, 32])
@pytest.mark.parametrize("pages,topk", [(250, 256), (250, 1000), (60, 128), (60, 4096), (20, 128), (2, 128), (1, 128)])
def test_no_more_pages_are_kept_than_the_table_has(plan, S, pages, topk):
    """A budget beyond the table's width divides the work like one of the whole table."""
    for B, Hkv in ((4, 4), (1, 4), (1, 1)):
        p = plan(B, Hkv, 64, S, pages, topk)
        assert p["g_run"] >= 2 and p["g_run"] <= p["g"] and p["chunk_run"] * p["g_run"] >= pages
        if pages >= 4 * p["g"]:      # (as many members as fit either way)
            q = plan(B, Hkv, 64, S, pages, pages)
            assert (p["g_run"], p["chunk_run"], p["lds_run"]) == (q["g_run"], q["chunk_run"], q["lds_run"])
        assert p["g_run"] == 2 or (p["g_run"] - 1) * p["chunk_run"] < pages, "a member that never has a page"


@pytest.mark.parametrize("d,S,Hkv", [(64, 4, 4), (64, 16, 4), (128, 8, 8), (128, 16, 1)])
def test_only_rebuilds_of_many_boxes_write_them_through(plan, d, S, Hkv):
    """From 18 MiB of boxes on, by the rows of the tables or the pages of the pool, whichever are
    fewer: 6 to 17 MB of them were 1 to 6 % slower written through."""
    least = (18 << 20) // (4 * d * Hkv)
    for B in (1, 4):
        wide = 2 * least // B
        assert plan.through(B, Hkv, d, S, least // B, 2 * least) == 1
        assert plan.through(B, Hkv, d, S, least // B - 1, 2 * least) == 0
        assert plan.through(B, Hkv, d, S, wide, least) == 1
        assert plan.through(B, Hkv, d, S, wide, least - 1) == 0
        assert plan.through(B, Hkv, d, 32, wide, 2 * least) == 0
