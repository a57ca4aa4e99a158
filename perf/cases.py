"""The decode-time work this library is used for, as cases that can be timed and compared.

A case is one pass of a serving program over the attention layers of a model: every layer has
its own paged KV pool and page metadata, so that a layer finds its data in HBM and not in the
caches the layer before left warm.  Operations ("op"):

  step     one decode step: append one token per sequence, score, select, attend
           (append_and_decode per layer; the step's lengths are uploaded first, as a scheduler
           does, in one small copy for all layers)
  decode   the same without the append (query_aware_decode), the selection reported
  dense    attention over every cached token (dense_decode_attention): the full-cache path
  build    page metadata of freshly prefilled pools (build_page_meta)
  staged   score_pages, select_topk_pages, sparse_decode_attention with its log-denominators,
           as a quality measurement runs them

"launch" is how the layers' calls are issued: one by one from Python ("eager") or as one
captured graph ("graph").
"""
import math

import torch

from paper_2509_12211_amd import tinyserve as ts

DEVICE = "cuda:0"
OUT_FORMATS = {"f32": (ts.TS_OUT_F32, torch.float32), "bf16": (ts.TS_OUT_BF16, torch.bfloat16)}
HEADROOM = 32           # tokens of append room per sequence

BASE = dict(launch="eager", layers=1, L_min=0, topk=0, frac=0.0, kv="bf16", keys="normal",
            permute=True, keep_first=0, keep_last=0, out="f32")


def _case(name, op, **kw):
    c = dict(BASE, name=name, op=op)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one short sequence, one head, one layer; all of it is latency
        _case("tiny_step", "step", B=1, Hq=1, Hkv=1, d=64, S=16, L=4096, topk=32, permute=False),
        # one user chatting with a TinyLLaMA-shaped model: 22 layers, a short odd context,
        # attention sinks and the newest pages always kept, the output in the next layer's type
        _case("chat_step", "step", layers=22, B=1, Hq=32, Hkv=4, d=64, S=16, L=2999, topk=48,
              keys="offset", keep_first=1, keep_last=2, out="bf16"),
        # a GPT2-345M-shaped batch through all 24 layers, calls issued from Python
        _case("gpt2_345m_step", "step", layers=24, B=8, Hq=16, Hkv=16, d=64, S=16, L=8192, topk=64),
        # a TinyLLaMA-shaped batch through all 22 layers, replayed as a graph
        _case("tinyllama_step_graph", "step", launch="graph", layers=22, B=16, Hq=32, Hkv=4, d=64,
              S=16, L=16384, topk=128, keys="offset"),
        # the same model with the INT8 cache
        _case("tinyllama_int8_step", "step", layers=22, B=16, Hq=32, Hkv=4, d=64, S=16, L=16384,
              topk=128, kv="int8"),
        # long documents: few sequences, 128K tokens each, large pages, correlated keys
        _case("longctx_step", "step", layers=8, B=4, Hq=32, Hkv=4, d=64, S=32, L=131072, topk=128,
              keys="walk"),
        # mid-size ragged GQA batch in FP16: neither few nor many (sequence, head) units
        _case("gqa_fp16_step", "step", layers=8, B=24, Hq=32, Hkv=8, d=128, S=16, L=8192, L_min=512,
              frac=0.25, kv="fp16"),
        # the large ragged serving batch, the most work of all
        _case("ragged_step", "step", layers=1, B=64, Hq=32, Hkv=32, d=128, S=16, L=32768, L_min=1024,
              frac=0.25),
        # a second query over caches that stay as they are, large heads and pages, the selection
        # handed back to the caller
        _case("gqa_decode_report", "decode", launch="graph", layers=8, B=7, Hq=32, Hkv=8, d=128, S=32,
              L=50001, L_min=4096, frac=0.1),
        # the full-cache path of the GPT2-345M-shaped batch
        _case("gpt2_345m_dense", "dense", layers=12, B=8, Hq=16, Hkv=16, d=64, S=16, L=8192),
        # page metadata after prefilling the TinyLLaMA-shaped batch, half of the layers
        _case("tinyllama_build", "build", layers=11, B=16, Hq=32, Hkv=4, d=64, S=16, L=16384,
              keys="offset"),
        # the staged calls at another page size
        _case("staged_pages8", "staged", layers=6, B=16, Hq=32, Hkv=4, d=64, S=8, L=16384, topk=256),
    ]


# (query heads, KV heads) of models in use: multi-head, grouped, one KV head
HEADS = [(1, 1), (8, 8), (12, 12), (16, 16), (32, 32), (8, 1), (12, 4), (16, 2), (32, 4), (32, 8),
         (40, 8), (64, 8)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit_pool, limit_bytes = 6 << 30, work(_largest())["bytes"]
    while True:
        op = rng.choices(["step", "decode", "dense", "build", "staged"], [8, 2, 1, 1, 1])[0]
        Hq, Hkv = rng.choice(HEADS)
        c = dict(BASE, op=op, Hq=Hq, Hkv=Hkv, d=rng.choice([64, 128]),
                 S=rng.choices([4, 8, 16, 32, 64], [1, 1, 6, 3, 1])[0], B=_log_int(rng, 1, 64),
                 L=_log_int(rng, 1024, 131072), layers=_log_int(rng, 1, 24))
        if rng.random() < 0.5:
            c["L_min"] = max(64, int(c["L"] * rng.uniform(0.03, 0.9)))
        if op not in ("dense", "build"):
            if c["L_min"] or rng.random() < 0.3:
                c["frac"] = round(rng.uniform(0.05, 0.5), 3)
            else:
                c["topk"] = max(4, min(1024, int(_pages(c) * math.exp(rng.uniform(math.log(0.03), math.log(0.5))))))
            if rng.random() < 0.25:
                c["keep_first"], c["keep_last"] = 1, rng.choice([1, 2, 4])
        c["kv"] = rng.choices(["bf16", "fp16", "int8"], [5, 3, 2])[0]
        c["keys"] = rng.choice(["normal", "offset"])
        c["launch"] = rng.choice(["eager", "graph"])
        c["out"] = rng.choice(["f32", "f32", "bf16"])
        if _pages(c) <= 16384 and _pool_bytes(c) <= limit_pool and work(c)["bytes"] <= limit_bytes:
            return c


def _largest():
    return next(c for c in listed() if c["name"] == "ragged_step")


def _pages(c):
    """Rows of the block table: the pages of the longest sequence, append room included."""
    return -(-(c["L"] + HEADROOM) // c["S"])


def _mean_lens(c):
    """The sequence lengths a seed draws, with each draw at the middle of its share of the range."""
    if not c["L_min"]:
        return [c["L"]] * c["B"]
    span = c["L"] - c["L_min"]
    return [c["L_min"] + int(span * (i + 0.5) / c["B"]) for i in range(c["B"])]


def _pool_pages(c):
    """Pages of a layer's pool: room for every draw of the lengths, whatever the seed."""
    span = c["L"] - c["L_min"] if c["L_min"] else 0
    longest = [c["L"] - span + -(-span * (i + 1) // c["B"]) for i in range(c["B"])]
    return sum(-(-(n + HEADROOM) // c["S"]) for n in longest)


def _pool_bytes(c):
    tok = c["Hkv"] * (2 * c["d"] + 8 if c["kv"] == "int8" else 4 * c["d"])
    return c["layers"] * tok * c["S"] * _pool_pages(c)


def _k_max(c):
    return c["topk"] if c["topk"] else int(math.ceil(c["frac"] * _pages(c))) + 1


def _kept(c, pages):
    """Pages selected of a sequence with that many."""
    return min(pages, c["topk"] if c["topk"] else max(1, math.ceil(c["frac"] * pages)))


def work(case):
    c, d = case, case["d"]
    grow = 1 if c["op"] == "step" else 0
    lens = [n + grow for n in _mean_lens(c)]
    pages = [-(-n // c["S"]) for n in lens]
    out_bytes = c["B"] * c["Hq"] * d * (2 if c["out"] == "bf16" else 4)
    q_bytes = c["B"] * c["Hq"] * d * 2
    tok = 2 * d + 8 if c["kv"] == "int8" else 4 * d
    heads = c["Hkv"]
    meta = heads * 4 * d * sum(pages)
    if c["op"] == "build":
        key_tok = d + 4 if c["kv"] == "int8" else 2 * d
        return {"bytes": c["layers"] * (heads * key_tok * sum(lens) + meta),
                "flops": c["layers"] * heads * 2 * d * sum(lens)}
    if c["op"] == "dense":
        return {"bytes": c["layers"] * (heads * tok * sum(lens) + q_bytes + out_bytes),
                "flops": c["layers"] * 4 * c["Hq"] * d * sum(lens)}
    kept = sum(min(n, _kept(c, p) * c["S"]) for n, p in zip(lens, pages))
    by = meta + heads * tok * kept + q_bytes + out_bytes
    if c["op"] == "step":   # the new tokens in, their rows and boxes out
        by += c["B"] * heads * (2 * tok + 4 * d)
    if c["op"] == "staged":   # scores and the selection are results too
        by += c["B"] * heads * 4 * (_pages(c) + _k_max(c))
    return {"bytes": c["layers"] * by,
            "flops": c["layers"] * (heads * 4 * d * sum(pages) + 4 * c["Hq"] * d * kept)}


def tolerance(case):
    if case["op"] == "build":
        return "exact"
    # outputs are fp32 sums over 16-bit (or 8-bit) inputs with the softmax weights carried to
    # about 16 bits; a bf16 output may round the other way (half an ulp is 2^-9)
    if case["out"] == "bf16":
        return {"rel": 2e-3, "max": 1e-2, "differ": 1e-4}
    return {"rel": 1e-4, "max": 2e-3, "differ": 1e-4}


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _lens(c, seed):
    g = torch.Generator()
    g.manual_seed(int(seed) + 70)
    if not c["L_min"]:
        return torch.full((c["B"],), c["L"], dtype=torch.int64)
    span = c["L"] - c["L_min"]
    at = (torch.arange(c["B"]) + torch.rand(c["B"], generator=g)) / c["B"]
    return (c["L_min"] + (span * at).to(torch.int64))[torch.randperm(c["B"], generator=g)]


def _fill_walk(c, k_pool, table, lens, g):
    """Keys that drift along the sequence: a slow random walk per channel plus noise."""
    for b, n in enumerate(lens.tolist()):
        x = torch.randn((c["Hkv"], n, c["d"]), generator=g, device=DEVICE).mul_(0.05).cumsum_(1)
        x.add_(torch.randn(x.shape, generator=g, device=DEVICE), alpha=0.5)
        whole = n // c["S"]
        rows = table[b, :whole].to(torch.int64)
        x = x[:, :whole * c["S"]].view(c["Hkv"], whole, c["S"], c["d"])
        k_pool[rows] = x.permute(1, 0, 2, 3).to(k_pool.dtype)


class _Layer:
    """One layer's cache, metadata and this step's rows, as a model runner holds them."""

    def __init__(self, c, seed, lens, table, lens_row, out_row):
        g = _generator(seed)
        B, Hkv, d, S = c["B"], c["Hkv"], c["d"], c["S"]
        n_phys = _pool_pages(c)
        e16 = torch.float16 if c["kv"] == "fp16" else torch.bfloat16
        shape = (n_phys, Hkv, 2, S * d)
        self.k_scale = self.v_scale = None
        if c["kv"] == "int8":
            self.kv = torch.randint(-127, 128, shape, generator=g, device=DEVICE, dtype=torch.int8)
            self.k_scale, self.v_scale = (
                torch.rand((n_phys, Hkv, S), generator=g, device=DEVICE).mul_(0.004).add_(0.012) for _ in range(2))
        else:
            self.kv = torch.empty(shape, dtype=e16, device=DEVICE).normal_(generator=g)
        self.k_pool = self.kv[:, :, 0].view(n_phys, Hkv, S, d)
        self.v_pool = self.kv[:, :, 1].view(n_phys, Hkv, d, S)
        offset = torch.randn((Hkv, d), generator=g, device=DEVICE).mul_(2.0)
        if c["keys"] == "offset" and c["kv"] != "int8":   # outlier channels
            self.k_pool.add_(offset[None, :, None, :].to(e16))
        elif c["keys"] == "walk":
            _fill_walk(c, self.k_pool, table, lens, g)
        rows = [torch.randn((B, n, d), generator=g, device=DEVICE) for n in (c["Hq"], Hkv, Hkv)]
        if c["keys"] == "offset":
            rows[1] += offset[None]
        self.q, self.k_new, self.v_new = (x.to(e16) for x in rows)
        self.page_min = torch.zeros((B, Hkv, _pages(c), d), dtype=e16, device=DEVICE)
        self.page_max = torch.zeros_like(self.page_min)
        self.out = out_row
        self.layout = ts.make_layout(
            B, c["Hq"], Hkv, d, S, _pages(c), self.k_pool, self.v_pool, table, lens_row, self.page_min,
            self.page_max, keep_first_pages=c["keep_first"], keep_last_pages=c["keep_last"],
            out_format=OUT_FORMATS[c["out"]][0], k_scale=self.k_scale, v_scale=self.v_scale)


class _State:
    pass


def prepare(case, seed):
    c, s = case, _State()
    B = c["B"]
    lens = _lens(c, seed)
    per_seq = -(-(lens + HEADROOM) // c["S"])
    g = torch.Generator()
    g.manual_seed(int(seed) + 50)
    n_phys = _pool_pages(c)
    perm = torch.randperm(n_phys, generator=g) if c["permute"] else torch.arange(n_phys)
    table = torch.full((B, _pages(c)), -1, dtype=torch.int32)
    for b, part in enumerate(torch.split(perm[:int(per_seq.sum())], per_seq.tolist())):
        table[b, :part.numel()] = part
    s.case, s.op = c, c["op"]
    s.scale = 1.0 / math.sqrt(c["d"])
    s.table = table.to(DEVICE)
    s.lens_now = lens.to(torch.int32).to(DEVICE).repeat(c["layers"], 1)   # this step's lengths
    s.lens = s.lens_now.clone()                                          # what the layers advance
    s.out = torch.zeros((c["layers"], B, c["Hq"], c["d"]), dtype=OUT_FORMATS[c["out"]][1], device=DEVICE)
    s.layers = [_Layer(c, seed * 1009 + 17 * i + 1, lens, s.table, s.lens[i], s.out[i])
                for i in range(c["layers"])]
    for ly in s.layers:
        ts.build_page_meta(ly.layout)
    s.topk_per_seq, s.topk, s.k_max = None, 0, 0
    if c["op"] in ("step", "decode", "staged"):
        grown = lens + (1 if c["op"] == "step" else 0)
        pages = -(-grown // c["S"])
        s.k_max = _k_max(c)
        s.topk = s.k_max
        if not c["topk"]:
            s.topk_per_seq = torch.ceil(pages.double() * c["frac"]).clamp_(min=1).to(torch.int32).to(DEVICE)
        s.ws = ts.new_workspace(s.layers[0].layout, s.k_max, DEVICE)   # the layers run one after the other
        s.sel = torch.full((c["layers"], B, c["Hkv"], s.k_max), -1, dtype=torch.int32, device=DEVICE)
        s.count = torch.zeros((c["layers"], B), dtype=torch.int32, device=DEVICE)
    elif c["op"] == "dense":
        s.ws = ts.new_dense_workspace(s.layers[0].layout, DEVICE)
    if c["op"] in ("dense", "staged"):
        s.lse = torch.zeros((c["layers"], B, c["Hq"]), device=DEVICE)
    if c["op"] == "staged":
        s.scores = torch.zeros((c["layers"], B, c["Hkv"], _pages(c)), device=DEVICE)
    s.graph = None
    if c["launch"] == "graph":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _calls(s)
            side.synchronize()
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph, stream=side):
                _calls(s)
        torch.cuda.current_stream().wait_stream(side)
    return s


def _calls(s):
    """The layers' calls of one pass, in order, on the current stream."""
    for i, ly in enumerate(s.layers):
        if s.op == "step":
            ts.append_and_decode(ly.layout, ly.k_new, ly.v_new, ly.q, s.topk, s.k_max, s.scale, ly.out,
                                 s.ws, topk_per_seq=s.topk_per_seq)
        elif s.op == "decode":
            ts.query_aware_decode(ly.layout, ly.q, s.topk, s.k_max, s.scale, ly.out, s.ws,
                                  topk_per_seq=s.topk_per_seq, sel_out=s.sel[i], sel_count_out=s.count[i])
        elif s.op == "dense":
            ts.dense_decode_attention(ly.layout, ly.q, s.scale, ly.out, s.ws, lse_out=s.lse[i])
        elif s.op == "build":
            ts.build_page_meta(ly.layout)
        else:
            ts.score_pages(ly.layout, ly.q, s.scores[i])
            ts.select_topk_pages(ly.layout, s.scores[i], s.topk, s.k_max, s.sel[i], s.count[i],
                                 topk_per_seq=s.topk_per_seq)
            ts.sparse_decode_attention(ly.layout, ly.q, s.sel[i], s.count[i], s.k_max, s.scale, ly.out,
                                       s.ws, lse_out=s.lse[i])


def run(state):
    s = state
    if s.op == "step":
        s.lens.copy_(s.lens_now)
    if s.graph is not None:
        s.graph.replay()
    else:
        _calls(s)
    boxes = [t for ly in s.layers for t in (ly.page_min, ly.page_max)]
    if s.op == "build":
        return boxes
    if s.op == "dense":
        return [s.out, s.lse]
    if s.op == "decode":
        return [s.out, s.sel, s.count]
    if s.op == "staged":
        return [s.out, s.lse, s.scores, s.sel, s.count]
    # the step also changed the lengths, the boxes and the pools (the first and the last layer's
    # stand for all: every layer does the same)
    ends = {0, len(s.layers) - 1}
    state_out = [t for i in sorted(ends) for t in (s.layers[i].page_min, s.layers[i].page_max,
                                                   s.layers[i].kv, s.layers[i].k_scale, s.layers[i].v_scale)]
    return [s.out, s.lens] + [t for t in state_out if t is not None]
