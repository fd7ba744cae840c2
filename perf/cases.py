"""The calls whose speed matters to a user of this library, at the sizes they are made with.

A case is one pass of one of five programs, through the entry points of paper_2502_15734_amd.Context:

  step     a request from cached chunks to attention output: cc_rope_shift -> cc_select -> cc_sparse_prefill
  score    the first layer's half of it for a batch: cc_rope_shift -> cc_select
  layer    every later layer for a batch: the chunks are re-positioned, the rows to recompute come from the
           score list that a chunk's metadata keeps, then the partial prefill (cc_rope_shift or cc_rope_place ->
           [cc_gather_rows, cc_scatter_kv for chunks without a cache] -> cc_select_from_scores ->
           cc_sparse_prefill or cc_sparse_prefill_mass)
  decoder  a whole decoder layer for the recomputed rows: cc_gather_rows, cc_rope_shift, cc_rms_norm,
           cc_qkv_project, cc_sparse_prefill, cc_linear, cc_rms_norm, cc_gated_linear, cc_linear
  build    the full prefill that makes chunk-caches and their metadata: cc_sparse_prefill_pairs with every token

The batch programs are two (score, layer) because two correct scorings may order two nearly equal scores
differently, and every row behind such a pair would then be another one; a single request's step is whole.

Sizes, head geometries and value distributions are those of workload.config_spec(1..5) and of the decoder
layers that bench.py times; `draw` spreads them over the ranges between the smallest and the largest.
"""
import math
import random

import numpy as np
import torch

import paper_2502_15734_amd as P

BLOCK = 16
DEVICE = "cuda"


# ---- the cases -----------------------------------------------------------------------------------------
# requests, chunks (of one request), len (tokens of a chunk), question and frac (share of a chunk's tokens that is
# recomputed) are ranges, lo = hi where a workload has one size; store > 0: chunks come from that many stored ones
# by Zipf popularity, so requests share them; layout: seed of the batch's structure.
def _case(program, *, dtype="bf16", heads=(32, 8), dim=128, requests=1, chunks=(5, 5), length=(512, 512), question=(64, 64),
          frac=(0.15, 0.15), store=0, layout=1, mass=False, unrotated=False, miss=0, hidden=0, ffn=0, name=None):
    c = dict(program=program, dtype=dtype, q_heads=heads[0], kv_heads=heads[1], head_dim=dim, requests=requests,
             chunks_lo=chunks[0], chunks_hi=chunks[1], len_lo=length[0], len_hi=length[1], question_lo=question[0],
             question_hi=question[1], frac_lo=frac[0], frac_hi=frac[1], store=store, layout=layout, mass=mass,
             unrotated=unrotated, miss=miss, hidden=hidden, ffn=ffn)
    if name is not None:
        c["name"] = name
    return c


def listed():
    batch = dict(requests=32, chunks=(5, 10), length=(256, 1024), question=(32, 128), frac=(0.05, 0.40), store=200)
    big = dict(heads=(64, 8), requests=8, chunks=(10, 10), length=(1024, 1024), question=(128, 128), frac=(0.10, 0.10))
    long = dict(requests=4, chunks=(32, 32), length=(1000, 1000), question=(256, 256), frac=(0.10, 0.10))
    return [
        # the tiny fp32 workload: what every user runs first and what checks run against; all latency
        _case("step", dtype="f32", heads=(4, 2), dim=64, chunks=(3, 3), length=(64, 64), question=(16, 16), frac=(0.2, 0.2),
              name="tiny_fp32_step"),
        # one user, one question over five retrieved chunks, 8B model: time to first token is what counts
        _case("step", name="8b_single_step"),
        # the same request through a whole decoder layer
        _case("decoder", hidden=4096, ffn=14336, name="8b_single_decoder"),
        # 70B, one request whose unfocused chunks are settled: few rows, the weights stream past them
        _case("decoder", heads=(64, 8), chunks=(5, 5), length=(600, 900), question=(40, 40), frac=(0.05, 0.05), hidden=8192,
              ffn=28672, name="70b_few_rows_decoder"),
        # continuous batching, 8B: scores of the first layer ...
        _case("score", **batch, name="8b_batch_score"),
        # ... and a later layer, with the question's attention to every chunk (it decides which chunks stay in focus)
        _case("layer", mass=True, **batch, name="8b_batch_layer"),
        # a few requests on a store that keeps keys without rotation; one chunk of each has no cache yet
        _case("layer", unrotated=True, miss=1, requests=6, chunks=(4, 9), length=(200, 900), question=(20, 100),
              frac=(0.05, 0.40), name="8b_unrotated_miss_layer"),
        # 70B layer on one of four tensor-parallel shards
        _case("layer", **dict(big, heads=(16, 2)), name="70b_tp4_layer"),
        # 70B layer, all heads
        _case("layer", **big, name="70b_layer"),
        # 32k prompts: scores, and a whole decoder layer
        _case("score", **long, name="8b_32k_score"),
        _case("decoder", hidden=4096, ffn=14336, **long, name="8b_32k_decoder"),
        # prompts seen for the first time: full prefill, chunk-cache metadata
        _case("build", requests=4, chunks=(5, 10), length=(256, 1024), question=(32, 128), frac=(1.0, 1.0), name="8b_cache_build"),
    ]


_COST_CAP = None


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case out of the ranges the listed ones stand for."""
    global _COST_CAP
    if _COST_CAP is None:
        _COST_CAP = max(_cost(c) for c in listed())
    while True:
        c = _draw_any(rng)
        if _cost(c) <= _COST_CAP:
            return c


def _draw_any(rng):
    program = rng.choice(["step", "step", "score", "layer", "layer", "decoder", "decoder", "build"])
    layout = rng.randrange(1 << 20)
    f0 = rng.uniform(0.03, 0.2)
    frac = (f0, f0 + rng.choice([0.0, rng.uniform(0.0, 0.25)]))

    def span(lo, hi):                                  # a range of sizes, now and then a single one
        a = _log_int(rng, lo, hi)
        return (a, a) if rng.random() < 0.4 else tuple(sorted((a, _log_int(rng, lo, hi))))

    if program == "step" and rng.random() < 0.4:       # fp32
        return _case("step", dtype="f32", heads=rng.choice([(4, 2), (8, 2)]), dim=64, requests=rng.choice([1, 1, 2, 3]),
                     chunks=span(2, 5), length=span(17, 200), question=span(4, 40), frac=frac, layout=layout)
    if program == "step":
        return _case("step", heads=rng.choice([(32, 8), (64, 8), (16, 2)]), chunks=span(2, 10), length=span(60, 1024),
                     question=span(6, 128), frac=frac, layout=layout)
    if program == "decoder":
        model = rng.choice([dict(heads=(32, 8), hidden=4096, ffn=14336), dict(heads=(64, 8), hidden=8192, ffn=28672)])
        return _case("decoder", requests=_log_int(rng, 1, 12), chunks=span(2, 16), length=span(60, 1024), question=span(6, 256),
                     frac=frac, layout=layout, **model)
    requests = _log_int(rng, 1, 32)
    heads = rng.choice([(32, 8), (32, 8), (64, 8), (16, 2), (8, 2)])
    sizes = dict(heads=heads, requests=requests, chunks=span(2, 32), length=span(60, 1024), question=span(6, 256), layout=layout)
    if program == "build":
        return _case("build", frac=(1.0, 1.0), **dict(sizes, requests=_log_int(rng, 1, 8), chunks=span(2, 10)))
    if program == "score":
        return _case("score", frac=frac, store=200 if requests > 8 and rng.random() < 0.5 else 0, **dict(sizes, chunks=span(2, 32)))
    unrotated = rng.random() < 0.25
    return _case("layer", frac=frac, unrotated=unrotated, miss=int(unrotated and rng.random() < 0.5),
                 mass=not unrotated and rng.random() < 0.5, store=200 if requests > 8 and rng.random() < 0.5 else 0, **sizes)


# ---- structure of a batch ------------------------------------------------------------------------------
class _Layout:
    """Requests, segments and page counts of a case, from its layout seed alone."""

    def __init__(self, c):
        rng = random.Random(c["layout"])
        span = lambda key: rng.randint(c[key + "_lo"], c[key + "_hi"])
        full = c["program"] == "build"
        n_store = c["store"]
        self.store_len = [span("len") for _ in range(n_store)]
        weights = [(i + 1) ** -1.1 for i in range(n_store)]
        self.segments, self.descs, self.missing = [], [], []   # rows of cc_segment; (stored chunk, first page, tokens, new position)
        self.req_seg_off, self.cu_q = [0], [0]
        tab = tok = sel = 0
        for r in range(c["requests"]):
            k = span("chunks")
            if n_store:
                k = min(k, n_store)
                ids = []
                while len(ids) < k:
                    i = rng.choices(range(n_store), weights)[0]
                    if i not in ids:
                        ids.append(i)
            else:
                ids = []
                for _ in range(k):
                    ids.append(len(self.store_len))
                    self.store_len.append(span("len"))
            missed = set(rng.sample(range(k), min(c["miss"], k - 1)))
            pos = 0
            for j, i in enumerate(ids):
                n = self.store_len[i]
                ns = n if full else min(n, math.ceil(rng.uniform(c["frac_lo"], c["frac_hi"]) * n - 1e-9))
                if j in missed:
                    self.missing.append(len(self.segments))
                elif not full:
                    self.descs.append((i, tab, n, pos))
                self.segments.append((r, 0, pos, n, tab, ns, tok, sel))
                pos, tab, tok, sel = pos + n, tab + -(-n // BLOCK), tok + n, sel + ns
            m = span("question")
            self.segments.append((r, 1, pos, m, tab, m, tok, sel))
            tab, tok, sel = tab + -(-m // BLOCK), tok + m, sel + m
            self.req_seg_off.append(len(self.segments))
            self.cu_q.append(sel)
        self.n_pages, self.n_tok, self.n_rows = tab, tok, sel
        self.cached_at = [rng.randrange(0, 31000) for _ in self.store_len]
        self.max_rows_per_req = max(b - a for a, b in zip(self.cu_q, self.cu_q[1:]))
        self.max_segs_per_req = max(b - a for a, b in zip(self.req_seg_off, self.req_seg_off[1:]))
        self.n_pairs = sum((b - a) * (b - a + 1) // 2 for a, b in zip(self.req_seg_off, self.req_seg_off[1:]))


def work(c):
    """Bytes and operations of one pass: every input read once, every output written once, products over the keys a
    row sees.  Rows that a pass reads through a list count with their number; their positions with their mean."""
    lay = _Layout(c)
    e = 4 if c["dtype"] == "f32" else 2
    hq, hkv, d = c["q_heads"], c["kv_heads"], c["head_dim"]
    kv_tok, q_tok = hkv * d * e, hq * d * e
    stored = sum(lay.store_len[i] for i in {dsc[0] for dsc in lay.descs})
    placed = sum(dsc[2] for dsc in lay.descs)
    missing = sum(lay.segments[s][3] for s in lay.missing)
    n = lay.n_rows
    nbytes = (stored + placed) * kv_tok                             # keys re-positioned
    flops = 0.0
    program = c["program"]
    if program in ("step", "score"):
        scored = pairs = 0
        for _, kind, start, m, *_ in lay.segments:
            if kind == 0 and start > 0:
                scored += m
                pairs += m * start + m * (m + 1) // 2
        nbytes += scored * q_tok + lay.n_tok * 4 + n * 16           # queries; scores; four lists
        flops += 2.0 * d * hq * pairs
    if program == "layer":
        nbytes += lay.n_tok * 4 + n * 16
    if program != "score":                                          # attention of the rows, new keys and values
        seen = 0.0
        for _, kind, start, m, _, ns, *_ in lay.segments:
            seen += ns * (start + (m + 1) / 2)
        nbytes += 2 * n * q_tok + 4 * n * kv_tok + n * hq * 4
        nbytes += stored * kv_tok + (placed * kv_tok if c["unrotated"] else 0)   # stored values, copied into the pages or read in place
        nbytes += 4 * missing * kv_tok
        flops += 4.0 * d * hq * seen
    if program == "build":
        nbytes += lay.n_pairs * 4 + len(lay.segments) * 8
    if program == "decoder":
        h, f = c["hidden"], c["ffn"]
        params = h * (hq + 2 * hkv) * d + hq * d * h + 3 * h * f
        # (q, new keys and values and the attention output stay inside the pass; the output is still returned)
        nbytes += params * e + 2 * n * h * e - n * q_tok - 2 * n * kv_tok
        flops += 2.0 * n * params
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(c):
    # fp32: sums in another order; bf16: results rounded to 8 bits.  Lists: near-ties of the scores.
    if c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 4e-4, "differ": 0.01}
    return {"rel": 1e-2, "max": 0.4, "differ": 0.01 if c["program"] in ("step", "score") else 0.0}


# ---- what a program holds before the call --------------------------------------------------------------
class _State:
    pass


def prepare(c, seed):
    lay = _Layout(c)
    s = _State()
    s.program, s.mass, s.unrotated = c["program"], c["mass"], c["unrotated"]
    hq, hkv, d = c["q_heads"], c["kv_heads"], c["head_dim"]
    f32 = c["dtype"] == "f32"
    dt = torch.float32 if f32 else torch.bfloat16
    scale = 1.0 if f32 else 1.0 / math.sqrt(128)
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    rnd = lambda *shape, sc=scale: torch.empty(shape, dtype=dt, device=DEVICE).normal_(0.0, sc, generator=gen)
    ints = lambda v: torch.tensor(np.ascontiguousarray(v, dtype=np.int32), device=DEVICE)
    empty_i = lambda n: torch.zeros(n, dtype=torch.int32, device=DEVICE)
    empty = lambda *shape: torch.zeros(shape, dtype=dt, device=DEVICE)
    shuffled = np.random.RandomState(c["layout"] % (1 << 31))

    s.ctx = P.Context(hq, hkv, d, 1.0e4 if f32 else 5.0e5, P.CC_F32 if f32 else P.CC_BF16)
    # chunk store and request pages; physical blocks in no order, as a serving cache leaves them
    pages = [-(-n // BLOCK) for n in lay.store_len]
    first_page = np.concatenate([[0], np.cumsum(pages)]).astype(np.int64)
    s.store_tab = ints(shuffled.permutation(int(first_page[-1])))
    s.req_tab_host = shuffled.permutation(lay.n_pages).astype(np.int32)
    s.req_tab = ints(s.req_tab_host)
    if s.program != "build":
        s.k_store, s.v_store = rnd(int(first_page[-1]), hkv, BLOCK, d), rnd(int(first_page[-1]), hkv, d, BLOCK)
    s.k_req, s.v_req = empty(lay.n_pages, hkv, BLOCK, d), empty(lay.n_pages, hkv, d, BLOCK)
    s.v_map = torch.full((lay.n_pages,), -1, dtype=torch.int32, device=DEVICE)
    s.descs = ints([(first_page[i], tab, n, pos if s.unrotated else pos - lay.cached_at[i]) for i, tab, n, pos in lay.descs] or
                   np.zeros((0, 4)))
    s.n_instances, s.max_shift = len(lay.descs), max([dsc[2] for dsc in lay.descs] or [0])
    s.segs, s.req_seg_off, s.cu_q = ints(lay.segments), ints(lay.req_seg_off), ints(lay.cu_q)
    s.n_requests, s.n_tok, s.n_rows = c["requests"], lay.n_tok, lay.n_rows
    s.max_seg_tokens = max(sg[3] for sg in lay.segments)
    s.max_rows, s.max_segs, s.n_pairs = lay.max_rows_per_req, lay.max_segs_per_req, lay.n_pairs
    s.max_question = max(sg[3] for sg in lay.segments if sg[1] == 1)
    # lists, scores, outputs
    s.sel_idx, s.q_row, s.q_pos, s.slot_map = (empty_i(s.n_rows) for _ in range(4))
    s.scores = torch.zeros(s.n_tok, dtype=torch.float32, device=DEVICE)
    n_segs = len(lay.segments)
    byte_buf = lambda n: torch.empty(max(256, n), dtype=torch.uint8, device=DEVICE)
    s.ws_select = byte_buf(s.ctx.select_workspace_bytes(s.n_tok, n_segs))
    if s.program != "score":
        s.out = empty(s.n_rows, hq, d)
        s.lse = torch.zeros((s.n_rows, hq), dtype=torch.float32, device=DEVICE)
        s.ws = byte_buf(s.ctx.sparse_prefill_workspace_bytes(s.n_tok, n_segs))
    if s.mass:
        s.seg_mass = torch.zeros(n_segs, dtype=torch.float32, device=DEVICE)
        s.ws = byte_buf(s.ctx.sparse_prefill_mass_workspace_bytes(s.n_tok, n_segs, s.n_requests, s.max_question, s.max_segs))
    # per-token tensors
    if s.program != "decoder":
        s.q = rnd(s.n_tok, hq, d)
        if s.program != "score":
            s.k_new, s.v_new = rnd(s.n_tok, hkv, d), rnd(s.n_tok, hkv, d)
    # a chunk's stored score list: tokens that looked most at other chunks when the cache was made
    stored_scores = torch.rand(s.n_tok, dtype=torch.float32, device=DEVICE, generator=gen)
    if s.program == "layer":
        s.scores = stored_scores
        rows, pos, slot = [], [], []
        for sg in lay.missing:
            _, _, start, n, tab, _, tok, _ = lay.segments[sg]
            t = np.arange(n)
            rows.append(tok + t)
            pos.append(start + t)
            slot.append(s.req_tab_host[tab + t // BLOCK].astype(np.int64) * BLOCK + t % BLOCK)
        s.n_miss = sum(len(t) for t in rows)
        if s.n_miss:
            s.miss_rows, s.miss_pos, s.miss_slot = (ints(np.concatenate(v)) for v in (rows, pos, slot))
            s.k_miss, s.v_miss = empty(s.n_miss, hkv, d), empty(s.n_miss, hkv, d)
    if s.program == "decoder":
        # (the rows are chosen once, before the first layer)
        s.ctx.select_from_scores(stored_scores, s.req_tab, s.segs, s.sel_idx, s.q_row, s.q_pos, s.slot_map, s.ws_select)
        h, f, n = c["hidden"], c["ffn"], s.n_rows
        s.hidden = rnd(s.n_tok, h, sc=1.0)
        s.gain_attn, s.gain_ffn = rnd(h, sc=0.1) + 1, rnd(h, sc=0.1) + 1
        s.w_qkv, s.w_o = rnd((hq + 2 * hkv) * d, h, sc=0.02), rnd(h, hq * d, sc=(hq * d) ** -0.5)
        s.w_gate, s.w_up, s.w_down = rnd(f, h, sc=h ** -0.5), rnd(f, h, sc=h ** -0.5), rnd(h, f, sc=f ** -0.5)
        s.h, s.h1, s.x, s.act = empty(n, h), empty(n, h), empty(n, h), empty(n, f)
        s.q_c, s.k_c, s.v_c = empty(n, hq, d), empty(n, hkv, d), empty(n, hkv, d)
        s.out_flat = s.out.view(n, hq * d)
    if s.program == "build":
        s.ctx.select_from_scores(stored_scores, s.req_tab, s.segs, s.sel_idx, s.q_row, s.q_pos, s.slot_map, s.ws_select)
        s.seg_mass, s.self_mass = (torch.zeros(n_segs, dtype=torch.float32, device=DEVICE) for _ in range(2))
        s.pair_mass = torch.zeros(s.n_pairs, dtype=torch.float32, device=DEVICE)
        s.ws = byte_buf(s.ctx.sparse_prefill_pairs_workspace_bytes(s.n_tok, n_segs, s.n_rows, s.max_rows, s.max_segs))
    return s


# ---- one pass ------------------------------------------------------------------------------------------
def _shift(s):
    if s.unrotated:
        s.ctx.rope_place(s.k_store, s.v_store, s.k_req, s.v_req, s.store_tab, s.req_tab, s.descs, s.n_instances, s.max_shift)
    else:                                              # values stay in the store until a token of their page is recomputed
        s.ctx.rope_shift(s.k_store, None, s.k_req, None, s.store_tab, s.req_tab, s.descs, s.n_instances, s.max_shift, v_map=s.v_map)


def _select(s):
    s.ctx.select(s.q, s.k_req, s.req_tab, s.segs, s.req_seg_off, s.n_requests, s.max_seg_tokens, s.sel_idx, s.q_row, s.q_pos,
                 s.slot_map, s.scores, s.ws_select)


def _prefill(s, q, k_new, v_new, src_rows):
    s.ctx.sparse_prefill(q, k_new, v_new, s.q_pos, s.slot_map, s.cu_q, s.max_rows, s.k_req, s.v_req, s.req_tab, s.segs,
                         s.req_seg_off, s.n_requests, s.n_tok, s.out, s.lse, s.ws, src_rows=src_rows,
                         shared=None if s.unrotated else (s.v_store, s.v_map))


def run(s):
    ctx, program = s.ctx, s.program
    if program == "build":
        ctx.sparse_prefill_pairs(s.q, s.k_new, s.v_new, s.q_pos, s.slot_map, s.cu_q, s.max_rows, s.k_req, s.v_req, s.req_tab,
                                 s.segs, s.req_seg_off, s.n_requests, s.max_segs, s.n_tok, s.out, s.lse, s.seg_mass,
                                 s.pair_mass, s.self_mass, s.ws)
        return [s.out, s.lse, s.pair_mass, s.self_mass, s.seg_mass, s.k_req, s.v_req]
    if program == "decoder":
        ctx.gather_rows(s.hidden, s.q_row, s.h)
        _shift(s)
        ctx.rms_norm(s.h, s.gain_attn, 1e-5, s.x)
        ctx.qkv_project(s.x, s.w_qkv, s.q_c, s.k_c, s.v_c)
        _prefill(s, s.q_c, s.k_c, s.v_c, None)
        ctx.linear(s.out_flat, s.w_o, s.h1, residual=s.h)
        ctx.rms_norm(s.h1, s.gain_ffn, 1e-5, s.x)
        ctx.gated_linear(s.x, s.w_gate, s.w_up, s.act)
        ctx.linear(s.act, s.w_down, s.h, residual=s.h1)
        return [s.h, s.out, s.lse, s.k_req, s.v_req, s.v_map]
    _shift(s)
    lists = [s.sel_idx, s.q_row, s.q_pos, s.slot_map]
    if program == "layer":
        if s.n_miss:
            ctx.gather_rows(s.k_new, s.miss_rows, s.k_miss)
            ctx.gather_rows(s.v_new, s.miss_rows, s.v_miss)
            ctx.scatter_kv(s.k_miss, s.v_miss, s.miss_pos, s.miss_slot, s.k_req, s.v_req)
        ctx.select_from_scores(s.scores, s.req_tab, s.segs, s.sel_idx, s.q_row, s.q_pos, s.slot_map, s.ws_select)
        if s.mass:
            ctx.sparse_prefill_mass(s.q, s.k_new, s.v_new, s.q_pos, s.slot_map, s.cu_q, s.max_rows, s.max_question, s.k_req,
                                    s.v_req, s.req_tab, s.segs, s.req_seg_off, s.n_requests, s.max_segs, s.n_tok, s.out, s.lse,
                                    s.seg_mass, s.ws, src_rows=s.q_row, shared=(s.v_store, s.v_map))
            return lists + [s.out, s.lse, s.seg_mass, s.k_req, s.v_req, s.v_map]
        _prefill(s, s.q, s.k_new, s.v_new, s.q_row)
        return lists + [s.out, s.lse, s.k_req, s.v_req, s.v_map]
    _select(s)
    if program == "score":
        return lists + [s.scores, s.k_req, s.v_map]
    _prefill(s, s.q, s.k_new, s.v_new, s.q_row)
    return lists + [s.scores, s.out, s.lse, s.k_req, s.v_req, s.v_map]
