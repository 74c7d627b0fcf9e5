"""The decode loop of CHESS as a serving program runs it, as measurable cases.

A pass is the attention path of one model step (or of one prefill) over `layers` layers, called through
``paper_2602_20732_amd.Chess`` the way a serving loop calls it:

  step      every layer: ``decode_step`` with ``refresh_tail`` (tail summaries, selection, sparse attention)
  reselect  every layer: ``summarize_recent`` for the pages generated since the last selection, then ``decode_step``
  reuse     every layer: ``reuse_step`` over the kept list (token appended in the same launch), then one
            ``monitor_step`` over the step's logits
  prefill   every layer: ``summarize`` of the whole prompt
  shared    one page set for all layers: ``anchor`` + ``select_shared``, then ``sparse_decode`` in every layer
  dense     every layer: ``dense_decode`` over the whole cache

With ``graph`` the program has captured the model step in a HIP graph once and replays it (lengths, tables, lists and
tokens live in device memory, so the graph stays valid from step to step); without it every call is made from Python.

Inputs: topic segments (geometric lengths, mean 256 tokens), a key = its segment's topic vector + 0.5 N(0, I), a value
N(0, I), a query = the sum of three topic vectors of its sequence + 0.5 N(0, I), logits 3 N(0, 1); pages lie in the pool
in random order.  Shapes are those of the benchmark configurations of this repository, or between them."""
import math
import random

import torch

import paper_2602_20732_amd as pk

HEAD_DIM = 128
SINK, WINDOW = 1, 4
RECENT_PAGES = 10          # pages generated between two reselections
LIST_ROOM = 16             # page-list entries beyond the selection's own, for the pages a kept list gains
VOCAB = 151936             # logits a row, as in the benchmark of the monitor


def _case(name, kind, batch, lo, hi, heads, **more):
    c = {"name": name, "kind": kind, "batch": batch, "ctx_lo": lo, "ctx_hi": hi, "n_q_heads": heads[0], "n_kv_heads": heads[1],
         "page_size": 16, "fan_c": 8, "fan_g": 8, "plan": "budget", "budget_bp": 100, "summaries": "fp32", "layers": 1,
         "graph": False, "vocab": VOCAB}
    c.update(more)
    return c


def listed():
    return [
        # one short conversation, one call: the smallest step, where launch and latency are everything
        _case("step_b1_4k", "step", 1, 4096, 4096, (8, 8), budget_bp=625),
        # one user at 32K, the whole layer stack replayed as a graph
        _case("step_b1_32k", "step", 1, 32768, 32768, (32, 8), layers=32, graph=True),
        # a serving batch of ragged mid-length contexts, part of the layer stack as a graph
        _case("step_b32_ragged", "step", 32, 16384, 32768, (32, 8), layers=8, graph=True),
        # few long contexts at the 1 % budget
        _case("step_b8_128k", "step", 8, 131072, 131072, (32, 8), layers=2),
        # the same at a 5 % budget with bf16 summary vectors
        _case("step_b8_128k_5pct", "step", 8, 131072, 131072, (32, 8), budget_bp=500, summaries="bf16", layers=2),
        # one very long context, pages of 32 tokens and seven query heads to a KV head
        _case("step_b1_256k_page32", "step", 1, 262144, 262144, (28, 4), page_size=32, layers=8, graph=True),
        # a reselection under the paper's ratios for a large batch of odd lengths
        _case("reselect_b96_ragged", "reselect", 96, 4001, 21001, (32, 8), plan="ratio", summaries="bf16", layers=2),
        # between reselections, one user: the launch-bound inner loop
        _case("reuse_b1_32k", "reuse", 1, 32761, 32761, (32, 8), layers=32, graph=True),
        # between reselections, a serving batch, with the monitor over its logits
        _case("reuse_b32_ragged", "reuse", 32, 16384, 32768, (32, 8), layers=8),
        # the end of a prefill: summaries of whole prompts of odd lengths
        _case("prefill_b8_ragged", "prefill", 8, 30011, 131063, (32, 8)),
        # the paper's own scope: one page set for the model, attention in each of its layers
        _case("shared_b4_32k", "shared", 4, 24576, 32768, (32, 8), layers=32),
        # full attention over ragged contexts (layers or requests that are not sparsified)
        _case("dense_b16_ragged", "dense", 16, 8200, 65536, (32, 8)),
    ]


def draw(rng):
    kind = rng.choice(("step", "step", "step", "reselect", "reuse", "reuse", "prefill", "shared", "dense"))
    heads, page = rng.choice((((8, 8), 16), ((32, 8), 16), ((32, 8), 16), ((32, 8), 32), ((28, 4), 32)))

    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    hi = spread(4096, 262144)
    most = 1 << 20                                              # tokens of a layer, over the batch
    batch = spread(1, max(1, min(96, most // hi)))
    lo = hi if rng.random() < 0.4 else spread(max(2048, hi // 4), hi)
    if kind == "shared":
        layers = rng.choice((8, 28, 32))
        batch = max(1, min(batch, (4 << 20) // (hi * layers)))
    else:
        cap = (1 << 19) if kind in ("prefill", "dense") else (2 << 20)   # (these read every token)
        batch = max(1, min(batch, cap // hi))
        layers = max(1, min(32, spread(1, 32), cap // (hi * batch)))
    return {"kind": kind, "batch": batch, "ctx_lo": lo, "ctx_hi": hi, "n_q_heads": heads[0], "n_kv_heads": heads[1], "page_size": page,
            "fan_c": 8, "fan_g": rng.choice((4, 8, 8, 8)), "plan": rng.choice(("budget", "budget", "ratio")), "budget_bp": spread(100, 500),
            "summaries": rng.choice(("fp32", "fp32", "bf16")), "layers": layers, "graph": rng.random() < 0.5,
            "vocab": spread(32000, VOCAB)}


# ---- sizes that follow from a case
def _lengths(case):
    """The sequences' lengths: between ctx_lo and ctx_hi, the longest and the shortest among them."""
    lo, hi, n, B = case["ctx_lo"], case["ctx_hi"], case["batch"], case["page_size"]
    r = random.Random(lo * 7 + hi * 3 + n)
    lens = [hi] + [lo + r.randrange(hi - lo + 1) for _ in range(n - 1)]
    if n > 1:
        lens[-1] = lo
    if case["kind"] == "reuse":                                 # the token joins a page that has been begun
        lens = [n - 1 if n % B == 0 else n for n in lens]
    return lens


def _keep_counts(case, pages):
    """(grids, chunks, pages) the cascade keeps and (grids, chunks, pages) it has to score in a sequence of `pages` pages."""
    fc, fg = case["fan_c"], case["fan_g"]
    nc = -(-pages // fc)
    ng = -(-nc // fg)
    cand = max(0, pages - SINK - WINDOW)
    if case["plan"] == "ratio":                                 # the paper's Aggressive setting: 0.5 / 0.2 / 0.1
        kg = min(ng, max(1, -(-ng * 5000 // 10000)))
        chunks = min(nc, kg * fg)
        kc = min(chunks, max(1, -(-chunks * 2000 // 10000)))
        scored = min(cand, kc * fc)
        kp = min(scored, max(1, -(-scored * 1000 // 10000)))
    else:
        k = max(1, -(-pages * case["budget_bp"] // 10000))
        kct = -(-10 * k // fc)
        kg = min(ng, -(-5 * kct // fg))
        chunks = min(nc, kg * fg)
        kc = min(chunks, kct)
        scored = min(cand, kc * fc)
        kp = min(scored, k)
    return (kg, kc, kp), (ng, chunks, scored)


def _max_pages(case):
    return -(-case["ctx_hi"] // case["page_size"]) + RECENT_PAGES


def _plan(case):
    if case["plan"] == "ratio":
        return pk.SelectPlan(plan=pk.PLAN_RATIO, sink_pages=SINK, window_pages=WINDOW, rho_g_bp=5000, rho_c_bp=2000, rho_p_bp=1000)
    return pk.SelectPlan(sink_pages=SINK, window_pages=WINDOW, budget_bp=case["budget_bp"])


# ---- inputs
def _pools(case, seed, dev):
    """Per layer K pool, V pool and queries; the block table and the lengths they share."""
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    B, H, d = case["page_size"], case["n_kv_heads"], HEAD_DIM
    G = case["n_q_heads"] // H
    lens = torch.tensor(_lengths(case), device=dev)
    # (a program's pools have a page in hand for every sequence whose next token may open one)
    held = -(-lens // B) + 1
    n_phys, batch, width = int(held.sum()), case["batch"], _max_pages(case)
    order = torch.randperm(n_phys, generator=g, device=dev)
    table = torch.full((batch, width), -1, dtype=torch.int32, device=dev)
    there = torch.arange(width, device=dev)[None, :] < held[:, None]
    table[there] = order.to(torch.int32)

    # the topic segment of every token, numbered through the batch, in the pool's page order
    tokens = width * B
    seg = torch.zeros((batch, tokens), dtype=torch.int32, device=dev)
    for b in range(batch):
        seg[b] = (torch.rand(tokens, generator=g, device=dev) < 1.0 / 256).cumsum(0)
    n_seg = int(seg.max()) + 1
    seg += torch.arange(batch, dtype=torch.int32, device=dev)[:, None] * n_seg
    of_page = torch.empty((n_phys, B), dtype=torch.int32, device=dev)
    of_page[order] = seg.view(batch, width, B)[there]
    used = torch.stack([seg[b, n - 1] - b * n_seg + 1 for b, n in enumerate(lens.tolist())])   # segments inside the length

    layers = []
    for _ in range(case["layers"]):
        topics = torch.randn((batch * n_seg, H, d), generator=g, device=dev)
        k = torch.empty((n_phys, H, B, d), dtype=torch.bfloat16, device=dev)
        v = torch.empty((n_phys, H, d, B), dtype=torch.bfloat16, device=dev).normal_(generator=g)
        at = max(1, (1 << 26) // (B * H * d))
        for p in range(0, n_phys, at):
            rows = topics[of_page[p:p + at].long()]                                     # [pages, B, H, d]
            rows += 0.5 * torch.randn(rows.shape, generator=g, device=dev)
            k[p:p + at] = rows.permute(0, 2, 1, 3)
        pick = (torch.rand((batch, case["n_q_heads"], 3), generator=g, device=dev) * used[:, None, None]).long()
        pick += torch.arange(batch, device=dev)[:, None, None] * n_seg
        head = (torch.arange(case["n_q_heads"], device=dev) // G)[None, :, None]
        q = topics[pick, head].sum(2) + 0.5 * torch.randn((batch, case["n_q_heads"], d), generator=g, device=dev)
        layers.append({"k": k, "v": v, "q": q.to(torch.bfloat16)})
    return layers, table, lens.to(torch.int32), g


def _list_room(case):
    """Entries of a page list: what the plan keeps of the longest sequence the configuration admits, and some."""
    pages = _max_pages(case)
    return min(SINK + WINDOW + _keep_counts(case, pages)[0][2] + LIST_ROOM, pages)


def _tokens(case, n_layers, g, dev):
    """The token a reuse step appends, per layer, and the step's logits."""
    batch, H = case["batch"], case["n_kv_heads"]
    rows = [[torch.randn((batch, H, HEAD_DIM), generator=g, device=dev).to(torch.bfloat16) for _ in range(2)] for _ in range(n_layers)]
    stride = -(-case["vocab"] // 8) * 8
    return rows, (3 * torch.randn((batch, stride), generator=g, device=dev)).to(torch.bfloat16)


def prepare(case, seed):
    dev = torch.device("cuda")
    kind, batch, H = case["kind"], case["batch"], case["n_kv_heads"]
    layers, table, lens, g = _pools(case, seed, dev)
    pages = _max_pages(case)
    lib = pk.Chess(pk.Config(case["n_q_heads"], H, case["page_size"], batch, pages, _list_room(case), case["fan_c"], case["fan_g"],
                             summary_dtype=pk.SUMMARY_BF16 if case["summaries"] == "bf16" else pk.SUMMARY_F32))
    s = {"case": dict(case), "lib": lib, "plan": _plan(case), "table": table, "lens": lens, "layers": layers,
         "ws": lib.new_workspace(dev)}
    if kind == "reuse":
        tokens, s["logits"] = _tokens(case, len(layers), g, dev)
    for i, y in enumerate(layers):
        y["out"] = torch.empty((batch, case["n_q_heads"], HEAD_DIM), dtype=torch.float32, device=dev)
        y["ids"] = torch.full((batch, H, lib.cfg.max_selected_pages), -1, dtype=torch.int32, device=dev)
        y["n"] = torch.zeros((batch, H), dtype=torch.int32, device=dev)
        if kind != "dense":
            y["summ"] = lib.new_summaries(dev)
        if kind not in ("dense", "prefill"):
            lib.summarize(y["k"], table, lens, y["summ"])
        if kind == "reuse":
            lib.select(y["q"], y["summ"], lens, s["plan"], y["ids"], y["n"], s["ws"])
            y["k_new"], y["v_new"] = tokens[i]
            del y["summ"]
    if kind == "shared":
        s["anchors"] = [torch.empty((batch, H, HEAD_DIM), dtype=torch.float32, device=dev) for _ in layers]
    if kind == "reuse":
        s["entropy"] = torch.zeros(batch, dtype=torch.float32, device=dev)
        s["history"] = torch.zeros((batch, case["page_size"]), dtype=torch.float32, device=dev)
        s["count"] = torch.zeros(batch, dtype=torch.int32, device=dev)
        s["fire"] = torch.zeros(batch, dtype=torch.int32, device=dev)
    if case["graph"]:
        s["graph"] = _captured(s)
    return s


def _captured(s):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        _calls(s)
    torch.cuda.current_stream().wait_stream(side)
    if s["case"]["kind"] == "reuse":
        s["history"].zero_()
        s["count"].zero_()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _calls(s)
    return graph


# ---- the pass
def _calls(s):
    lib, table, lens, ws, plan, kind = s["lib"], s["table"], s["lens"], s["ws"], s["plan"], s["case"]["kind"]
    if kind == "step" or kind == "reselect":
        for y in s["layers"]:
            if kind == "reselect":
                lib.summarize_recent(y["k"], table, lens, RECENT_PAGES, y["summ"])
            lib.decode_step(y["q"], y["k"], y["v"], table, lens, y["summ"], plan, y["ids"], y["n"], y["out"], ws, refresh_tail=True)
    elif kind == "reuse":
        for y in s["layers"]:
            lib.reuse_step(y["q"], y["k_new"], y["v_new"], y["k"], y["v"], table, lens, y["ids"], y["n"], y["out"], ws)
        lib.monitor_step(s["logits"], s["case"]["page_size"], 9.0, 0.05, s["entropy"], s["history"], s["count"], s["fire"], ws,
                         vocab=s["case"]["vocab"])
    elif kind == "prefill":
        for y in s["layers"]:
            lib.summarize(y["k"], table, lens, y["summ"])
    elif kind == "shared":
        summ = [y["summ"] for y in s["layers"]]
        ids, n = s["layers"][0]["ids"], s["layers"][0]["n"]
        lib.anchor(summ, lens, WINDOW, s["anchors"])
        lib.select_shared(s["anchors"], summ, lens, plan, ids, n, ws)
        for y in s["layers"]:
            lib.sparse_decode(y["q"], y["k"], y["v"], table, lens, ids, n, y["out"], ws)
    else:
        for y in s["layers"]:
            lib.dense_decode(y["q"], y["k"], y["v"], table, lens, y["out"], ws)


def run(s):
    if "graph" in s:
        s["graph"].replay()
    else:
        _calls(s)
    kind, layers = s["case"]["kind"], s["layers"]
    if kind == "prefill":
        return [s["lib"].summary_views(y["summ"]) for y in layers]
    if kind == "dense":
        return [y["out"] for y in layers]
    if kind == "shared":
        return {"out": [y["out"] for y in layers], "ids": layers[0]["ids"], "n": layers[0]["n"]}
    # (of the state a step updates, the first layer's: summaries, or the pools with the appended token)
    if kind == "reuse":
        got = {"k": layers[0]["k"], "v": layers[0]["v"], "entropy": s["entropy"], "history": s["history"], "count": s["count"], "fire": s["fire"]}
    else:
        got = {"summaries": s["lib"].summary_views(layers[0]["summ"])}
    for i, y in enumerate(layers[:16]):
        got["out %d" % i], got["ids %d" % i], got["n %d" % i] = y["out"], y["ids"], y["n"]
    return got


# ---- what a pass cannot do without
def work(case):
    kind, B, H, Hq, d = case["kind"], case["page_size"], case["n_kv_heads"], case["n_q_heads"], HEAD_DIM
    vec = d * (2 if case["summaries"] == "bf16" else 4)
    fc, fg, L = case["fan_c"], case["fan_g"], case["layers"]
    nbytes = flops = 0
    shared_bytes = shared_flops = 0                             # what is paid once and not in every layer
    for n in _lengths(case):
        pages = -(-n // B)
        chunks = -(-pages // fc)
        grids = -(-chunks // fg)
        (kg, kc, kp), scored = _keep_counts(case, pages)
        units = sum(scored)
        listed_pages = pages if pages <= SINK + WINDOW else SINK + kp + WINDOW
        if kind == "dense":
            tokens = n
        elif kind == "prefill":
            nbytes += H * (n * d * 2 + (pages + chunks + grids) * vec)
            flops += H * n * d
            continue
        else:
            tokens = listed_pages * B
        nbytes += H * tokens * d * 2 * 2 + Hq * d * (2 + 4)     # K and V rows, q, out
        flops += 4 * Hq * tokens * d
        if kind in ("step", "reselect"):
            renewed = 1 if kind == "step" else RECENT_PAGES
            nbytes += H * (units * vec + renewed * B * d * 2 + (renewed + 2) * vec + (fc + fg) * vec) + H * 4 * listed_pages
            flops += 2 * H * units * d + H * renewed * B * d
        elif kind == "shared":
            shared_bytes += L * H * (units + WINDOW) * vec + 2 * L * H * d * 4
            shared_flops += 2 * L * H * units * d
        elif kind == "reuse":
            nbytes += 2 * H * d * 2 * 2 + H * 4 * listed_pages  # the new token's rows in and out, the list
            shared_bytes += 2 * case["vocab"]
            shared_flops += 4 * case["vocab"]
    return {"bytes": L * nbytes + shared_bytes, "flops": L * flops + shared_flops}


def tolerance(case):
    # summaries, page lists and appended rows: sums that are exact in fp64, rounded once
    if case["kind"] == "prefill":
        return "exact"
    # attention: bf16 inputs, fp32 accumulation, weights to 2^-17 (against itself in 64 bits: rel 2.1e-6, largest
    # difference 1.9e-5 of the rms, in every case); entropy: fp32 over the vocabulary (rel 8e-8); page lists do not differ
    return {"rel": 1e-5, "max": 1e-4}


# ---- the same in 64 bits, with plain torch
def _stored(case, mean):
    """A mean as the summaries store it, as fp64."""
    m = mean.to(torch.float32)
    return (m.to(torch.bfloat16) if case["summaries"] == "bf16" else m).double()


def _means(x, fan):
    """Means over `fan` consecutive members of dim 1 (the last one over those that exist), fp64."""
    n = -(-x.shape[1] // fan)
    full = torch.nn.functional.pad(x, (0, 0, 0, n * fan - x.shape[1])).view(x.shape[0], n, fan, x.shape[2]).sum(2)
    count = torch.full((n,), fan, device=x.device)
    count[-1] = x.shape[1] - (n - 1) * fan
    return full / count[None, :, None]


def _sequence_means(case, k, table_row, n):
    """Page, chunk and grid means [H, units, d] of one sequence in one layer, each over its children as stored."""
    B, H = case["page_size"], case["n_kv_heads"]
    pages = -(-n // B)
    rows = k[table_row[:pages].long()].transpose(0, 1).reshape(H, pages * B, HEAD_DIM)[:, :n].double()
    page = _means(rows, B)
    chunk = _means(_stored(case, page), case["fan_c"])
    return page, chunk, _means(_stored(case, chunk), case["fan_g"])


def _top(score, active, k):
    """Boolean mask of the k (one per row) highest active scores of every row, ties to the lower index."""
    order = torch.where(active, score, -math.inf).sort(dim=1, descending=True, stable=True).indices
    rank = torch.empty_like(order).scatter_(1, order, torch.arange(score.shape[1], device=score.device).expand_as(order))
    return active & (rank < k[:, None])


def _select(case, grid_s, chunk_s, page_s):
    """The cascade over scores [rows, units]: ids [rows, list room] (-1 padded) and their number [rows]."""
    fc, fg, dev = case["fan_c"], case["fan_g"], page_s.device
    P, nc, ng = page_s.shape[1], chunk_s.shape[1], grid_s.shape[1]
    ratio = case["plan"] == "ratio"
    k = max(1, -(-P * case["budget_bp"] // 10000))
    kct = -(-10 * k // fc)

    def cut(score, active, rho, target):
        n = active.sum(1)
        return _top(score, active, torch.clamp(-(-n * rho // 10000), min=1) if ratio else torch.clamp(n, max=target))

    grids = cut(grid_s, torch.ones_like(grid_s, dtype=torch.bool), 5000, -(-5 * kct // fg))
    chunks = cut(chunk_s, grids.repeat_interleave(fg, 1)[:, :nc], 2000, kct)
    pages = chunks.repeat_interleave(fc, 1)[:, :P].clone()
    pages[:, :SINK] = pages[:, P - WINDOW:] = False
    pages = cut(page_s, pages, 1000, k)
    pages[:, :SINK] = pages[:, P - WINDOW:] = True
    n = pages.sum(1)
    ids = torch.full((pages.shape[0], _list_room(case)), -1, dtype=torch.int32, device=dev)
    at = torch.nonzero(pages)
    ids[at[:, 0], (pages.cumsum(1) - 1)[pages]] = at[:, 1].to(torch.int32)
    return ids, n.to(torch.int32)


def _attend(case, q, k, v, table_row, n, ids=None):
    """Attention [n_q_heads, d] of one sequence of n tokens over the listed pages (ids [H, pages], None: all)."""
    B, H = case["page_size"], case["n_kv_heads"]
    pages = -(-n // B)
    if ids is None:
        ids = torch.arange(pages, device=q.device)[None].expand(H, pages)
    ids = ids.long()
    head = torch.arange(H, device=q.device)[:, None]
    phys = table_row[ids.clamp(min=0)].long()
    token = (ids[:, :, None] * B + torch.arange(B, device=q.device)).view(H, 1, -1)
    there = (ids >= 0).repeat_interleave(B, 1)[:, None] & (token < n)
    keys = k[phys, head].double().view(H, -1, HEAD_DIM)
    values = v[phys, head].double().transpose(2, 3).reshape(H, -1, HEAD_DIM)
    score = torch.matmul(q.double().view(H, -1, HEAD_DIM), keys.transpose(1, 2).contiguous()) / math.sqrt(HEAD_DIM)
    p = torch.where(there, score, -math.inf).softmax(2)
    return torch.matmul(p, values).view(-1, HEAD_DIM)


def exact(case, seed):
    dev = torch.device("cuda")
    kind, batch, H, B = case["kind"], case["batch"], case["n_kv_heads"], case["page_size"]
    layers, table, _, g = _pools(case, seed, dev)
    lens = _lengths(case)
    if kind == "dense":
        return [torch.stack([_attend(case, y["q"][b], y["k"], y["v"], table[b], lens[b]) for b in range(batch)]) for y in layers]

    units = [_max_pages(case)]
    units += [-(-units[0] // case["fan_c"])]
    units += [-(-units[1] // case["fan_g"])]

    def summaries(per_seq):
        full = [torch.zeros((batch, H, u, HEAD_DIM), dtype=torch.float64, device=dev) for u in units]
        for b, means in enumerate(per_seq):
            for f, m in zip(full, means):
                f[b, :, :m.shape[1]] = m
        return tuple(full)

    def scores(means, probe):                                   # [H, units] of a level, from what is stored of it
        return torch.matmul(_stored(case, means), probe[:, :, None])[:, :, 0]

    if kind == "prefill":
        return [summaries([_sequence_means(case, y["k"], table[b], lens[b]) for b in range(batch)]) for y in layers]

    if kind == "shared":
        lists, counts = [], []
        for b in range(batch):
            total = None
            for y in layers:
                page, chunk, grid = _sequence_means(case, y["k"], table[b], lens[b])
                anchor = _stored(case, page)[:, -WINDOW:].mean(1).to(torch.float32).double()
                s = [scores(m, anchor).sum(0, keepdim=True) for m in (grid, chunk, page)]
                total = s if total is None else [t + x for t, x in zip(total, s)]
            ids, n = _select(case, *total)
            lists.append(ids.expand(H, -1))
            counts.append(n.expand(H))
        out = [torch.stack([_attend(case, y["q"][b], y["k"], y["v"], table[b], lens[b], lists[b]) for b in range(batch)]) for y in layers]
        return {"out": out, "ids": torch.stack(lists), "n": torch.stack(counts)}

    got = {}
    if kind == "reuse":
        tokens, logits = _tokens(case, len(layers), g, dev)
        logp = logits[:, :case["vocab"]].double().log_softmax(1)
        got.update({"k": None, "v": None, "history": None, "count": None, "fire": None, "entropy": -(logp.exp() * logp).sum(1)})
    for i, y in enumerate(layers[:16]):
        means = [_sequence_means(case, y["k"], table[b], lens[b]) for b in range(batch)]
        if i == 0 and kind != "reuse":
            got["summaries"] = summaries(means)
        outs, lists, counts = [], [], []
        for b in range(batch):
            probe = y["q"][b].double().view(H, -1, HEAD_DIM).sum(1)
            ids, n = _select(case, *[scores(m, probe) for m in means[b][::-1]])
            grown = lens[b]
            if kind == "reuse":
                phys, tok = int(table[b, grown // B]), grown % B
                y["k"][phys, :, tok], y["v"][phys, :, :, tok] = tokens[i][0][b], tokens[i][1][b]
                grown += 1
            outs.append(_attend(case, y["q"][b], y["k"], y["v"], table[b], grown, ids))
            lists.append(ids)
            counts.append(n)
        got["out %d" % i], got["ids %d" % i], got["n %d" % i] = torch.stack(outs), torch.stack(lists), torch.stack(counts)
    return got
