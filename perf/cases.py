"""The workloads whose speed is measured, each one pass through the public entry points.

A case is a dict of plain values.  Its "kind" names the call a serving engine makes:

  h2o      H2ODecoder.step: one layer's H2O decode step (append, attention, score update,
           eviction) in the steady state, every unit at its budget ("ragged": some below it)
  quest    QuestDecoder.step: one layer's Quest decode step (page bounds, top-k pages, append,
           attention over the selection)
  omnikv   OmniKVDecoder.layer: an observation layer (attention over the whole history, slot
           selection) and the sparse layers that reuse its selection, in order
  snapkv   se_snapkv_compact with SE_SNAPKV_SCORE_ONLY: the observation window's pooled scores
           of whole prompts, as a pruning policy asks for them (and as compaction starts)
  prefill  se_h2o_prefill_chunk with a budget that keeps everything: the scores of a prefill
           chunk's queries over the retained slots and the chunk
  prune    se_prune_interval: idle chains give up part of a history interval; the layers of a
           model are stacked in one call

Decode cases carry on from pass to pass like a generation does: every pass is the next step,
with the next position and other inputs.  The caches that grow by a token a step start over
from their prompt after STEPS passes.  Scores, positions and keys follow the synthetic
workloads of this repository: N(0, 1) in bf16, queries shifted by one unit vector per KV head,
a hundredth of the positions heavy hitters with keys shifted by four times that vector.
"""

import math

import numpy as np
import torch

import paper_2609_39068_amd as se

PAGE = 16
STEPS = 128       # decode steps before a growing cache starts over from its prompt
RING = 4          # different step inputs, taken in turn
POSITIONS = 4096  # rows of the table of step positions


def listed():
    return [
        # the smallest call: two short requests of a small model (head_dim 64), all latency
        dict(name="h2o-tiny", kind="h2o", req=2, hkv=2, g=4, d=64, budget=128, recent=64, ragged=False),
        # one user's generation on an 8B-shaped layer: eight units in all
        dict(name="h2o-one-request", kind="h2o", req=1, hkv=8, g=4, d=128, budget=2048, recent=256, ragged=False),
        # continuous batching: retained lengths of every size up to the budget
        dict(name="h2o-ragged", kind="h2o", req=128, hkv=8, g=4, d=128, budget=4096, recent=512, ragged=True),
        # the throughput setting: one layer of the 32-layer, 256-request decode
        dict(name="h2o-batch", kind="h2o", req=256, hkv=8, g=4, d=128, budget=4096, recent=512, ragged=False),
        # page selection over 32K contexts at the usual batch
        dict(name="quest-layer", kind="quest", req=32, hkv=8, g=4, d=128, ctx=32768, top_k=64),
        # two 128K contexts, eight query heads per KV head, 1472 selected tokens
        dict(name="quest-long", kind="quest", req=2, hkv=4, g=8, d=128, ctx=131072, top_k=92),
        # an observation layer and the four sparse layers that follow it, 32K histories
        dict(name="omnikv-layers", kind="omnikv", req=32, hkv=8, g=4, d=128, ctx=32768, budget=2048, layers=5),
        # the same for a single 128K history of an odd length
        dict(name="omnikv-long", kind="omnikv", req=1, hkv=8, g=4, d=128, ctx=130001, budget=2048, layers=5),
        # one prompt has finished its prefill
        dict(name="snapkv-one-prompt", kind="snapkv", req=1, hkv=8, g=4, d=128, ctx=32768, window=32, kernel=7),
        # a batch of prompts has
        dict(name="snapkv-batch", kind="snapkv", req=64, hkv=8, g=4, d=128, ctx=32768, window=32, kernel=7),
        # the fourth 8192-token chunk of eight prompts, 2048 slots retained before it
        dict(name="prefill-chunk", kind="prefill", req=8, hkv=8, g=4, d=128, ctx=10240, chunk=8192, window=128),
        # one agent chain drops 80 % of a 4096-token tool result in all 32 layers
        dict(name="prune-chain", kind="prune", req=1, layers=32, hkv=8, d=128, ctx=32768, lo=16384, hi=20480, keep=819,
             mask=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd(rng, n):
    """Mostly an ordinary multiple of 16, otherwise any size nearby."""
    return max(16, n // 16 * 16) if rng.random() < 0.5 else max(16, n + rng.randint(-7, 7))


def draw(rng):
    kind = rng.choice(["h2o", "h2o", "quest", "omnikv", "snapkv", "prefill", "prune"])
    d = rng.choice([64, 128, 128, 128])
    hkv = rng.choice([2, 4, 8, 8])
    g = rng.choice([1, 2, 4, 4, 8])
    if kind == "h2o":
        budget = _odd(rng, _log(rng, 128, 4096))
        return dict(kind=kind, req=_log(rng, 1, 256), hkv=hkv, g=min(g, 4) if budget > 2048 else g, d=d,
                    budget=min(budget, 4096), recent=max(16, budget // rng.choice([2, 4, 8])), ragged=rng.random() < 0.3)
    if kind == "quest":
        ctx = _odd(rng, _log(rng, 2048, 131072))
        return dict(kind=kind, req=_log(rng, 1, max(1, min(64, (1 << 20) // ctx))), hkv=hkv, g=g, d=d, ctx=ctx,
                    top_k=_log(rng, 16, 128))
    if kind == "omnikv":
        ctx = _odd(rng, _log(rng, 4096, 131072))
        return dict(kind=kind, req=_log(rng, 1, max(1, min(32, (1 << 20) // ctx))), hkv=hkv, g=min(g, 4), d=d, ctx=ctx,
                    budget=min(_odd(rng, _log(rng, 512, 4096)), ctx // 2), layers=rng.choice([2, 3, 5, 5]))
    if kind == "snapkv":
        window = rng.choice([16, 32, 32, 33, 64])
        ctx = _odd(rng, _log(rng, 2048, 65536))
        rows = -(-window * g // 128) * 128
        most = max(1, min(64, (1 << 21) * 128 // (rows * ctx)))
        return dict(kind=kind, req=_log(rng, 1, most), hkv=hkv, g=g, d=d, ctx=ctx, window=window, kernel=rng.choice([3, 5, 7, 7, 13]))
    if kind == "prefill":
        chunk = _odd(rng, _log(rng, 512, 8192))
        return dict(kind=kind, req=_log(rng, 1, 8), hkv=hkv, g=g, d=d, ctx=chunk + _log(rng, 64, 2048), chunk=chunk,
                    window=rng.choice([32, 64, 128, 128]) if g <= 4 else rng.choice([32, 64]))
    ctx = _odd(rng, _log(rng, 4096, 65536))
    layers = _log(rng, 1, max(1, min(32, (1 << 20) // ctx)))
    n = _log(rng, 256, ctx // 4)
    lo = rng.randint(0, ctx - n)
    return dict(kind="prune", req=1, layers=layers, hkv=hkv, d=d, ctx=ctx, lo=lo, hi=lo + n, keep=int(n * rng.choice([0.1, 0.2, 0.5])),
                mask=rng.random() < 0.4)


# ---------------------------------------------------------------- inputs

def _gen(seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


class Cache:
    """One layer's paged cache of `units` units, their pages scattered over the pools."""

    def __init__(self, units, hkv, d, slots, lengths, positions, uvec, gen, dev, scores=False, meta=False, heavy=0.01):
        self.units, self.hkv, self.d = units, hkv, d
        self.max_pages = -(-slots // PAGE)
        n = units * self.max_pages
        self.table = torch.randperm(n, generator=gen, device=dev).to(torch.int32).view(units, self.max_pages)
        self.kv = torch.empty((n, 2, PAGE, d), dtype=torch.bfloat16, device=dev)
        step = max(1, (1 << 28) // (2 * PAGE * d))
        for i in range(0, n, step):
            self.kv[i:i + step].normal_(generator=gen)
        owner = torch.empty(n, dtype=torch.int64, device=dev)
        owner[self.table.view(-1).long()] = torch.arange(units, device=dev).repeat_interleave(self.max_pages)
        if heavy > 0:
            page, row = (torch.rand((n, PAGE), generator=gen, device=dev) < heavy).nonzero(as_tuple=True)
            self.kv[page, 0, row] = (self.kv[page, 0, row].float() + 4.0 * uvec[owner[page] % hkv]).to(torch.bfloat16)
        self.pos = torch.full((n, PAGE), -1, dtype=torch.int32, device=dev)
        at = self.table.long()
        cap = self.max_pages * PAGE
        p = torch.full((units, cap), -1, dtype=torch.int32, device=dev)
        p[:, :positions.shape[1]] = positions.to(torch.int32)
        p[torch.arange(cap, device=dev)[None, :] >= lengths[:, None]] = -1
        self.pos[at.view(-1)] = p.view(-1, PAGE)
        self.score = None
        if scores:
            self.score = -0.15 * torch.log1p(-torch.rand((n, PAGE), generator=gen, device=dev))
        self.meta = torch.zeros((n, 2, d), dtype=torch.bfloat16, device=dev) if meta else None
        self.lengths = lengths.to(torch.int32)
        self.first_lengths = self.lengths.clone()
        self.view = se.KVView(self.kv, self.pos, self.score, self.meta, self.table, self.lengths, num_kv_heads=hkv)
        self.bits = self.kv.view(torch.int16)  # keys and values are only ever copied: compared bit for bit

    def state(self):
        out = {"kv": self.bits, "pos": self.pos, "lengths": self.lengths}
        if self.score is not None:
            out["score"] = self.score
        return out


def _retained(units, budget, recent, ctx, gen, dev):
    """Positions of `budget` retained slots: the last `recent` ones and one of each stratum of the older."""
    old = budget - recent
    i = torch.arange(old, device=dev, dtype=torch.float64)
    width = (ctx - recent) / max(1, old)
    r = torch.rand((units, old), generator=gen, device=dev, dtype=torch.float64)
    older = torch.floor(i * width) + torch.floor(r * max(1.0, math.floor(width)))
    last = torch.arange(ctx - recent, ctx, device=dev, dtype=torch.float64).expand(units, recent)
    return torch.cat([older, last], dim=1).to(torch.int64)


def _unit_vectors(hkv, d, gen, dev):
    u = torch.randn((hkv, d), generator=gen, device=dev)
    return u / u.norm(dim=-1, keepdim=True)


def _queries(shape, hkv, g, uvec, gen, dev):
    return (torch.randn((*shape, hkv * g, uvec.shape[1]), generator=gen, device=dev) + uvec.repeat_interleave(g, dim=0)).to(torch.bfloat16)


def _scale(d):
    return float(np.float32(1.0 / np.sqrt(d)))


class _Steps:
    """The inputs of a generation's steps: RING different ones in turn, the positions going on."""

    def __init__(self, layers, req, hkv, g, ctx, uvec, gen, dev):
        d = uvec.shape[1]
        self.q = [[_queries((req,), hkv, g, uvec, gen, dev) for _ in range(layers)] for _ in range(RING)]
        kv = torch.randn((RING, layers, 2, req, hkv, d), generator=gen, device=dev).to(torch.bfloat16)
        self.k = [[kv[t, l, 0] for l in range(layers)] for t in range(RING)]
        self.v = [[kv[t, l, 1] for l in range(layers)] for t in range(RING)]
        self.table = (ctx + torch.arange(POSITIONS, device=dev, dtype=torch.int32)[:, None]).expand(POSITIONS, req).contiguous()
        self.pos = list(self.table.unbind(0))
        self.t = 0

    def next(self):
        """The step's number, its inputs for every layer, its positions."""
        t = self.t
        if t and t % POSITIONS == 0:
            self.table.add_(POSITIONS)
        self.t = t + 1
        r = t % RING
        return t, self.q[r], self.k[r], self.v[r], self.pos[t % POSITIONS]


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = _gen(seed, dev)
    hkv, d, kind = case["hkv"], case["d"], case["kind"]
    req = case["req"]
    units = req * hkv * case.get("layers", 1) if kind == "prune" else req * hkv
    uvec = _unit_vectors(hkv, d, gen, dev)
    s = {"case": case}

    if kind == "h2o":
        g, budget, recent = case["g"], case["budget"], case["recent"]
        ctx = 8 * budget + 1024
        pos = _retained(units, budget, recent, ctx, gen, dev)
        lengths = torch.full((units,), budget, dtype=torch.int64, device=dev)
        if case["ragged"]:  # any length from a quarter of the budget; those that would reach it within STEPS are full
            lengths = torch.randint(max(1, budget // 4), budget + 1, (units,), generator=gen, device=dev)
            lengths[lengths > budget - STEPS] = budget
            # a shorter unit holds the last of the sampled positions, the newest run among them
            i = torch.arange(budget, device=dev)[None, :] + (budget - lengths)[:, None]
            pos = pos.gather(1, i.clamp(max=budget - 1))
        s["cache"] = c = Cache(units, hkv, d, budget + 1, lengths, pos, uvec, gen, dev, scores=True)
        s["steps"] = _Steps(1, req, hkv, g, ctx, uvec, gen, dev)
        s["dec"] = se.H2ODecoder(c.view, g, _scale(d), budget, recent, budget + 1, dev)
        s["out"] = torch.empty((req, hkv * g, d), dtype=torch.float32, device=dev)
        s["lse"] = torch.empty((req, hkv * g), dtype=torch.float32, device=dev)
        return s

    ctx = case["ctx"]
    whole = torch.arange(ctx, device=dev)[None, :].expand(units, ctx)
    lengths = torch.full((units,), ctx, dtype=torch.int64, device=dev)
    if kind == "quest":
        g = case["g"]
        s["cache"] = c = Cache(units, hkv, d, ctx + STEPS, lengths, whole, uvec, gen, dev, meta=True)
        s["steps"] = _Steps(1, req, hkv, g, ctx, uvec, gen, dev)
        s["dec"] = se.QuestDecoder(c.view, g, _scale(d), case["top_k"], ctx + STEPS, dev)
        s["dec"].summarize()
        s["out"] = torch.empty((req, hkv * g, d), dtype=torch.float32, device=dev)
        s["lse"] = torch.empty((req, hkv * g), dtype=torch.float32, device=dev)
    elif kind == "omnikv":
        g, n = case["g"], case["layers"]
        s["caches"] = cs = [Cache(units, hkv, d, ctx + STEPS, lengths, whole, uvec, gen, dev) for _ in range(n)]
        s["steps"] = _Steps(n, req, hkv, g, ctx, uvec, gen, dev)
        s["dec"] = se.OmniKVDecoder(g, _scale(d), case["budget"], (0,), units, hkv, ctx + STEPS, cs[0].max_pages, d, dev)
        s["out"] = [torch.empty((req, hkv * g, d), dtype=torch.float32, device=dev) for _ in range(n)]
        s["lse"] = [torch.empty((req, hkv * g), dtype=torch.float32, device=dev) for _ in range(n)]
    elif kind in ("snapkv", "prefill"):
        g = case["g"]
        s["cache"] = c = Cache(units, hkv, d, ctx, lengths, whole, uvec, gen, dev, scores=True)
        s["q"] = _queries((req, case["window"]), hkv, g, uvec, gen, dev)
        op = se.SE_OP_SNAPKV if kind == "snapkv" else se.SE_OP_H2O_PREFILL
        n = se.se_workspace_bytes(op, units, ctx, c.max_pages, g, d, case["window"])
        s["ws"] = torch.empty(max(1, n), dtype=torch.uint8, device=dev)
        s["err"] = torch.zeros(1, dtype=torch.int32, device=dev)
    else:
        s["cache"] = c = Cache(units, hkv, d, ctx, lengths, whole, uvec, gen, dev, scores=True, heavy=0.0)
        s["first"] = (c.pos.clone(), c.score.clone())
        s["interval"] = torch.tensor([[case["lo"], case["hi"]]], dtype=torch.int32, device=dev).repeat(units, 1)
        s["mask"] = s["keep"] = None
        if case["mask"]:
            n = case["hi"] - case["lo"]
            s["mask"] = (torch.rand((units, n), generator=gen, device=dev) < case["keep"] / n).to(torch.uint8)
        else:
            s["keep"] = torch.full((units,), case["keep"], dtype=torch.int32, device=dev)
        s["freed"] = torch.zeros((units, c.max_pages), dtype=torch.int32, device=dev)
        s["count"] = torch.zeros(units, dtype=torch.int32, device=dev)
        s["err"] = torch.zeros(1, dtype=torch.int32, device=dev)
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "h2o":
        t, q, k, v, pos = s["steps"].next()
        c = s["cache"]
        if case["ragged"] and t and t % STEPS == 0:
            c.lengths.copy_(c.first_lengths)
        s["dec"].step(q[0], k[0], v[0], pos, s["out"], s["lse"])
        return {"out": s["out"], "lse": s["lse"], **c.state()}
    if kind == "quest":
        t, q, k, v, pos = s["steps"].next()
        c = s["cache"]
        if t and t % STEPS == 0:
            c.lengths.copy_(c.first_lengths)
        s["dec"].step(q[0], k[0], v[0], pos, s["out"], s["lse"], max_len=case["ctx"] + t % STEPS + 1)
        return {"out": s["out"], "lse": s["lse"], "sel": s["dec"].sel, **c.state()}
    if kind == "omnikv":
        t, q, k, v, pos = s["steps"].next()
        if t and t % STEPS == 0:
            for c in s["caches"]:
                c.lengths.copy_(c.first_lengths)
        bound = case["ctx"] + t % STEPS + 1
        for l, c in enumerate(s["caches"]):
            s["dec"].layer(l, c.view, q[l], k[l], v[l], pos, s["out"][l], s["lse"][l], max_len=bound)
        return {"out": s["out"], "lse": s["lse"], "sel": s["dec"].sel, "state": [c.state() for c in s["caches"]]}
    c = s["cache"]
    if kind == "snapkv":
        se.se_snapkv_compact(c.view, case["g"], s["q"], case["window"], case["kernel"], _scale(case["d"]), 2 * case["window"],
                             case["ctx"], se.SE_SNAPKV_SCORE_ONLY, None, 0, None, s["ws"], s["err"])
        return {"score": c.score}
    if kind == "prefill":
        se.se_h2o_prefill_chunk(c.view, case["g"], s["q"], case["window"], case["chunk"], _scale(case["d"]), case["ctx"], 0,
                                case["ctx"], None, 0, None, s["ws"], s["err"])
        return {"score": c.score, "lengths": c.lengths}
    # the next chain: its whole history is resident, with its own positions and scores
    c.lengths.copy_(c.first_lengths)
    c.pos.copy_(s["first"][0])
    c.score.copy_(s["first"][1])
    se.se_prune_interval(c.view, s["interval"], s["mask"], 0 if s["mask"] is None else s["mask"].shape[1], s["keep"], case["ctx"],
                         s["freed"], c.max_pages, s["count"], s["err"])
    return {**c.state(), "freed": s["freed"], "count": s["count"]}


# ---------------------------------------------------------------- what a pass cannot do without

def _mean_length(case):
    if not case.get("ragged"):
        return case["budget"]
    b = case["budget"]
    lo = max(1, b // 4)
    n = b + 1 - lo
    full = min(n, STEPS)  # lengths above budget - STEPS count as the budget
    return (full * b + (n - full) * (lo + b - full) / 2.0) / n


def work(case):
    kind, hkv, d, req = case["kind"], case["hkv"], case["d"], case["req"]
    units = req * hkv
    row = 4 * d  # a slot's key and value in bf16
    if kind == "prune":
        units *= case["layers"]
        moved = case["ctx"] - case["hi"] + case["keep"]
        kept = units * moved
        # positions, the interval's scores or mask; moved rows read and written with position and score; and the
        # histories' positions and scores put back first
        return {"bytes": units * (4 * case["ctx"] + (1 if case["mask"] else 4) * (case["hi"] - case["lo"])) + kept * 2 * (row + 8)
                + units * case["ctx"] * 16, "flops": 0}
    g = case["g"]
    io = units * (g * d * 2 + g * d * 4 + g * 4 + 2 * row)  # query, output, lse, the new token's rows in and out
    if kind == "h2o":
        slots = units * (_mean_length(case) + 1)
        return {"bytes": slots * (row + 12) + io, "flops": slots * 4 * g * d}
    if kind == "quest":
        pages = case["ctx"] // PAGE
        slots = (case["top_k"] + 1) * PAGE
        return {"bytes": units * (pages * row + slots * row + 4 * case["top_k"]) + io, "flops": units * (pages * 4 * g * d + slots * 4 * g * d)}
    if kind == "omnikv":
        n = case["ctx"] + (case["layers"] - 1) * case["budget"]
        return {"bytes": units * n * row + case["layers"] * io + req * case["budget"] * 4 * case["layers"], "flops": units * n * 4 * g * d}
    w = case["window"]
    q = units * w * g * d * 2
    flops = units * case["ctx"] * w * g * 2 * d
    if kind == "snapkv":  # keys and positions in, scores out
        return {"bytes": units * case["ctx"] * (2 * d + 4 + 4) + q, "flops": flops}
    return {"bytes": units * (case["ctx"] * (2 * d + 4) + (case["ctx"] - case["chunk"]) * 4) + q, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "prune":  # moves and selections of given scores
        return "exact"
    if kind == "h2o":
        # sums in 32 bits, and weights held with 11 bits until they are added to the scores: 1.3e-5 off 64 bits where
        # the budget is smallest; a victim that changes with the rounding changes two slots of its unit
        return {"rel": 5e-5, "max": 5e-3, "differ": 4e-3}
    if kind == "quest":
        # 32-bit sums (2e-7) until a page bound ties with the last selected one's: a unit that reads another page there
        # is about 0.2 off by itself; one of 256 units made 1e-2 against 64 bits
        return {"rel": 2e-2, "max": 0.9, "differ": 1e-2}
    # 32-bit sums: up to 7e-7 off 64 bits; a slot selection changes only where a 32-bit logit ties
    return {"rel": 1e-5, "max": 1e-3, "differ": 4e-3}


# ---------------------------------------------------------------- the same in 64 bits

def _rows(c, unit, n):
    """One unit's first n keys and values in float64, from the pages of its table row."""
    pg = c.kv[c.table[unit, :-(-n // PAGE)].long()]
    return pg[:, 0].reshape(-1, c.d)[:n].double(), pg[:, 1].reshape(-1, c.d)[:n].double()


def _attend(q, k, v, scale):
    z = scale * (q @ k.T)
    lse = torch.logsumexp(z, dim=1)
    w = torch.exp(z - lse[:, None])
    return z, w, w @ v, lse


def exact(case, seed):
    s = prepare(case, seed)
    kind, hkv, d = case["kind"], case["hkv"], case["d"]
    if kind == "prune":
        return None  # whole values and copies of bits
    g, scale = case["g"], _scale(d)
    units = case["req"] * hkv
    dev = torch.device("cuda")
    if kind == "omnikv":
        c, steps, n = s["caches"], s["steps"], case["ctx"]
        _, qs, ks, vs, _ = steps.next()
        outs, lses, picked = [], [], []
        for l in range(case["layers"]):
            out = torch.empty((units, g, d), dtype=torch.float64, device=dev)
            lse = torch.empty((units, g), dtype=torch.float64, device=dev)
            best = None
            for u in range(units):
                r, h = divmod(u, hkv)
                k, v = _rows(c[l], u, n)
                k, v = torch.cat([k, ks[l][r, h][None].double()]), torch.cat([v, vs[l][r, h][None].double()])
                if l > 0:
                    k, v = k[picked[r]], v[picked[r]]
                z, _, out[u], lse[u] = _attend(qs[l][r, h * g:(h + 1) * g].double(), k, v, scale)
                if l == 0:
                    top = z.max(dim=0).values
                    best = top if h == 0 else torch.maximum(best, top)
                    if h == hkv - 1:
                        picked.append(torch.sort(best, descending=True, stable=True).indices[:case["budget"]].sort().values)
            outs.append(out.view(case["req"], hkv * g, d))
            lses.append(lse.view(case["req"], hkv * g))
        return {"out": outs, "lse": lses, "sel": None, "state": [{"kv": None, "pos": None, "lengths": None} for _ in c]}
    c = s["cache"]
    if kind in ("h2o", "quest"):
        _, q, k_new, v_new, pos_new = s["steps"].next()
        out = torch.empty((units, g, d), dtype=torch.float64, device=dev)
        lse = torch.empty((units, g), dtype=torch.float64, device=dev)
        score = c.score.double() if kind == "h2o" else None
        lens = c.lengths.tolist()
        for u in range(units):
            r, h = divmod(u, hkv)
            n = lens[u]
            qu = q[0][r, h * g:(h + 1) * g].double()
            k, v = _rows(c, u, n)
            k, v = torch.cat([k, k_new[0][r, h][None].double()]), torch.cat([v, v_new[0][r, h][None].double()])
            if kind == "quest":
                pages = n // PAGE
                kp = k[:pages * PAGE].view(pages, PAGE, d)
                lo, hi = kp.amin(dim=1), kp.amax(dim=1)
                bound = (qu.clamp(min=0) @ hi.T + qu.clamp(max=0) @ lo.T).amax(dim=0)
                sel = torch.sort(bound, descending=True, stable=True).indices[:case["top_k"]]
                keep = torch.zeros(pages + 1, dtype=torch.bool, device=dev)
                keep[sel] = True
                keep[n // PAGE] = True
                slots = keep.repeat_interleave(PAGE)[:n + 1]
                k, v = k[slots], v[slots]
            _, w, out[u], lse[u] = _attend(qu, k, v, scale)
            if kind == "h2o":
                at = torch.arange(n + 1, device=dev)
                page, rr = c.table[u].long()[at // PAGE], at % PAGE
                sc = score[page, rr]
                sc[n] = 0.0
                sc = sc + w.sum(dim=0)
                score[page, rr] = sc
                if n + 1 > case["budget"]:
                    p = c.pos[page, rr].long()
                    p[n] = pos_new[r].long()
                    recent = min(case["recent"], case["budget"])
                    cand = (p <= p.max() - recent).nonzero().view(-1)
                    victim = cand[sc[cand].argmin()]
                    score[page[victim], rr[victim]] = sc[n]
        got = {"out": out.view(case["req"], hkv * g, d), "lse": lse.view(case["req"], hkv * g), "kv": None, "pos": None, "lengths": None}
        if kind == "h2o":
            got["score"] = score
        else:
            got["sel"] = None
        return got
    # scores of a window of queries over every slot, summed over the group
    w, n = case["window"], case["ctx"]
    score = c.score.double()
    t = torch.arange(w, device=dev).repeat_interleave(g)
    seen = torch.arange(n, device=dev)[None, :] <= (n - w + t)[:, None]
    at = torch.arange(n, device=dev)
    for u in range(units):
        r, h = divmod(u, hkv)
        k, _ = _rows(c, u, n)
        z = scale * (s["q"][r, :, h * g:(h + 1) * g].reshape(w * g, d).double() @ k.T)
        x = torch.softmax(z.masked_fill(~seen, -math.inf), dim=1).sum(dim=0)
        page, rr = c.table[u].long()[at // PAGE], at % PAGE
        if kind == "snapkv":
            pooled = torch.nn.functional.max_pool1d(x[:n - w].view(1, 1, -1), case["kernel"], 1, case["kernel"] // 2).view(-1)
            x = torch.cat([pooled, torch.zeros(w, dtype=torch.float64, device=dev)])
            score[page, rr] = x
        else:
            old = score[page, rr]
            old[n - case["chunk"]:] = 0.0
            score[page, rr] = old + x
    return {"score": score, "lengths": None} if kind == "prefill" else {"score": score}
