"""The work a user of this package has it do, as cases that can be timed and compared.

Two ways of use:

  step  `Finch.step` on the KV heads of one layer (of one or a few requests).  A model runs
        its layers one after the other, so a chunked prefill that compresses as it goes calls
        this once per layer and chunk: small batches, where launches and latency count.
        `calls` = "stages" makes the same step of `score`, `topk` and `compact`;
        "static" of `step_static`.
  loop  `ChunkLoop.run` on all layers and KV heads of one or several requests whose keys
        and values are there already: the whole chunk loop in one call, the batch the
        library is built for (the workloads of `workloads/configs.py` and `bench.py`).

Options in both: the prompt's own keys in the denominator (`exact`), one selection per layer
(`layerwise`), kept keys turned to their new positions (`rope`); loops also take rows of the
chunk's own tokens (`doc_rows`).

Values.  Q, K, V are N(0,1) per element; the prompt rows lean towards one direction, and so do
the relevant keys, as many in every chunk as the schedule adds to the cache there.  The
direction lies in the channel pairs that rotary embeddings turn slowest (where models carry
meaning rather than position), so relevant keys stay relevant when `rope` moves them.  As in
attention that has something to find, relevant keys stand clear of the others: two correct
implementations keep the same rows although their scores differ in the last bits.
"""
import math

import torch

import paper_2408_00167_amd as F
from paper_2408_00167_amd.driver import ChunkLoop

DEV = "cuda"
ROPE_BASE = 500000.0
LEAN = 2.5          # how far prompt rows lean towards the common direction
REACH = (1.6, 2.4)  # the same of relevant keys, in units of sqrt(head_dim)

_DEFAULTS = dict(dtype="bf16", head_dim=128, group=4, kv_heads=8, layers=1, requests=1, n_que=48, chunk=4096,
                 exact=False, layerwise=False, rope=False)


def _step(name, **kw):
    """One prefill step of one layer: `cache` kept rows and `chunk` new ones, `keep` stay."""
    return {"name": name, "kind": "step", **_DEFAULTS, "calls": "step", **kw}


def _loop(name, **kw):
    """The chunk loop over documents of `tokens` rows; with several requests their lengths
    go from `tokens_min` to `tokens` and their prompts from `n_que_min` to `n_que`."""
    return {"name": name, "kind": "loop", **_DEFAULTS, "layers": 32, "doc_rows": False, "ratio": 16, **kw,
            "tokens_min": kw.get("tokens_min", kw["tokens"]), "n_que_min": kw.get("n_que_min", kw.get("n_que", 48))}


def listed():
    return [
        # the smallest job: four fp32 heads, 1024 tokens in four chunks (tests, reference runs on small models)
        _loop("loop_f32_small", dtype="f32", head_dim=64, group=1, kv_heads=4, layers=1, tokens=1024, n_que=16, chunk=256),
        # one layer of a Llama-2-7B-shaped model (32 heads, no grouping), a 512-token chunk in mid-document
        _step("step_mha_layer", group=1, kv_heads=32, n_que=32, chunk=512, cache=512, keep=640),
        # one layer of a Llama-3-8B-shaped model, a 4096-token chunk halfway through 131072 tokens
        _step("step_gqa_layer", n_que=48, chunk=4096, cache=704, keep=748),
        # the same layer as the paper words the method: exact denominator, one selection per
        # layer, kept keys turned to their new positions; a 2048-token chunk
        _step("step_gqa_layer_paper", n_que=64, chunk=2048, cache=1000, keep=1128, exact=True, layerwise=True, rope=True),
        # narrow heads, a short last chunk with odd sizes, called without a workspace
        _step("step_narrow_odd", head_dim=64, group=2, kv_heads=12, n_que=19, chunk=777, cache=123, keep=211, calls="static"),
        # stage by stage for four requests of a Mistral-7B-shaped layer (a caller that wants the scores in between)
        _step("step_stages_batch", requests=4, n_que=64, chunk=2048, cache=896, keep=1024, calls="stages"),
        # the workloads of the benchmark: 1024 heads at 4096 tokens, 256 heads at 32768 and at 131072
        _loop("loop_mha_4k", group=1, kv_heads=32, tokens=4096, n_que=32, chunk=512, ratio=4),
        _loop("loop_gqa_32k", tokens=32768, n_que=64, chunk=2048, ratio=16),
        _loop("loop_gqa_128k", tokens=131072, n_que=48, chunk=4096, ratio=93),
        # a ragged serving batch: four requests of 2047 to 50001 tokens and 16 to 128 prompt rows
        _loop("loop_ragged", requests=4, tokens_min=2047, tokens=50001, n_que_min=16, n_que=128, chunk=2048, ratio=32),
        # a short document, all layers, as the paper words the method
        _loop("loop_gqa_8k_paper", tokens=8000, n_que=37, chunk=2048, ratio=8, exact=True, layerwise=True, rope=True),
        # the paper's ablation: conditioning on the chunk's own rows as well
        _loop("loop_doc_rows", tokens=4096, n_que=48, chunk=1024, ratio=8, doc_rows=True),
    ]


# ------------------------------------------------------------------------------ drawn cases

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [dict(head_dim=128, group=1, kv_heads=32), dict(head_dim=128, group=4, kv_heads=8),
          dict(head_dim=128, group=4, kv_heads=8), dict(head_dim=128, group=8, kv_heads=4),
          dict(head_dim=64, group=2, kv_heads=12), dict(head_dim=64, group=4, kv_heads=8)]


def draw(rng):
    what = rng.random()
    if what < 0.1:  # small fp32 jobs
        case = _loop("", dtype="f32", head_dim=64, group=rng.choice([1, 1, 2]), kv_heads=rng.choice([4, 8, 12]), layers=1,
                     tokens=_log(rng, 300, 2048), n_que=rng.randint(8, 24), chunk=_log(rng, 128, 512), ratio=rng.choice([4, 8, 16]))
    elif what < 0.6:
        heads = rng.choice(_HEADS)
        chunk, cache = _log(rng, 128, 8192), _log(rng, 1, 2048) - 1
        case = _step("", **heads, requests=rng.choice([1, 1, 1, 2, 4]) if heads["kv_heads"] < 32 else 1,
                     n_que=_log(rng, 8, 96), chunk=chunk, cache=cache, keep=cache + max(1, chunk // _log(rng, 2, 64)),
                     calls=rng.choice(["step", "step", "step", "static", "stages"]))
        if rng.random() < 0.3:
            case.update(exact=rng.random() < 0.7, layerwise=rng.random() < 0.7, rope=rng.random() < 0.7)
    else:
        heads = rng.choice(_HEADS)
        tokens = _log(rng, 1024, 131072)
        several = rng.random() < 0.3
        case = _loop("", **heads, layers=rng.choice([8, 16, 32, 32]), requests=rng.choice([2, 3, 4]) if several else 1,
                     tokens=tokens, n_que=_log(rng, 16, 96), chunk=min(tokens, _log(rng, 512, 4096)), ratio=_log(rng, 4, 96))
        case.update(tokens_min=max(512, tokens // rng.randint(1, 16)) if several else tokens,
                    n_que_min=_log(rng, 8, case["n_que"]) if several else case["n_que"])
        if rng.random() < 0.3:
            case.update(exact=rng.random() < 0.7, layerwise=rng.random() < 0.7, rope=rng.random() < 0.7)
        elif rng.random() < 0.1:
            case.update(doc_rows=True, chunk=min(case["chunk"], 1024), tokens=min(tokens, 4096),
                        tokens_min=min(case["tokens_min"], 4096))
        # no more work than the largest listed loop, and no more descriptors
        case["ratio"] = max(case["ratio"], -(-tokens // 8192))
        while _cost(case) > 1.0:
            if case["layers"] > 1:
                case["layers"] //= 2
            else:
                case["tokens"], case["tokens_min"] = case["tokens"] // 2, max(512, case["tokens_min"] // 2)
    del case["name"]
    return case


def _cost(case):
    """Against loop_gqa_128k: logits, bytes and descriptors, whichever is most."""
    w = work(case)
    steps = sum(-(-n // case["chunk"]) for n, _ in _requests(case)) * case["layers"] * case["kv_heads"]
    return max(w["flops"] / 1.9e12, w["bytes"] / 1.6e10, steps / 8192)


# ------------------------------------------------------------------------------------ inputs

def _requests(case):
    """(tokens, n_que) of each request of a loop, in equal ratios between the two ends."""
    n = case["requests"]
    out = []
    for i in range(n):
        x = i / (n - 1) if n > 1 else 1.0
        out.append((int(case["tokens_min"] * (case["tokens"] / case["tokens_min"]) ** x),
                    int(case["n_que_min"] * (case["n_que"] / case["n_que_min"]) ** (1.0 - x if i % 2 else x))))
    return out


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


class _Draw:
    """Tensors of one seed."""

    def __init__(self, case, seed):
        self.case, self.d, self.dt = case, case["head_dim"], _dtype(case)
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed))

    def normal(self, *shape, dtype=None):
        return torch.randn(*shape, generator=self.gen, device=DEV, dtype=dtype or self.dt)

    def direction(self, heads):
        """[heads][d] unit vectors in the slow channel pairs (u, u + d/2)."""
        a = torch.zeros(heads, self.d, device=DEV)
        lo, half = 3 * self.d // 8, self.d // 2
        a[:, lo:half] = self.normal(heads, half - lo, dtype=torch.float32)
        a[:, half + lo:] = self.normal(heads, half - lo, dtype=torch.float32)
        return a / a.norm(dim=1, keepdim=True)

    def rows(self, a, n):
        """[heads][n][d] query rows that lean towards `a`."""
        return (self.normal(a.shape[0], n, self.d, dtype=torch.float32) + LEAN * a[:, None]).to(self.dt)

    def plant(self, k, a, lo, hi, count, share):
        """Makes `count` keys of rows [lo, hi) of k [heads][n][d] relevant; runs of `share`
        heads (a layer's) have them at the same places."""
        if count <= 0:
            return
        heads = k.shape[0]
        at = torch.rand(heads // share, hi - lo, generator=self.gen, device=DEV).topk(count, dim=1).indices + lo
        at = at.repeat_interleave(share, dim=0)
        reach = torch.rand(heads, count, 1, generator=self.gen, device=DEV) * (REACH[1] - REACH[0]) + REACH[0]
        x = self.normal(heads, count, self.d, dtype=torch.float32) + reach * math.sqrt(self.d) * a[:, None]
        k.scatter_(1, at[:, :, None].expand(-1, -1, self.d), x.to(self.dt))


def _context(case):
    fin = F.Finch(F.FINCH_F32 if case["dtype"] == "f32" else F.FINCH_BF16, case["head_dim"], case["group"], device=DEV)
    if case["layerwise"]:
        F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_GROUP, case["kv_heads"])
    if case["rope"]:
        fin.set_reposition(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING, ROPE_BASE)
    return fin


def prepare(case, seed):
    fin, mk = _context(case), _Draw(case, seed)
    share = case["kv_heads"] if case["layerwise"] else 1
    if case["kind"] == "step":
        P, d, dt = case["requests"] * case["kv_heads"], case["head_dim"], _dtype(case)
        c, m, r, n_que, rows = case["cache"], case["chunk"], case["keep"], case["n_que"], case["group"] * case["n_que"]
        a = mk.direction(P)
        q, kc, vc, km, vm = mk.rows(a, rows), mk.normal(P, c, d), mk.normal(P, c, d), mk.normal(P, m, d), mk.normal(P, m, d)
        mk.plant(kc, a, 0, c, c, share)
        mk.plant(km, a, 0, m, r - c, share)
        kq = mk.normal(P, n_que, d) if case["exact"] else None
        extra = torch.zeros(P, rows, device=DEV) if case["exact"] else None
        ko, vo = torch.zeros(P, r, d, dtype=dt, device=DEV), torch.zeros(P, r, d, dtype=dt, device=DEV)
        scores, idx = torch.zeros(P, c + m, device=DEV), torch.zeros(P, r, dtype=torch.int32, device=DEV)
        batch = F.Batch([dict(q=q[p], k_cache=kc[p], v_cache=vc[p], k_chunk=km[p], v_chunk=vm[p], k_out=ko[p], v_out=vo[p],
                              scores=scores[p], idx=idx[p], n_que=n_que, c=c, m=m, r=r,
                              k_que=None if kq is None else kq[p], lse_extra=None if extra is None else extra[p])
                         for p in range(P)], device=DEV)
        if case["calls"] != "static":
            fin.reserve(batch)
        return dict(case=case, fin=fin, batch=batch, keep=(q, kc, vc, km, vm, kq, extra), out=(ko, vo, scores, idx))
    problems = []
    for tokens, n_que in _requests(case):
        heads, rows, chunk = case["layers"] * case["kv_heads"], case["group"] * n_que, case["chunk"]
        budget = max(1, tokens // case["ratio"])
        a = mk.direction(heads)
        q, k, v = mk.rows(a, rows), mk.normal(heads, tokens, case["head_dim"]), mk.normal(heads, tokens, case["head_dim"])
        kept = 0
        for i, r in enumerate(F.finch_schedule(tokens, chunk, budget)):
            lo, hi = i * chunk, min(tokens, (i + 1) * chunk)
            # (a chunk's last tokens are seen by few of the chunk's own rows)
            mk.plant(k, a, lo, lo + max(r - kept, (hi - lo) * 3 // 4) if case["doc_rows"] else hi, r - kept, share)
            kept = r
        kq = mk.normal(heads, n_que, case["head_dim"]) if case["exact"] else None
        qd = mk.rows(a, case["group"] * chunk).reshape(heads, case["group"], chunk, -1) if case["doc_rows"] else None
        for p in range(heads):
            problems.append(dict(Q=q[p], K=k[p], V=v[p], n_que=n_que, budget=budget))
            if kq is not None:
                problems[-1]["K_que"] = kq[p]
            if qd is not None:
                problems[-1]["Q_doc"] = qd[p]
    return dict(case=case, loop=ChunkLoop(fin, problems, case["chunk"]))


def run(state):
    if "loop" in state:
        loop = state["loop"]
        loop.run()
        # the caches of the last and the last but one step, and the last step's scores and indices
        return loop.kbuf[0], loop.kbuf[1], loop.vbuf[0], loop.vbuf[1], loop.scores, loop.idx
    fin, batch, case = state["fin"], state["batch"], state["case"]
    if case["exact"]:
        fin.prompt_lse(batch)
    if case["calls"] == "stages":
        fin.score(batch)
        fin.topk(batch)
        fin.compact(batch)
    elif case["calls"] == "static":
        fin.step_static(batch)
    else:
        fin.step(batch)
    return state["out"]


# ----------------------------------------------------------------- what a pass cannot do without

def _step_work(case, c, m, r, n_que, doc):
    e, d, n, rows = (4 if case["dtype"] == "f32" else 2), case["head_dim"], c + m, case["group"] * n_que
    # candidate keys and query rows read, kept K and V rows read and written, scores and indices written
    b = n * d * e + rows * d * e + 4 * min(r, n) * d * e + 4 * n + 4 * min(r, n)
    f = 2.0 * n * rows * d  # every logit once
    if case["exact"]:
        b += n_que * d * e
        f += 2.0 * rows * (n_que + 1) / 2 * d
    if doc:
        b += case["group"] * m * d * e
        f += 2.0 * case["group"] * (m * c + m * (m + 1) / 2) * d
    return b, f


def work(case):
    b = f = 0.0
    if case["kind"] == "step":
        P = case["requests"] * case["kv_heads"]
        x, y = _step_work(case, case["cache"], case["chunk"], case["keep"], case["n_que"], False)
        return {"bytes": P * x, "flops": P * y}
    heads = case["layers"] * case["kv_heads"]
    for tokens, n_que in _requests(case):
        c = 0
        for i, r in enumerate(F.finch_schedule(tokens, case["chunk"], max(1, tokens // case["ratio"]))):
            x, y = _step_work(case, c, min(case["chunk"], tokens - i * case["chunk"]), r, n_que, case["doc_rows"])
            b, f, c = b + heads * x, f + heads * y, r
    return {"bytes": b, "flops": f}


def tolerance(case):
    # scores are fp32 sums of fp32 weights; K and V rows are copies, but turned keys are rounded
    # to the storage type once more, at every step a key moves in
    if case["rope"]:
        return {"rel": 1e-2 if case["dtype"] == "bf16" else 1e-5}
    return {"rel": 1e-5, "max": 1e-3}
