"""Kept rows that the whole-loop kernels leave where they are until the last two steps: every
buffer a loop writes must end up bit for bit as after one finch_step per chunk, whatever the
descriptors look like - also where rows have to be moved at every step, because something else
reads or writes the buffers."""
import pytest
import torch

import paper_2408_00167_amd as F
from paper_2408_00167_amd.driver import ChunkLoop

pytestmark = pytest.mark.gpu

# (rows of the first cache, [(m, r) per step]) per slot
GROWING = [(0, [(257, 40), (257, 80), (257, 121), (257, 160), (100, 175)]), (0, [(257, 64), (257, 128), (31, 130)]), (0, [(5, 3)])]
FORMS = {
    "growing": dict(slots=GROWING),
    "first_cache": dict(slots=[(33, [(300, 90), (300, 91), (300, 200), (300, 201)])]),
    "shrinking": dict(slots=[(0, [(400, 300), (400, 250), (400, 200), (400, 260), (400, 300), (400, 310)])]),
    "all_kept_none_kept": dict(slots=[(0, [(64, 64), (64, 500), (0, 500), (64, 0), (64, 20), (70, 30), (1, 31)])]),
    "three_buffers": dict(slots=GROWING, buffers=3),
    "part_of_cache": dict(slots=[(0, [(300, 90), (300, 120), (300, 150), (300, 180)])], drop=7),
    "separate_chunks": dict(slots=GROWING, separate=True),
    "chunk_in_cache": dict(slots=[(0, [(300, 90), (300, 120), (40, 150), (300, 180), (300, 200)])], chunk_in_cache=2),
    "scores_in_chunk": dict(slots=[(0, [(300, 90), (300, 120), (300, 150), (300, 180)])], scores_in_chunk=True),
    "most_that_fits": dict(slots=[(0, [(5200, 5100), (700, 5300), (700, 5400), (700, 5500), (700, 5600)])]),
    "rope": dict(slots=GROWING, rope=(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING)),
    "rank": dict(slots=GROWING, rope=(F.FINCH_ROPE_INTERLEAVED, F.FINCH_ORDER_RANK)),
    "layer": dict(slots=GROWING[:1] * 4, layer=2),
    "doc_rows": dict(slots=GROWING, doc=True),
    "doc_rows_rope": dict(slots=GROWING, doc=True, rope=(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING)),
    "layer_rope": dict(slots=GROWING[:1] * 4, layer=2, rope=(F.FINCH_ROPE_INTERLEAVED, F.FINCH_ORDER_ASCENDING)),
}
# (turned keys: the values stay from 384 rows of 128 channels and 768 rows of 64 on; both sides of the line,
# enough rows for the values to stay with either width, and with as many document rows, and too few steps to stay)
for _d, _r in ((128, 384), (64, 768)):
    for _off in (-1, 0):
        FORMS[f"rope_line_{_d}_{_off}"] = dict(slots=[(9, [(900, _r // 2), (300, _r + _off), (257, _r - 40), (31, _r + _off), (64, _r - 1)])],
                                              rope=(F.FINCH_ROPE_INTERLEAVED, F.FINCH_ORDER_ASCENDING))
LONG = [(0, [(1025, 300), (513, 700), (257, 800), (257, 811), (100, 830)]), (0, [(900, 64), (900, 820), (31, 830)]), (0, [(5, 3)])]
for _name, _more in (("", {}), ("doc_rows_", dict(doc=True)), ("layer_", dict(slots=LONG[:1] * 4, layer=2)), ("three_buffers_", dict(buffers=3))):
    FORMS[f"{_name}rope_long"] = dict(dict(slots=LONG, rope=(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING)), **_more)
FORMS["two_steps"] = dict(slots=[(0, [(257, 40), (257, 80)]), (9, [(257, 64)])])
# (kernels for 2, 4 and 6 row blocks; GROWING's chunks take the one for 8)
for _m in (40, 100, 180):
    FORMS[f"doc_rows_rope_{_m}"] = dict(slots=[(17, [(_m, 20), (_m, 41), (_m, 45), (_m - 7, 66)])], doc=True,
                                        rope=(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING))
    FORMS[f"doc_rows_rope_long_{_m}"] = dict(slots=[(900, [(_m, 800), (_m, 810), (_m, 811), (_m - 7, 820)])], doc=True,
                                             rope=(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING))



def _case(form, d, group, n_que, seed):
    """Buffers and descriptors of one loop, drawn from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def rand(n):
        return torch.randn(max(n, 1), d, generator=g, device="cuda", dtype=torch.bfloat16)

    written, slots = [], []
    for c0, steps in form["slots"]:
        q, first = rand(group * n_que), (rand(c0), rand(c0))
        tokens = sum(m for m, _ in steps)
        cap = c0 + max(r for _, r in steps) + 1
        docs = (rand(tokens), rand(tokens))
        bufs = [(rand(cap), rand(cap)) for _ in range(form.get("buffers", 2))]
        scores = torch.zeros(cap + max(m for m, _ in steps), device="cuda")
        idx = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
        written += [t for b in bufs for t in b] + [scores, idx] + list(docs)
        c, lo, descs = c0, 0, []
        for i, (m, r) in enumerate(steps):
            k_chunk, v_chunk = docs[0][lo:lo + m], docs[1][lo:lo + m]
            if form.get("separate"):
                k_chunk, v_chunk = (k_chunk.clone(), v_chunk.clone()) if i % 2 else (v_chunk.clone(), k_chunk.clone())
            if form.get("chunk_in_cache") == i:  # some of the cache's rows once more
                k_chunk, v_chunk = bufs[i % 2][0][:m], bufs[i % 2][1][:m]
            cache = first if i == 0 else bufs[i % len(bufs)]
            out = bufs[(i + 1) % len(bufs)]
            keep = min(r, c + m)
            at = scores[:max(c + m, 1)]
            if form.get("scores_in_chunk") and i == 2:  # a chunk that has been read by then
                at = docs[0][:m].view(torch.float32).flatten()[:c + m]
            desc = dict(q=q, k_cache=cache[0][:c], v_cache=cache[1][:c], k_chunk=k_chunk, v_chunk=v_chunk, k_out=out[0][:max(keep, 1)],
                        v_out=out[1][:max(keep, 1)], scores=at, idx=idx[:max(keep, 1)], n_que=n_que, c=c, m=m, r=r)
            if form.get("doc"):
                desc["q_doc"] = rand(group * m)
            descs.append(desc)
            c, lo = max(0, keep - form.get("drop", 0)), lo + m
        slots.append(descs)
    steps = [[s[i] for s in slots if i < len(s)] for i in range(max(len(s) for s in slots))]
    return steps, written


@pytest.mark.parametrize("d,group,n_que", [(128, 4, 9), (64, 1, 70)])
@pytest.mark.parametrize("name", list(FORMS))
def test_loop_leaves_what_single_steps_leave(name, d, group, n_que):
    form = FORMS[name]
    left = []
    passes = 1 if "scores_in_chunk" in form else 2  # (what a pass leaves behind must not change the next one)
    for whole in (True, False):
        fin = F.Finch(F.FINCH_BF16, d, group)
        fin.set_step_path(F.FINCH_PATH_OWNER)
        if "rope" in form:
            fin.set_reposition(*form["rope"], 10000.0)
        if "layer" in form:
            F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_GROUP, form["layer"])
        steps, written = _case(form, d, group, n_que, seed=5)
        if whole:
            lb = F.LoopBatch(steps)
            for _ in range(passes):
                fin.loop(lb)
        else:
            batches = [F.Batch(s) for s in steps]
            for b in batches * passes:
                fin.step(b)
        torch.cuda.synchronize()
        left.append([t.cpu() for t in written])
        fin.close()
    for n, (a, b) in enumerate(zip(*left)):
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8)), f"{name}: buffer {n} differs"


@pytest.mark.parametrize("slots,lengths", [(63, [4]), (64, [4]), (64, [4, 2]), (160, [3]), (177, [3, 1]), (300, [2])])
def test_routes_of_loops_that_do_not_fill_the_chip(slots, lengths):
    """AUTO takes the one-launch loop from some number of slots on: the same results either side."""
    g = torch.Generator(device="cuda")
    g.manual_seed(slots)
    d, group, n_que, chunk, steps = 64, 2, 5, 160, max(lengths)
    rand = lambda *shape: torch.randn(*shape, generator=g, device="cuda", dtype=torch.bfloat16)
    problems = [dict(Q=rand(group * n_que, d), K=rand(chunk * lengths[p % len(lengths)] - 7, d), V=rand(chunk * lengths[p % len(lengths)] - 7, d),
                     n_que=n_que, budget=60) for p in range(slots)]
    left = []
    for path in (F.FINCH_PATH_AUTO, F.FINCH_PATH_OWNER):
        fin = F.Finch(F.FINCH_BF16, d, group)
        fin.set_step_path(path)
        loop = ChunkLoop(fin, problems, chunk)
        loop.run()
        torch.cuda.synchronize()
        left.append([t.cpu() for t in (*loop.kbuf, *loop.vbuf, loop.scores, loop.idx)])
        fin.close()
    worst = float(((left[0][4] - left[1][4]).abs() / left[1][4].clamp_min(1e-30)).max())
    assert worst < 1e-5, f"scores of the routes differ by {worst:.1e}"  # fp32 sums in another order
    for a, b in zip(left[0][:4] + left[0][5:], left[1][:4] + left[1][5:]):
        rows = (a != b).reshape(a.shape[0], -1).any(dim=1).float().mean() if a.dim() == 2 and a.shape[0] > 1 else (a != b).float().mean()
        assert float(rows) < 1e-3  # (two nearly equal scores may change places)
