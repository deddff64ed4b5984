"""Whole loops that select on one pass over the keys in steps whose scores the next step overwrites
(RowEstimates in csrc/owner_body.h): caches, indices and the last scores must be those of one
finch_step per chunk, which makes both passes - where no key is near the line, where many are and
some or all of them have to be scored exactly, where guesses are of no use (rows that find far
larger logits than before, and rows that are not numbers), and where a step's scores are seen.  The launches
write down which way each step took, so that a test knows that its data has taken the way it is there for."""
import ctypes

import pytest
import torch

import paper_2408_00167_amd as F
from paper_2408_00167_amd.driver import ChunkLoop

pytestmark = pytest.mark.gpu

# kWay... in csrc/finch_internal.h
ONCE, SETTLED, LIST, ALL, RANGE, AGAIN = 1, 2, 4, 8, 16, 32
BITS = {torch.float32: torch.int32, torch.bfloat16: torch.int16, torch.int32: torch.int32}  # (compared so: NaN as well)


def _record_ways(fin, steps, slots):
    """Where the loops of `fin` will write how each step of each slot has selected (-1: not by these kernels, or not there)."""
    ways = torch.full((steps, slots), -1, dtype=torch.int32, device="cuda")
    assert F.load_library().finch_debug_loop_ways(fin.ctx, ctypes.c_void_p(ways.data_ptr())) == F.FINCH_OK
    return ways


def _problems(kind, d, group, n_que, tokens, chunk, budget, count, seed, exact):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def rand(*shape):
        return torch.randn(*shape, generator=g, device="cuda")

    out = []
    for _ in range(count):
        q, k, v = rand(group * n_que, d), rand(tokens, d), rand(tokens, d)
        a = rand(d)
        a /= a.norm()
        if kind == "gap":  # relevant keys, as many in every chunk as the schedule adds, far above the others
            q += 2.5 * a
            kept = 0
            for i, r in enumerate(F.finch_schedule(tokens, chunk, budget)):
                n = min(chunk, tokens - i * chunk)
                at = torch.rand(n, generator=g, device="cuda").topk(min(n, r - kept)).indices + i * chunk
                k[at] += (1.6 + 0.8 * torch.rand(len(at), 1, generator=g, device="cuda")) * d ** 0.5 * a
                kept = r
        elif kind == "ties":  # every key many times
            k = k[:37].repeat(-(-tokens // 37), 1)[:tokens].contiguous()
        elif kind == "jump":  # half of the rows meet a key from the third chunk on that outweighs all before
            q[::2] += 4 * a
            k[2 * chunk::chunk] += 30 * a
        elif kind == "peaked":  # nearly all scores below the least that fp32 can hold
            q *= 40
        elif kind == "nan":
            q[1, 0] = float("nan")
        out.append(dict(Q=q.bfloat16(), K=k.bfloat16(), V=v.bfloat16(), n_que=n_que, budget=budget))
        if exact:
            out[-1]["K_que"] = rand(n_que, d).bfloat16()
    return out


def _run(kind, d, group, n_que, tokens, chunk, budget, seed=0, rope=False, exact=False, want_scores=True, count=3,
         seen=0, once=True):
    """`seen`: one of these ways has been taken by some step; `once`: the kernels with one pass ran (else: they did not)."""
    probs = _problems(kind, d, group, n_que, tokens, chunk, budget, count, seed, exact)
    got = []
    for per_step in (False, True):
        fin = F.Finch(F.FINCH_BF16, d, group)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_STEP_PATH, F.FINCH_PATH_OWNER)
        if rope:
            fin.set_reposition(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING, 10000.0)
        loop = ChunkLoop(fin, probs, chunk, want_scores=want_scores)
        ways = _record_ways(fin, loop.n_steps, count)
        for _ in range(2):  # (the second time with what the first has left in the buffers)
            loop.run(per_step=per_step)
        torch.cuda.synchronize()
        got.append([loop.final_cache(p) for p in range(count)] + [loop.idx, loop.scores])
        got[-1] = [x for y in got[-1] for x in (y if isinstance(y, tuple) else (y,)) if x is not None]
        assert bool((ways[0] >= 0).all()) == (once and not per_step), ways
        assert per_step or not seen or bool(((ways > 0) & (ways & seen > 0)).any()), ways
    for a, b in zip(*got):
        assert torch.equal(a.view(BITS[a.dtype]), b.view(BITS[b.dtype]))


@pytest.mark.parametrize("kind", ["gap", "dense", "ties", "jump", "peaked"])
@pytest.mark.parametrize("d,group,n_que", [(128, 1, 16), (128, 2, 33), (128, 4, 48), (128, 4, 64), (64, 4, 40)])
def test_as_step_by_step(kind, d, group, n_que):
    """Row blocks 1, 3, 6, 8 and 5; a last chunk that is shorter (the one before it is seen) and ragged key blocks."""
    seen = {"gap": SETTLED, "dense": LIST | ALL, "ties": 0, "jump": LIST | ALL | RANGE, "peaked": RANGE}[kind]
    _run(kind, d, group, n_que, tokens=9401, chunk=2215, budget=600, seen=seen)


@pytest.mark.parametrize("rows", [32, 64, 96, 128, 160, 192, 224, 256])
@pytest.mark.parametrize("d", [64, 128])
def test_every_number_of_row_blocks(rows, d):
    _run("gap", d, 1, rows, tokens=9000, chunk=2600, budget=400, count=2, seen=SETTLED)
    _run("dense", d, 1, rows - 31, tokens=9000, chunk=2600, budget=400, count=2)
    line = 400 * ((rows + 31) // 32 + 1) * d >= 2600 * 128  # (few rows: below it, by the kernels for two passes)
    _run("gap", d, 1, rows, tokens=1600, chunk=320, budget=100, once=line)


@pytest.mark.parametrize("kind", ["gap", "dense", "ties", "jump", "nan"])
@pytest.mark.parametrize("d,group,n_que", [(128, 1, 257), (128, 4, 96), (64, 8, 70), (64, 4, 260)])
def test_several_chunks_of_rows(kind, d, group, n_que):
    """257, 384 and 560 rows in chunks of 256, and more rows than guesses are kept for; open keys start the step over."""
    _run(kind, d, group, n_que, tokens=2500, chunk=515, budget=190, want_scores=kind != "nan", count=2,
         seen=SETTLED if kind == "gap" and group * n_que <= 1024 else 0)


@pytest.mark.parametrize("kind", ["gap", "dense"])
def test_options(kind):
    _run(kind, 128, 4, 24, 5600, 900, 400, rope=True)
    seen = SETTLED if kind == "gap" else LIST
    _run(kind, 128, 4, 24, 11200, 1800, 400, exact=True, seen=seen)
    _run(kind, 128, 4, 24, 11200, 1800, 400, want_scores=False, seen=seen)
    _run(kind, 128, 2, 24, 15000, 2500, 2400, seen=seen)   # many kept rows
    _run(kind, 128, 1, 40, 4800, 400, 4400, seen=seen)     # nearly all rows are kept
    _run(kind, 128, 8, 24, 1500, 400, 60)       # small chunks


def test_mixed_lengths_in_one_launch():
    """Slots with other numbers of rows and steps beside each other (a kernel for more row blocks than a slot has)."""
    probs = [p for i, (t, n) in enumerate([(2900, 64), (2100, 9), (1500, 33), (300, 50)])
             for p in _problems("gap" if i % 2 else "dense", 128, 4, n, t, 300, max(1, t // 12), 2, 5 + i, False)]
    outs = []
    for per_step in (False, True):
        fin = F.Finch(F.FINCH_BF16, 128, 4)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_STEP_PATH, F.FINCH_PATH_OWNER)
        loop = ChunkLoop(fin, probs, 300)
        loop.run(per_step=per_step)
        torch.cuda.synchronize()
        outs.append([t for p in range(len(probs)) for t in loop.final_cache(p)] + [loop.idx, loop.scores])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


def test_rows_that_are_not_numbers_end_the_same_way():
    """A row of NaN makes every score NaN; nothing is taken to stand clear, and the launch ends with the
    indices of the two passes."""
    _run("nan", 128, 2, 20, 4000, 900, 100, want_scores=False)
    _run("nan", 128, 2, 20, 1500, 300, 100, want_scores=False, once=False)


def _free_loop(q, chunks, kept, d, group):
    """One slot whose steps see these chunks alone and keep `kept` rows of them, in one launch and step by step: the
    indices of all steps, and the ways they took.  (The chunks in one allocation: with some of them more than
    16 GiB apart, where an allocator may put them, the loop takes the kernels for two passes.)"""
    q, chunks = q.bfloat16().cuda(), torch.stack(chunks).bfloat16().cuda()
    n, big = chunks.shape[1], max(kept)
    outs = []
    for per_step in (False, True):
        fin = F.Finch(F.FINCH_BF16, d, group)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_STEP_PATH, F.FINCH_PATH_OWNER)
        scores, idx = torch.zeros(n, device="cuda"), torch.zeros(len(chunks), big, dtype=torch.int32, device="cuda")
        rows = torch.zeros(2, len(chunks), big, d, dtype=torch.bfloat16, device="cuda")
        steps = [[dict(q=q, k_cache=None, v_cache=None, k_chunk=k, v_chunk=k, k_out=rows[0, i, :r], v_out=rows[1, i, :r],
                       scores=scores, idx=idx[i, :r], n_que=len(q) // group, c=0, m=n, r=r)]
                 for i, (k, r) in enumerate(zip(chunks, kept))]
        if per_step:
            for s in steps:
                batch = F.Batch(s)
                fin.reserve(batch)
                fin.step(batch)
        else:
            batch = F.LoopBatch(steps)
            fin.reserve_loop(batch)
            ways = _record_ways(fin, len(chunks), 1)
            fin.loop(batch)
        torch.cuda.synchronize()
        outs.append([idx, scores, rows])
        fin.close()
    for a, b in zip(*outs):
        assert torch.equal(a.view(BITS[a.dtype]), b.view(BITS[b.dtype]))
    return outs[0][0].cpu(), ways[:, 0].tolist()


@pytest.mark.parametrize("way", ["up", "down"])
@pytest.mark.parametrize("rows,first,top", [(192, 0, 34.5), (384, 0, 34.25), (384, 256, 34.75)])
def test_rows_that_all_move_far_at_once(way, rows, first, top):
    """All log-sum-exps of two groups of rows (from row `first` on; the others stay) move by one step.  They rise by 2^109
    and 2^123, so that sums over the rows leave fp32's range while every row's sum is in it (`top`: two keys' sums are
    infinite, a third's within 5 % below 2^128, which share the selection's highest bin), or fall by 2^120, so that a
    row's sum loses the many terms below 2^-126.  Guesses are of no use, and the step makes both passes."""
    d, group, n, half = 128, 4, 2000, (rows - first) // 2
    q = torch.zeros(rows, d)
    q[first:first + half, 0] = 32  # (a key's channel counts 32 / sqrt(128) * log2(e) = 4.08 octaves)
    q[first + half:, 1] = 32
    noise = 0.05 * torch.randn(3, n, d, generator=torch.Generator().manual_seed(rows + first))
    noise[:, :, :2] = 0
    chunks = list(noise)
    chunks[0][700, :2] = 4.5 if way == "up" else 34.0  # stands clear: the next step tries one pass
    if way == "up":
        chunks[1][[10, 20], 0] = top   # two fifths of the first group's weight each ...
        chunks[1][30, 0] = top - 0.25  # (half of that)
        chunks[1][1500, 1] = 31.25     # ... and all of the second's
        want = [10, 1500]
    else:
        chunks[1][:, 0] = 2.75         # nearly all of the first group's weight together
        chunks[1][10, 0] = 4.5
        chunks[1][[1500, 1600], :2] = torch.tensor([0.0, 4.5])  # half of the second group's each
        want = [1500, 1600]
    k = chunks[1].bfloat16().double()
    exact = torch.softmax(q.double() @ k.T / d ** 0.5, 1).sum(0)
    assert sorted(torch.sort(exact, descending=True, stable=True).indices[:2].tolist()) == want
    got, ways = _free_loop(q, chunks, [1, 2, 2], d, group)
    assert got[0, 0] == 700 and got[1].tolist() == want
    assert ways[1] == ONCE | RANGE


@pytest.mark.parametrize("rows", [31, 192, 384])
@pytest.mark.parametrize("kind", ["open", "tiny", "nan"])
def test_keys_that_one_pass_leaves_open(kind, rows):
    """A step whose first group of rows rises by three octaves, with keys of either group near the line; one that keeps keys
    whose sums are too small for bounds; and one that meets a key that is not a number.  One chunk of rows and two."""
    d, n, kept = 128, 2000, 40
    g = torch.Generator().manual_seed(rows)
    q = torch.zeros(rows, d)
    q[:rows // 2, 0] = q[rows // 2:, 1] = 32
    chunks = list(0.05 * torch.randn(3, n, d, generator=g))
    chunks[0][700, :2] = 4.5  # stands clear: the next step tries one pass
    near = torch.randperm(n, generator=g)[:2 * kept]
    if kind == "tiny":
        chunks[1][:, :2] = -20 - torch.rand(n, 1, generator=g)
        chunks[1][near[:kept // 2], :2] = 4.5
    else:
        for i in range(2):
            chunks[1][near[i::2], i] = 3.0 + 0.1 * torch.rand(kept, generator=g)
        chunks[1][900, 0] = 5.25
    if kind == "nan":
        chunks[1][5, 7] = float("nan")
    got, ways = _free_loop(q, chunks, [1, kept, kept], d, 1)
    assert got[0, 0] == 700
    assert ways[1] == ONCE | {"nan": RANGE, "tiny": ALL if rows <= 256 else AGAIN, "open": LIST if rows <= 256 else AGAIN}[kind]


def test_what_a_step_has_learned_outlives_it():
    """Half of 384 rows rise or fall by three octaves each step, and a key two and a half octaves below the kept one is open to
    the step that tries one pass.  That step starts over; the next one still knows how far it had to look, and
    leaves it at two passes, and so does the one behind it."""
    d, n, rows = 128, 900, 384
    q = torch.zeros(rows, d)
    q[:rows // 2, 0] = q[rows // 2:, 1] = 32
    chunks = list(0.05 * torch.randn(6, n, d, generator=torch.Generator().manual_seed(1)))
    for i, k in enumerate(chunks):
        k[300, :2], k[400, :2] = 4.5, 4.5 - 0.625
        k[[300, 400], 0] += 0.75 * (i % 2)
    _, ways = _free_loop(q, chunks, [1] * 6, d, 1)
    assert ways[1] == ONCE | AGAIN
    assert ways[2] == ways[3] == 0


@pytest.mark.parametrize("rows", [192, 384])
@pytest.mark.parametrize("kind", ["range", "open", "tiny"])
def test_tries_of_no_use_become_rare(kind, rows):
    """Steps whose guesses never serve - half of the rows rise or fall by 30 octaves each time, by 3 with another key within
    them of the line, or the scores are too small - and then some whose guesses do.  What a try costs is paid once in
    the first eight steps and once more in the sixteen after them, and tries that serve are made again."""
    d, n, steps, calm = 128, 900, 22, 30
    g = torch.Generator().manual_seed(rows)
    q = torch.zeros(rows, d)
    q[:rows // 2, 0] = q[rows // 2:, 1] = 32
    chunks, kept = list(0.05 * torch.randn(steps + calm, n, d, generator=g)), [1] * (steps + calm)
    for i, k in enumerate(chunks):
        k[300, :2] = 4.5  # stands clear
        if i < steps and kind == "tiny" and i > 0:
            k[:, :2] = -20 - torch.rand(n, 1, generator=g)
            k[:20, :2] = 4.5
            kept[i] = 40
        elif i < steps and kind != "tiny":
            k[400, :2] = 4.5 - 0.625  # two and a half octaves below
            k[[300, 400], 0] += (7.5 if kind == "range" else 0.75) * (i % 2)
    _, ways = _free_loop(q, chunks, kept, d, 1)
    no_use = {"range": RANGE, "open": AGAIN, "tiny": ALL if rows <= 256 else AGAIN}[kind]
    if kind == "open" and rows <= 256:  # a list of two keys: it pays
        assert all(w == ONCE | LIST for w in ways[1:steps])
    else:
        assert ways[1] == ONCE | no_use
        assert sum(w & no_use > 0 for w in ways[:steps]) <= 2
    assert sum(w & SETTLED > 0 for w in ways[steps:]) >= calm // 2 - 2
