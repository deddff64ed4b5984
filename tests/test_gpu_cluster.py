"""Steps in which several workgroups share a problem (bf16, batches much smaller than the
chip): sizes at the edges of slices, row chunks, row splits and of the batch sizes that take
this launch; the waits between workgroups forced to run out (every workgroup then does the
others' work as well); layer groups, turned keys and the exact denominator; replays of a
captured graph."""
import pytest
import torch

import paper_2408_00167_amd as F
from tests import gpu_harness as H
from tests.test_gpu_layer import validate_layers
from tests.test_gpu_parity import _which_scoring_kernels

pytestmark = pytest.mark.gpu

# name -> (specs, whether this launch takes them)
BATCHES = {
    "tiny": ([dict(n_que=3, c=0, m=1, r=1), dict(n_que=1, c=0, m=0, r=4), dict(n_que=9, c=5, m=26, r=7),
              dict(n_que=8, c=1, m=31, r=31), dict(n_que=8, c=1, m=32, r=33), dict(n_que=2, c=70, m=0, r=0)], True),
    "one": ([dict(n_que=48, c=704, m=4096, r=748)], True),
    "row_chunks": ([dict(n_que=160, c=100, m=500, r=77), dict(n_que=65, c=0, m=300, r=20)], True),
    "sliced": ([dict(n_que=40 + p, c=37 * p, m=900 + 61 * p, r=100 + p) for p in range(12)], True),
    "two_slices": ([dict(n_que=5, c=10, m=150 + p % 7, r=60) for p in range(128)], True),
    "too_many": ([dict(n_que=5, c=10, m=150, r=60)] * 129, False),
    "longest": ([dict(n_que=6, c=5872, m=10000, r=5000), dict(n_que=6, c=0, m=64, r=9)], True),
    "too_long": ([dict(n_que=6, c=5873, m=10000, r=5000)], False),
}


@pytest.mark.parametrize("d,group", [(128, 4), (64, 2)])
@pytest.mark.parametrize("name", list(BATCHES))
def test_batches(name, d, group):
    specs, taken = BATCHES[name]
    fin = F.Finch(F.FINCH_BF16, d, group)
    batch, ts = H.single_step_case(fin, specs, torch.bfloat16, d, group, seed=31)
    assert (_which_scoring_kernels(fin, batch) == {"owner"}) == taken
    H.validate_single_step(ts, f"{name} d={d}")
    fin.close()


@pytest.mark.parametrize("layer,exact", [(1, False), (4, True)])
def test_work_of_missing_workgroups_is_done_by_the_others(layer, exact):
    """With a wait of 0 every workgroup finds some of the others missing and does their slices
    too: the same bits as with the usual wait, at every repetition."""
    specs = [dict(n_que=33, c=64 * (p // 4), m=700, r=150 + p // 4, prompt_keys=exact) for p in range(8)]
    want = None
    for ticks in (20_000_000, 0, 0, 20_000_000):
        fin = F.Finch(F.FINCH_BF16, 128, 4)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_GROUP, layer)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_WAIT_TICKS, ticks)
        if exact:
            fin.set_reposition(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING, 10000.0)
        batch, ts = H.single_step_case(fin, specs, torch.bfloat16, 128, 4, seed=5)
        if exact:
            fin.prompt_lse(batch)
        for _ in range(3):
            fin.step(batch)
        assert fin.workspace_status() == 0
        got = [t[k].clone() for t in ts for k in ("scores", "idx", "k_out", "v_out")]
        if want is None:
            want = got
            if layer == 1:
                H.validate_single_step(ts, "usual wait")
        for a, b in zip(got, want):
            assert torch.equal(a, b)
        fin.close()


# Slices of several key blocks and row blocks: the tiles a wave holds are formed once more after it
# has helped, by waves with four tiles beside waves with none; and what is not held in registers.
HELPED = {
    "held_5x5": [dict(n_que=40, c=100 + p, m=4900 - 3 * p, r=300 + p) for p in range(8)],
    "held_5x6": [dict(n_que=48, c=700, m=4096, r=750)] * 8,
    "held_6x3": [dict(n_que=24, c=0, m=6140 - p, r=90) for p in range(8)],
}


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("name", list(HELPED))
def test_helping_over_several_blocks(name, d):
    """As above, where a slice is several key blocks: bits of the usual wait, which the oracle checks."""
    want = None
    for ticks in (20_000_000, 0, 0, 0):
        fin = F.Finch(F.FINCH_BF16, d, 4)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_WAIT_TICKS, ticks)
        batch, ts = H.single_step_case(fin, HELPED[name], torch.bfloat16, d, 4, seed=41)
        for _ in range(4):
            for t in ts:
                t["scores"][:-1].fill_(-3.0)
            fin.step(batch)
            got = [t[k].clone() for t in ts for k in ("scores", "idx", "k_out", "v_out")]
            if want is None:
                want = got
                H.validate_single_step(ts, f"{name} d={d}")
            for a, b in zip(got, want):
                assert torch.equal(a, b), (name, d, ticks)
        fin.close()


def test_helping_where_heads_share_prompt_rows():
    """Problems of a layer with the same query pointer and different numbers of prompt rows: a
    workgroup that helps must not go on with the rows it has staged for the shorter prompt."""
    want = None
    for ticks in (20_000_000, 0, 0, 0):
        fin = F.Finch(F.FINCH_BF16, 128, 4)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_GROUP, 4)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_WAIT_TICKS, ticks)
        _, ts = H.single_step_case(fin, [dict(n_que=40 - p % 4, c=64, m=700, r=150) for p in range(8)], torch.bfloat16,
                                   128, 4, seed=55)
        for p, t in enumerate(ts):
            t["q"] = ts[p - p % 4]["q"][:4 * t["n_que"]]
        batch = F.Batch([dict(t, scores=t["scores"][:-1], idx=t["idx"][:-1], k_out=t["k_out"][:-1], v_out=t["v_out"][:-1])
                         for t in ts])
        for _ in range(4):
            fin.step(batch)
            got = [t[k].clone() for t in ts for k in ("scores", "idx", "k_out", "v_out")]
            if want is None:
                want = got
                validate_layers(ts, 4, "shared rows")
            for a, b in zip(got, want):
                assert torch.equal(a, b), ticks
        fin.close()


def _kernels_of(fin, call, batch):
    F.finch_profile(fin.ctx, True)
    call(batch)
    torch.cuda.synchronize()
    prof = F.finch_profile_read(fin.ctx)
    F.finch_profile(fin.ctx, False)
    return {k for k, v in prof.items() if v["launches"]}


@pytest.mark.parametrize("d,layer,rows,problems,n,taken", [
    (64, 1, 32, 128, 3599, True), (64, 1, 32, 128, 3600, False), (128, 1, 256, 128, 3600, False),
    (128, 1, 288, 128, 3600, True), (64, 8, 256, 128, 3600, True), (64, 8, 288, 128, 3600, False),
    (64, 1, 32, 88, 6000, True), (64, 1, 32, 80, 6000, False)])
def test_batches_at_the_line_to_one_kernel_per_stage(d, layer, rows, problems, n, taken):
    """Where the kernels per stage would put as many slices on the chip in one round they take over
    (128 problems: from 3600 candidates); both sides of the line against the oracle."""
    specs = [dict(n_que=rows, c=100, m=n - 100, r=77)] * problems
    fin = F.Finch(F.FINCH_BF16, d, 1)
    F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_GROUP, layer)
    batch, ts = H.single_step_case(fin, specs, torch.bfloat16, d, 1, seed=77)
    assert (_kernels_of(fin, fin.step, batch) == {"owner"}) == taken
    if layer == 1:
        H.validate_single_step(ts[::9], "line")
    else:
        validate_layers(ts[:2 * layer], layer, "line")
    fin.close()


def test_scores_alone_take_the_line_earlier():
    fin = F.Finch(F.FINCH_BF16, 64, 1)
    for n, scores_taken in ((5999, True), (6000, False)):  # 64 problems: four slices here, three per stage
        batch, ts = H.single_step_case(fin, [dict(n_que=32, c=100, m=n - 100, r=77)] * 64, torch.bfloat16, 64, 1, seed=78)
        assert (_kernels_of(fin, fin.score, batch) == {"owner"}) == scores_taken
        fin.topk(batch)
        fin.compact(batch)
        H.validate_single_step(ts[::9], f"scores alone n={n}")
        assert _kernels_of(fin, fin.step, batch) == {"owner"}
    fin.close()


def _fastest(f, repeats=8):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(repeats):
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_work_that_is_being_done_is_not_done_twice():
    """Slices whose passes take longer than the 0.1 ms after which a workgroup that waits in vain
    helps (here 0.17 ms a pass): nobody is missing, so the launch takes no longer than the kernels
    per stage do.  0.76 of their time; 1.7 times when the time spent working counted as time waited."""
    specs = [dict(n_que=256, c=625, m=4375, r=833)] * 85
    fin = F.Finch(F.FINCH_BF16, 128, 4)
    batch, _ = H.single_step_case(fin, specs, torch.bfloat16, 128, 4, seed=3)
    assert _which_scoring_kernels(fin, batch) == {"owner"}
    shared = _fastest(lambda: fin.step(batch))
    fin.set_step_path(F.FINCH_PATH_SEPARATE)
    per_stage = _fastest(lambda: fin.step(batch))
    print(f"shared {shared * 1e3:.0f} us, per stage {per_stage * 1e3:.0f} us", flush=True)
    assert shared < 1.25 * per_stage
    fin.close()


OUT = ("scores", "idx", "k_out", "v_out")


def _clobber(ts):
    for t in ts:
        t["scores"][:-1].fill_(-6.0)
        t["idx"][:-1].fill_(-7)
        t["k_out"][:-1].fill_(7.0)
        t["v_out"][:-1].fill_(7.0)


@pytest.mark.parametrize("static", [False, True])
def test_graphs_outlive_their_context(static):
    """A captured step uses nothing of its context: replays after the context is gone, with other
    contexts made and used in between, give the eager results."""
    specs = [dict(n_que=20 + p, c=100, m=600 + 40 * p, r=120) for p in range(8)]
    fin = F.Finch(F.FINCH_BF16, 128, 4)
    batch, ts = H.single_step_case(fin, specs, torch.bfloat16, 128, 4, seed=16)
    call = fin.step_static if static else fin.step
    call(batch)
    H.validate_single_step(ts, "eager")
    want = [t[k].clone() for t in ts for k in OUT]
    ws = fin.ws  # (the workspace stays with the graph)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(batch)
    fin.close()
    del fin, call
    others = []
    for i in range(4):
        others.append(F.Finch(F.FINCH_BF16, 64, 2))
        b2, t2 = H.single_step_case(others[-1], specs, torch.bfloat16, 64, 2, seed=17 + i)
        _clobber(ts)
        g.replay()
        others[-1].step(b2)  # eager work of the program's own between the replays
        if i == 2:
            others.pop(0).close()
        torch.cuda.synchronize()
        for a, b in zip([t[k] for t in ts for k in OUT], want):
            assert torch.equal(a, b), i
        H.validate_single_step(t2, f"between {i}")
    del ws


def test_graphs_of_one_context_side_by_side():
    """Two captured steps of one context, each with a workspace of its own, replayed on two streams
    at once and beside eager steps of the context."""
    fin = F.Finch(F.FINCH_BF16, 128, 4)
    cases, graphs, spaces = [], [], []
    for i in range(3):
        specs = [dict(n_que=24, c=50 * i, m=900 + 64 * i, r=130 + i)] * 8
        cases.append(H.single_step_case(fin, specs, torch.bfloat16, 128, 4, seed=60 + i))
    for batch, ts in cases:
        fin.step(batch)
        H.validate_single_step(ts, "eager")
    want = [[t[k].clone() for t in ts for k in OUT] for _, ts in cases]
    for batch, _ in cases[:2]:
        need = F.finch_workspace_size(fin.ctx, batch.host, batch.n)
        spaces.append(torch.empty(need, dtype=torch.uint8, device="cuda"))
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            F.finch_step(fin.ctx, batch.host, batch.dev_ptr, batch.n, spaces[-1].data_ptr(), need,
                         torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for round_ in range(5):
        for _, ts in cases:
            _clobber(ts)
        torch.cuda.synchronize()
        for _ in range(10):
            for s, g in zip(streams, graphs):
                with torch.cuda.stream(s):
                    g.replay()
            fin.step(cases[2][0])
        torch.cuda.synchronize()
        for (_, ts), w in zip(cases, want):
            for a, b in zip([t[k] for t in ts for k in OUT], w):
                assert torch.equal(a, b), round_
    fin.close()


def test_contexts_come_and_go_during_a_capture():
    specs = [dict(n_que=20, c=100, m=600, r=120)] * 8
    gone = F.Finch(F.FINCH_BF16, 128, 4)
    batch, ts = H.single_step_case(gone, specs, torch.bfloat16, 128, 4, seed=18)
    gone.step(batch)
    H.validate_single_step(ts, "eager")
    want = [t[k].clone() for t in ts for k in OUT]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        gone.close()
        fin = F.Finch(F.FINCH_BF16, 128, 4)
        fin.step_static(batch)
        fin.close()
    for i in range(3):
        _clobber(ts)
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip([t[k] for t in ts for k in OUT], want):
            assert torch.equal(a, b), i


def test_replays_of_a_captured_step():
    specs = [dict(n_que=20, c=100, m=600, r=120)] * 8
    fin = F.Finch(F.FINCH_BF16, 128, 4)
    batch, ts = H.single_step_case(fin, specs, torch.bfloat16, 128, 4, seed=6)
    fin.step_static(batch)
    H.validate_single_step(ts, "eager")
    want = [t[k].clone() for t in ts for k in ("scores", "idx", "k_out", "v_out")]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fin.step_static(batch)
    for i in range(4):
        for t in ts:
            t["scores"].fill_(-5.0)
            t["k_out"].fill_(7.0)
        g.replay()
        if i == 1:
            fin.step_static(batch)  # eager work of the program's own between the replays
        torch.cuda.synchronize()
        for a, b in zip([t[k] for t in ts for k in ("scores", "idx", "k_out", "v_out")], want):
            assert torch.equal(a, b), i
    fin.close()


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("blocks,n_que", [(12, 64), (17, 64), (24, 50), (24, 96), (25, 64)])
def test_three_key_blocks_a_wave(blocks, n_que, d):
    """Eight slices of 12 to 25 key blocks: waves with three blocks in registers beside waves with two,
    one chunk of rows and two (where pass 2 loads them again), the first size past it, and ragged
    ends; the same bits where workgroups do others' slices in between."""
    n = 8 * 32 * blocks
    specs = [dict(n_que=n_que, c=100, m=n - 100 - 33 * (p % 5), r=200 + p) for p in range(32)]
    want = None
    for ticks in (20_000_000, 0):
        fin = F.Finch(F.FINCH_BF16, d, 4)
        F.finch_set_option(fin.ctx, F.FINCH_OPT_LAYER_WAIT_TICKS, ticks)
        batch, ts = H.single_step_case(fin, specs, torch.bfloat16, d, 4, seed=blocks)
        fin.step(batch)
        assert fin.workspace_status() == 0
        got = [t[k].clone() for t in ts for k in ("scores", "idx", "k_out", "v_out")]
        if want is None:
            want = got
            H.validate_single_step(ts, f"{blocks} blocks, {n_que} prompt tokens, d={d}")
        for a, b in zip(got, want):
            assert torch.equal(a, b)
        fin.close()
