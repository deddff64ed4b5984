"""Which launches AUTO makes, on both sides of the lines it draws: counted by kernel class while the call
runs.  (Inputs are shared by the problems of a batch: only sizes matter here.)"""
import pytest
import torch

import paper_2408_00167_amd as F
from paper_2408_00167_amd.driver import ChunkLoop

pytestmark = pytest.mark.gpu


def _launches(fin, call):
    F.finch_profile(fin.ctx, True)
    call()
    torch.cuda.synchronize()
    prof = F.finch_profile_read(fin.ctx)
    F.finch_profile(fin.ctx, False)
    return {k: v["launches"] for k, v in prof.items() if v["launches"]}


def _lines_hold():
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines are shares of the compute units, the sizes here those of 256")


# (problems, channels, rows, candidates, scores alone, one workgroup per problem)
STEPS = [
    (176, 128, 192, 512, False, False), (177, 128, 192, 512, False, True),           # 69 % of a round
    (177, 64, 256, 8192, False, True), (177, 64, 256, 8193, False, False),           # candidates of one round
    (199, 128, 192, 8193, False, False), (200, 128, 192, 12288, False, True), (200, 128, 192, 12289, False, False),
    (177, 128, 224, 9000, False, False), (177, 128, 225, 9000, False, True), (177, 128, 480, 9000, True, False), (177, 128, 481, 9000, True, True),
    (200, 128, 384, 9000, False, True), (200, 64, 385, 9000, False, False), (218, 128, 192, 12289, False, True),  # 85 %
    (177, 128, 257, 1024, False, True), (177, 128, 257, 1025, False, False), (177, 128, 257, 128, True, True),
    (177, 128, 320, 129, True, False), (177, 128, 321, 1025, False, True), (177, 64, 384, 1025, False, False),
    (177, 64, 385, 1025, False, True), (177, 64, 384, 300, True, False), (354, 64, 384, 300, False, False),
    (354, 128, 192, 2048, False, True), (354, 128, 192, 2049, False, False), (353, 128, 192, 2048, False, False),
    (354, 64, 65, 300, False, True), (354, 64, 65, 300, True, False), (354, 64, 64, 300, True, True), (354, 128, 300, 300, False, True), (354, 128, 300, 301, False, False),
]


@pytest.mark.parametrize("problems,d,rows,n,scores_alone,one", STEPS)
def test_steps(problems, d, rows, n, scores_alone, one):
    _lines_hold()
    fin = F.Finch(F.FINCH_BF16, d, 1)
    rand = lambda *shape: torch.randn(*shape, device="cuda", dtype=torch.bfloat16)
    q, k, v, r = rand(rows, d), rand(n, d), rand(n, d), 8
    outs = [torch.zeros(problems, r, d, device="cuda", dtype=torch.bfloat16) for _ in range(2)]
    scores, idx = torch.zeros(problems, n, device="cuda"), torch.zeros(problems, r, device="cuda", dtype=torch.int32)
    batch = F.Batch([dict(q=q, k_cache=None, v_cache=None, k_chunk=k, v_chunk=v, k_out=outs[0][p], v_out=outs[1][p],
                          scores=scores[p], idx=idx[p], n_que=rows, c=0, m=n, r=r) for p in range(problems)])
    fin.reserve(batch)
    got = _launches(fin, lambda: (fin.score if scores_alone else fin.step)(batch))
    assert got == {"owner": 1} if one else "rowstats" in got and "owner" not in got, got
    fin.close()


# (slots, channels, rows, tokens a chunk, steps, rows kept, keys turned, whole loop in one launch)
LOOPS = [
    (63, 128, 64, 500, 16, 512, False, False), (64, 128, 64, 500, 16, 512, False, True), (64, 128, 64, 500, 9, 512, False, False),
    (64, 128, 64, 500, 16, 512, True, False), (72, 128, 64, 500, 16, 512, True, True), (72, 128, 160, 500, 16, 512, False, False),
    (64, 128, 192, 1024, 16, 1024, False, False), (64, 64, 64, 1024, 8, 512, False, True), (64, 64, 65, 1024, 8, 512, False, False),
    (64, 64, 192, 500, 16, 512, False, True), (64, 64, 193, 500, 16, 512, False, False), (72, 64, 37, 652, 18, 1055, False, True),
    (72, 64, 37, 652, 18, 1055, True, False), (64, 128, 64, 540, 16, 512, False, False), (64, 128, 64, 500, 16, 2000, False, False),
    (86, 128, 192, 1024, 10, 512, False, True), (95, 128, 192, 1024, 8, 512, False, False), (96, 128, 192, 1024, 8, 512, False, True),
    (112, 128, 192, 2048, 4, 512, False, False), (128, 128, 192, 2048, 4, 512, False, True), (96, 64, 256, 1024, 8, 512, False, True),
    (96, 64, 256, 1100, 8, 512, False, False), (96, 64, 64, 2500, 4, 512, True, False), (96, 64, 64, 2500, 4, 512, False, True),
    (130, 128, 192, 3800, 4, 400, True, True), (130, 128, 192, 3900, 4, 400, True, False),
    # (from 69 % on by the tokens of a chunk, with turned keys by the candidates)
    (177, 128, 192, 13300, 4, 400, False, True), (177, 128, 192, 13500, 4, 400, False, False), (177, 128, 192, 13100, 4, 400, True, False),
    (177, 64, 256, 7100, 4, 2000, False, True), (177, 64, 256, 7100, 4, 2000, True, False), (177, 64, 256, 8400, 4, 400, False, False),
    (354, 128, 192, 7100, 4, 400, False, True), (354, 128, 192, 7200, 4, 400, False, False), (354, 128, 192, 7100, 4, 400, True, False),
    (384, 128, 192, 7200, 4, 400, False, True), (354, 128, 481, 6700, 4, 400, True, True),
    (177, 128, 480, 7100, 4, 2000, False, True), (177, 128, 480, 7200, 4, 2000, False, False), (410, 128, 480, 6100, 4, 400, False, True),
    (354, 128, 300, 1500, 4, 100, False, True), (354, 128, 300, 1600, 4, 100, False, False), (354, 128, 192, 2100, 16, 8400, False, True), (354, 128, 192, 2100, 16, 8400, True, False),
    (354, 64, 256, 3050, 4, 400, False, True), (354, 64, 256, 3200, 4, 400, False, False), (354, 64, 64, 13000, 4, 400, False, True),
    (354, 128, 384, 2500, 4, 400, False, True), (354, 128, 384, 2700, 4, 400, False, False), (354, 64, 257, 300, 4, 40, False, False),
]


@pytest.mark.parametrize("slots,d,rows,chunk,steps,budget,turned,one", LOOPS)
def test_loops(slots, d, rows, chunk, steps, budget, turned, one):
    _lines_hold()
    fin = F.Finch(F.FINCH_BF16, d, 1)
    if turned:
        fin.set_reposition(F.FINCH_ROPE_HALF, F.FINCH_ORDER_ASCENDING, 10000.0)
    rand = lambda *shape: torch.randn(*shape, device="cuda", dtype=torch.bfloat16)
    q, k, v = rand(rows, d), rand(chunk * steps, d), rand(chunk * steps, d)
    loop = ChunkLoop(fin, [dict(Q=q, K=k, V=v, n_que=rows, budget=budget) for _ in range(slots)], chunk)
    got = _launches(fin, loop.run)
    assert (got == {"owner": 1}) == one, got
    assert one or sum(got.values()) >= steps, got
    fin.close()
