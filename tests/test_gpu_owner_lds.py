"""One workgroup per problem: the launch's LDS is what its largest problem's selection needs, so
single-problem batches are the tightest fit.  Sizes around what fits a step's order keys into
LDS at all (15872 candidates; kept indices and keys together 60 KB), and slots by rank at the
edges of the records' power of two."""
import pytest
import torch

import paper_2408_00167_amd as F
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n_que", [(64, 5), (64, 100), (128, 200)])
@pytest.mark.parametrize("n,r", [(1, 1), (2, 1), (33, 32), (513, 100), (7000, 6999), (15000, 200), (15000, 400),
                                 (12000, 3300), (15872, 1), (15873, 1), (15873, 15000)])
def test_selection_scratch_fits(d, n_que, n, r):
    fin = F.Finch(F.FINCH_BF16, d, 1)
    fin.set_step_path(F.FINCH_PATH_OWNER)
    specs = [dict(n_que=n_que, c=n // 3, m=n - n // 3, r=r)]
    batch, ts = H.single_step_case(fin, specs, torch.bfloat16, d, 1, seed=n + r)
    fin.step(batch)
    H.validate_single_step(ts, f"d={d} n={n} r={r}")
    ts[0]["scores"][:-1].fill_(-5.5)
    fin.score(batch)
    H.validate_single_step(ts, f"scores alone d={d} n={n} r={r}")
    fin.close()


@pytest.mark.parametrize("r", [1, 63, 64, 65, 1024, 1025, 2047, 2048])
def test_ranked_slots_fit(r):
    fin = F.Finch(F.FINCH_BF16, 64, 1)
    fin.set_step_path(F.FINCH_PATH_OWNER)
    fin.set_reposition(F.FINCH_ROPE_HALF, F.FINCH_ORDER_RANK, 10000.0)
    batch, ts = H.single_step_case(fin, [dict(n_que=7, c=0, m=max(r, 40), r=r)], torch.bfloat16, 64, 1, seed=r)
    fin.step(batch)
    H.validate_single_step(ts, f"rank r={r}", repos=("half", "rank", 10000.0))
    fin.close()
