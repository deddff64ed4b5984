"""fp32 inputs, one workgroup per problem: candidates and rows at the edges of the 16 x 16 tiles
and of what is kept between the passes (1024 candidates), with prompt rows, rows of the
chunk's own tokens, or both."""
import pytest
import torch

import paper_2408_00167_amd as F
from tests import gpu_harness as H
from tests.test_gpu_parity import _which_scoring_kernels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,group", [(64, 1), (128, 2)])
@pytest.mark.parametrize("rows", ["prompt", "document", "both"])
def test_tile_edges(d, group, rows):
    fin = F.Finch(F.FINCH_F32, d, group)
    fin.set_step_path(F.FINCH_PATH_OWNER)
    sizes = [(1, 0), (3, 12), (0, 16), (10, 7), (100, 28), (1000, 23), (1008, 16), (1000, 25), (1500, 48)]
    specs = [dict(n_que=n, c=c, m=m, r=max(1, (c + m) // 3), doc_rows=rows != "prompt", no_prompt=rows == "document")
             for (c, m), n in zip(sizes, (1, 15, 16, 17, 31, 32, 33, 8, 16)) if rows == "prompt" or m > 0]
    batch, ts = H.single_step_case(fin, specs, torch.float32, d, group, seed=12)
    fin.step(batch)
    H.validate_single_step(ts, f"tiles d={d} {rows}")
    fin.close()


@pytest.mark.parametrize("d,rows,problems,n,owner", [
    (64, 5, 1, 1024, True), (64, 5, 1, 1025, False), (64, 6, 1, 4096, True), (128, 1, 1, 4096, True),
    (64, 1, 100, 1500, True), (64, 1, 100, 1501, False), (64, 4, 192, 2881, False), (64, 1, 193, 4096, True)])
def test_few_rows_and_many_candidates(d, rows, problems, n, owner):
    """Which launch AUTO takes where the tiles of 16 rows are mostly padding; both against the oracle."""
    fin = F.Finch(F.FINCH_F32, d, 1)
    batch, ts = H.single_step_case(fin, [dict(n_que=rows, c=100, m=n - 100, r=60)] * problems, torch.float32, d, 1, seed=14)
    assert (_which_scoring_kernels(fin, batch) == {"owner"}) == owner
    H.validate_single_step(ts[::20], f"d={d} rows={rows} n={n}")
    fin.close()
