"""The prompt's own share of the denominators at the edges of its blocks (16 rows, 16 keys, a
block per wave; one, two or four waves), against the oracle."""
import numpy as np
import pytest
import torch

import paper_2408_00167_amd as F
import workloads as W
from oracle import finch_oracle as O
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,group", [(torch.bfloat16, 128, 4), (torch.bfloat16, 64, 1), (torch.float32, 64, 3),
                                           (torch.float32, 128, 1)])
def test_prompt_lse_edges(dtype, d, group):
    fin = F.Finch(H.finch_dtype(torch.empty(0, dtype=dtype)), d, group)
    specs = [dict(n_que=n, c=0, m=1, r=1, prompt_keys=True, qscale=q)
             for n in (1, 15, 16, 17, 32, 33, 63, 64, 65, 130) for q in (1.0, 3.0)]
    batch, ts = H.single_step_case(fin, specs, dtype, d, group, seed=8)
    fin.prompt_lse(batch)
    torch.cuda.synchronize()
    for t in ts:
        got = t["lse_extra"].cpu().numpy()
        want = O.prompt_lse(W.to_numpy_storage(t["q"]), W.to_numpy_storage(t["k_que"]), group)
        # computed in fp64, rounded once to fp32
        assert np.all(np.abs(got[:-1] - want) <= 2.0 ** -24 * np.abs(want) + 1e-12), (t["n_que"], d)
        assert got[-1] == -77.0
    # (how many waves a workgroup has goes by the longest prompt: one problem at a time as well)
    want = [t["lse_extra"].clone() for t in ts]
    for t, w in zip(ts, want):
        t["lse_extra"][:-1].fill_(-55.0)
        fin.prompt_lse(F.Batch([dict(t, lse_extra=t["lse_extra"][:-1])]))
        torch.cuda.synchronize()
        assert torch.equal(t["lse_extra"], w), t["n_que"]
    fin.close()
