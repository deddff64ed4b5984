"""Top-r where its histogram rounds can go wrong: sizes at the edges of the register
variants and of the LDS, and scores whose spread makes the rounds narrow slowly, at once, or
end in a bin of many, few or equal candidates.  The oracle's stable sort gives the answer
bit for bit."""
import numpy as np
import pytest
import torch

import paper_2408_00167_amd as F
from oracle import finch_oracle as O

pytestmark = pytest.mark.gpu


def _scores(kind, n, rng):
    if kind == "normal":
        return np.exp(0.1 * rng.standard_normal(n))
    if kind == "wide":        # every exponent a float has, both signs
        return rng.choice([-1.0, 1.0], n) * 2.0 ** rng.integers(-126, 127, n) * rng.uniform(1, 2, n)
    if kind == "neighbours":  # consecutive floats: the last round's bins hold one value each
        return np.arange(1065353216, 1065353216 + n, dtype=np.uint32).view(np.float32)[rng.permutation(n)]
    if kind == "far_groups":  # a crowd in one bin of the first round, few values far above
        s = 1.0 + 1e-4 * rng.random(n)
        s[:: max(1, n // 9)] = 1e30 * (1 + rng.random(len(s[:: max(1, n // 9)])))
        return s
    return rng.integers(0, 17, n) * 0.5   # "ties": more equal values than are resolved directly


@pytest.mark.parametrize("kind", ["normal", "wide", "neighbours", "far_groups", "ties"])
def test_topk_edges(kind):
    rng = np.random.default_rng(5)
    fin = F.Finch(F.FINCH_BF16, 128, 1)
    descs, keep = [], []
    for n in (2, 16, 17, 1023, 1025, 7168, 7169, 11264, 11265, 31744, 31745):
        s = _scores(kind, n, rng).astype(np.float32)
        for r in sorted({1, n // 3 + 1, n - 1}):
            st = torch.from_numpy(s).cuda()
            idx = torch.full((r + 1,), -9, dtype=torch.int32, device="cuda")
            descs.append(dict(scores=st, idx=idx[:r], n_que=1, c=0, m=n, r=r))
            keep.append((st, idx, O.top_r(s, r)))
    # (batches of one size as well: the launch's LDS is sized by the largest problem)
    fin.topk(F.Batch(descs))
    for d in descs[:6]:
        fin.topk(F.Batch([d]))
    torch.cuda.synchronize()
    for st, idx, want in keep:
        got = idx.cpu().numpy()
        assert np.array_equal(got[:-1], want), (kind, st.numel(), len(want))
        assert got[-1] == -9
    fin.close()
