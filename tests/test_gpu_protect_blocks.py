"""Protected token-row set at the edges of its blocks: row counts around the 4 and
the 4096 rows that a thread and a block classify, around the 1024 count blocks of
2048 rows from which the offsets come from a launch of their own, and scores and
flags that start off the vector loads' alignment.  Whole numbers, compared exactly."""
import numpy as np
import pytest

from oracle import mla_oracle as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [3, 4, 2049, 4095, 4097, 1024 * 2048, 1024 * 2048 + 1])
def test_protect_blocks(n, shift):
    import torch
    from paper_2609_07008_amd import mla
    rng = np.random.default_rng(n)
    n_segs = min(n, 7)
    cut = np.sort(rng.choice(np.arange(1, n), size=n_segs - 1, replace=False)) if n_segs > 1 else np.zeros(0, int)
    starts = np.concatenate(([0], cut))
    lens = np.diff(np.concatenate((starts, [n])))
    order = rng.permutation(n_segs)                      # order[k]: the segment at place k of the request
    req = np.zeros(n_segs, dtype=np.int64)
    req[order] = np.concatenate(([0], np.cumsum(lens[order])[:-1]))
    segs = np.stack([starts, lens, req], axis=1).astype(np.int64)
    q = int(order[-1])
    flags = rng.choice(np.array([0, 1, 2, 3], np.uint8), size=n, p=[.94, .02, .03, .01])
    scores = rng.standard_normal(n).astype(np.float32)
    scores[rng.integers(0, n, size=n // 3)] = 0.5         # ties across blocks
    ws = torch.empty(mla.protected_rows_query(segs), dtype=torch.uint8, device="cuda")
    d_sc = torch.zeros(n + 1, dtype=torch.float32, device="cuda")[shift:shift + n]
    d_fl = torch.zeros(n + 1, dtype=torch.uint8, device="cuda")[shift:shift + n]
    d_sc.copy_(torch.from_numpy(scores))
    d_fl.copy_(torch.from_numpy(flags))
    out = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for budget in (0.15, 0.6):
        print(n, shift, budget, flush=True)
        out.fill_(-1)
        mla.protected_rows(segs, q, 2, n // 50, budget, d_fl, d_sc, out, cnt, ws)
        torch.cuda.synchronize()
        want = M.protected_rows(segs, q, flags, scores, 2, n // 50, budget)
        k = int(cnt.item())
        got = out.cpu().numpy()
        assert k == want.size and np.array_equal(got[:k], want) and np.all(got[k:] == -1)
