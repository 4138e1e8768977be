"""The MoE fanout's 16-lane ranking where its 32-bit keys do not decide: weights
that differ only in the low bits of their codes, equal weights, more of the top
experts in one lane than a lane keeps (in both register layouts: four neighbours
and every 64th expert, or every 16th), negative weights and the extreme codes;
one row in four, so that a wave mixes such rows with ordinary ones.  Bit-exact
against the oracle."""
import numpy as np
import pytest

from workloads import router_weights

from test_gpu_moe import check

pytestmark = pytest.mark.gpu


def hard_rows(n, e, seed):
    rng = np.random.default_rng(seed)
    p = router_weights(n, e, seed=seed)
    for r in range(0, n, 4):
        kind = (r // 4) % 6
        if kind == 0:     # neighbours in rank one unit in the last place apart
            top = rng.choice(e, size=min(e, 9), replace=False)
            bits = np.float32(0.11).view(np.uint32) + rng.permutation(len(top)).astype(np.uint32)
            p[r, top] = bits.view(np.float32)
        elif kind == 1:   # equal weights
            p[r, rng.choice(e, size=min(e, 7), replace=False)] = 0.12
        elif kind == 2:   # the largest in one lane: 4 l .. 4 l + 3 and + 64 j
            lane = int(rng.integers(0, 16))
            own = [x for j in range(0, e, 64) for x in range(j + 4 * lane, j + 4 * lane + 4) if x < e]
            p[r, own] = rng.uniform(1.0, 2.0, len(own)).astype(np.float32)
        elif kind == 3:   # the largest in one lane: l + 16 j
            own = np.arange(int(rng.integers(0, min(16, e))), e, 16)
            p[r, own] = rng.uniform(1.0, 2.0, len(own)).astype(np.float32)
        elif kind == 4:   # all negative
            p[r] = -p[r]
        else:
            sp = np.array([np.inf, -np.inf, np.nan, -np.nan, 0.0, -0.0], dtype=np.float32)
            p[r, rng.choice(e, size=6, replace=False)] = sp
            p[r, e - 1] = np.uint32(0xFFFFFFFF).view(np.float32)
    return p


@pytest.mark.parametrize("e", [16, 32, 64, 70, 72, 128, 130, 160, 250, 256])
@pytest.mark.parametrize("top_k,min_k", [(6, 3), (8, 1)])
def test_hard_rows(e, top_k, min_k):
    check(hard_rows(1001, e, 40 + e), 0.85, top_k, min_k)
