"""The softmax reference of the 512 + 64 attention: a head-row's weights are taken
against its max over the item's first 64 keys (of its first document), so a key
there that outweighs the rest has weight exactly 1 and no bf16 rounding.  Such a
row's lse is then its score to f32 accuracy (64 * 2^-23 a step, a few steps); a
reference from fewer keys leaves the rounded weight's log, up to 2^-9."""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rotary", [False, True])
@pytest.mark.parametrize("split", [0, 10 ** 9])
@pytest.mark.parametrize("n,u", [(200, 0), (200, 15), (200, 16), (200, 31), (200, 32), (200, 47), (200, 63), (16, 15), (33, 32), (40, 35)])
def test_dominant_key_among_the_first_64(n, u, split, rotary):
    import torch
    from paper_2609_07008_amd import step
    g = SimpleNamespace(n_heads=8, n_groups=2, d_latent=512, d_rope=64, d_model=128, n_proj_groups=2, softmax_scale=1.0,
                        rope_base=10000.0, value_rope=rotary)
    lens = [n, 70, 9]
    N, starts = sum(lens), np.cumsum([0] + lens[:-1])
    segs = np.stack([starts, lens, starts], axis=1)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * n + u)

    def draw(*shape):
        x = torch.empty(shape, device="cuda").normal_(0, 0.05, generator=gen).to(torch.bfloat16)
        x[..., 512:] = 0     # no RoPE part: the relocation rounds nothing
        return x

    kv = draw(N, 576)
    kv[:, 0] = 0
    kv[u] = 0
    kv[u, 0] = 8.0
    prot = np.arange(0, N, 3, dtype=np.int32)
    q_glob, q_loc = draw(N, 2, 576), draw(len(prot), 2, 3, 576)
    for q in (q_glob, q_loc):   # scores of key u between 24 and 40
        q[..., 0] = torch.empty(q.shape[:-1], device="cuda").uniform_(3.0, 5.0, generator=gen).to(torch.bfloat16)
    st = step.OnlineStep(g, segs, prot, np.zeros(2, np.int32), min(split, N))
    st.attend(kv, q_glob, q_loc)
    st.merge()
    torch.cuda.synchronize()

    def lse(q, rows):   # [rows, heads, 576] in 64 bits, causal in storage order
        s = q.double() @ kv.double().t()
        s.masked_fill_(torch.arange(N, device="cuda")[None, None, :] > rows[:, None, None], -np.inf)
        return torch.logsumexp(s, dim=-1).reshape(-1)

    rows = torch.arange(N, device="cuda")
    loc = torch.from_numpy(prot.astype(np.int64)).cuda()
    ref = torch.cat([lse(q_glob, rows), lse(q_loc.reshape(len(prot), 6, 576), loc)])
    row = torch.cat([rows.repeat_interleave(2), loc.repeat_interleave(6)])
    err = (st.out_lse.double() - ref).abs()[row >= u]
    assert float(err.max()) < 1e-4
