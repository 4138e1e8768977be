"""The device plan at the edges of its forms: one launch up to 65,536 rows, 512
segments and 2048 item groups, separate launches above; the protected list searched
in LDS up to 8192 rows, in memory above, in both.  Against the host-plan calls on the
same inputs: merged head outputs, lse, the partial index with its segments and the
protected flags are bit-identical, and nothing past them is written.  A list that
either form has to reject leaves status MLA_ERR_ROWS, an empty index and no flags."""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MLA_ERR_ROWS = 5


def geom(H, G):
    return SimpleNamespace(n_heads=H, n_groups=G, d_latent=64, d_rope=16, d_model=128, n_proj_groups=1, softmax_scale=0.1,
                           rope_base=10000.0, value_rope=False)


def table(lens, seed):
    """Segments of these lengths in storage order, the documents at permuted request offsets."""
    lens = np.asarray(lens, dtype=np.int64)
    order = np.random.default_rng(seed).permutation(len(lens))
    req = np.zeros(len(lens), np.int64)
    req[order] = np.concatenate([[0], np.cumsum(lens[order])[:-1]])
    return np.stack([np.concatenate([[0], np.cumsum(lens)[:-1]]), lens, req], axis=1)


def even(n, s):
    return [n // s + (i < n % s) for i in range(s)]


# heads, groups, segment lengths, protected rows, split_keys (0: a partial per visible document)
CASES = {
    "rows_65536": (2, 1, even(65536, 512), 4000, 1 << 30),
    "rows_65537": (2, 1, even(65537, 512), 4000, 1 << 30),
    "rows_65536_long_list": (2, 1, even(65536, 7), 50001, 1 << 30),
    "rows_65537_long_list": (2, 1, even(65537, 7), 50001, 1 << 30),
    "rows_65536_all_protected": (2, 1, even(65536, 300), 65536, 1 << 30),
    "list_8192": (4, 2, even(16000, 40), 8192, 1 << 30),
    "list_8193": (4, 2, even(16000, 40), 8193, 1 << 30),
    "list_8193_partials": (4, 2, even(9000, 9), 8193, 0),
    "segments_512": (3, 1, even(2000, 512), 333, 1 << 30),
    "segments_513": (3, 1, even(2000, 513), 333, 1 << 30),
    "groups_2048": (2, 1, [20] * 63, 200, 40),      # 1024 chunks, Global and Local
    "groups_2112": (2, 1, [20] * 64, 200, 40),
    "groups_2016_no_local": (1, 1, [20] * 63, 200, 0),
    "groups_2080_no_local": (1, 1, [20] * 64, 200, 0),
    "none_protected": (4, 2, even(3000, 30), 0, 1 << 30),
}


def inputs(name):
    import torch
    H, G, lens, p, split = CASES[name]
    segs, n = table(lens, len(lens)), int(sum(lens))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + p)
    draw = lambda *s: torch.empty(s, device="cuda").normal_(0, 1, generator=gen).to(torch.bfloat16)  # noqa: E731
    prot = np.sort(np.random.default_rng(p).choice(n, p, replace=False)).astype(np.int32)
    q_loc = draw(max(p, 1), G, H // G - 1, 80) if H > G else None
    return geom(H, G), segs, n, prot, min(split, n), draw(n, 80), draw(n, G, 80), q_loc


def planned(g, segs, split, cap, prot, n_prot, kv, q_glob, q_loc):
    import torch
    from paper_2609_07008_amd import step
    ps = step.PlannedStep(g, segs, np.zeros(g.n_groups, np.int32), split, cap)
    for t in (ps.out_o, ps.out_lse, ps.part_ptr, ps.part_seg, ps.row_src):
        t.view(torch.uint8).fill_(0xFF)
    rows = torch.full((max(cap, 1),), -7, dtype=torch.int32, device="cuda")
    rows[:len(prot)] = torch.from_numpy(prot).cuda()
    ps.attend(rows, torch.tensor([n_prot], dtype=torch.int32, device="cuda"), kv, q_glob, q_loc)
    torch.cuda.synchronize()
    return ps


def untouched(t):
    import torch
    return bool((t.contiguous().view(torch.uint8) == 0xFF).all())


@pytest.mark.parametrize("name", sorted(CASES))
def test_plan_equals_host_plan(name):
    import torch
    from paper_2609_07008_amd import step
    g, segs, n, prot, split, kv, q_glob, q_loc = inputs(name)
    host = step.OnlineStep(g, segs, prot, np.zeros(g.n_groups, np.int32), split)
    host.attend(kv, q_glob, q_loc)
    host.merge()
    ps = planned(g, segs, split, min(n, len(prot) + 5), prot, len(prot), kv, q_glob, q_loc)
    assert int(ps.status.item()) == 0
    slots, parts = host.n_slots, host.n_parts
    assert torch.equal(ps.part_ptr[:slots + 1], host.part_ptr)
    assert torch.equal(ps.part_seg[:parts], host.part_seg)
    assert torch.equal(ps.row_src, host.row_src)
    assert torch.equal(ps.out_lse[:slots].view(torch.int32), host.out_lse.view(torch.int32))
    assert torch.equal(ps.out_o[:slots].view(torch.int16), host.out_o.view(torch.int16))
    for t, used in ((ps.part_ptr, slots + 1), (ps.part_seg, parts), (ps.out_lse, slots), (ps.out_o, slots)):
        assert untouched(t[used:])
    assert int(host.row_src.sum()) == len(prot)


@pytest.mark.parametrize("name", ["list_8192", "list_8193", "rows_65537_long_list", "segments_513"])
@pytest.mark.parametrize("fault", ["last_row_out_of_range", "equal_rows_at_the_end", "too_many"])
def test_rejected_lists(name, fault):
    g, segs, n, prot, split, kv, q_glob, q_loc = inputs(name)
    cap, count = len(prot), len(prot)
    if fault == "last_row_out_of_range":
        prot[-1] = n
    elif fault == "equal_rows_at_the_end":
        prot[-1] = prot[-2]
    else:
        count += 1
    ps = planned(g, segs, split, cap, prot, count, kv, q_glob, q_loc)
    assert int(ps.status.item()) == MLA_ERR_ROWS
    assert int(ps.part_ptr[0]) == 0 and not bool(ps.row_src.any())
    for t in (ps.out_o, ps.out_lse, ps.part_ptr[1:], ps.part_seg):
        assert untouched(t)
