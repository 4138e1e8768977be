"""Attention at the edges of its tiles (512+64 latent): documents that end on
either side of a 16- or 32-key boundary, work items of one to 128 head-rows
whose last 16- or 32-row block is partly filled, every key tile count from one
on, in both output forms (partials then merge, and the head output itself);
every row and head against the fp64 oracle."""
import numpy as np
import pytest

from workloads import make_custom

from parity import check_bookkeeping, compare_rows, run

pytestmark = pytest.mark.gpu

LENGTHS = [1, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 96, 97, 129]
PARTITIONS = [(8, 8), (16, 2), (21, 3), (5, 5), (9, 1)]   # head-rows per row: G Global, H - G Local


def case(n):
    i = LENGTHS.index(n)
    H, G = PARTITIONS[i % len(PARTITIONS)]
    return make_custom([n, LENGTHS[-1 - i], 1 + i], req_perm=[2, 0, 1], tq=1 + i % 3, H=H, G=G, d_c=512, d_r=64,
                       d_model=64 * G, prot_frac=0.3, seed=7000 + n, fp32=False,
                       std=dict(c=1.0, kr=1.0, qc=1.0, qr=1.0, wo=0.02, zoff=0.05))


@pytest.mark.parametrize("n", LENGTHS)
def test_partials(n):
    wl = case(n)
    st, _ = run(wl, 0)
    check_bookkeeping(wl, st, 0)
    compare_rows(wl, st, np.arange(wl.n_rows), wl.z_off())


@pytest.mark.parametrize("n", LENGTHS)
def test_direct_output_equals_one_partial(n):
    """The plan-once path with one chunk per slot writes the head outputs itself:
    the same bits as one partial per slot and the merge."""
    import torch
    from paper_2609_07008_amd import step
    wl = case(n)
    st, inputs = run(wl, wl.n_rows)
    compare_rows(wl, st, np.arange(wl.n_rows), wl.z_off())
    for dtype in (0, 1):
        ps = step.PlannedStep(wl.geom, wl.segs, wl.glob_head, wl.n_rows, wl.n_rows, out_dtype=dtype)
        prot = torch.from_numpy(np.ascontiguousarray(wl.prot_rows, dtype=np.int32)).cuda()
        count = torch.tensor([wl.n_prot], dtype=torch.int32, device="cuda")
        ps.out_o.fill_(float("nan"))
        ps.attend(prot, count, inputs["kv"], inputs["q_glob"], inputs["q_loc"])
        torch.cuda.synchronize()
        assert int(ps.status.item()) == 0
        n_slots = st.out_o.shape[0]
        assert torch.equal(ps.out_o[:n_slots].to(torch.bfloat16), st.out_o)
        assert torch.equal(ps.out_lse[:n_slots], st.out_lse)
        assert torch.isnan(ps.out_o[n_slots:]).all()
