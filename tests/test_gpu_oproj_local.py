"""The o-proj's Local pass at each of its tiles (64, 128, 256 rows of 256 channels, 32
and 64 rows of 128: picked by how the protected rows fill the compute units, asserted
for each case) and around their edges, with more tiles than workgroups, projection
groups of 1024, 512, 448, 128 and 96 channels (whole, ragged and part column tiles),
dense and sliced, head widths of 64, 512 and 576, f32 and bf16 z, and a device count
below the capacity.  Reference: z_online of eq:offonline in float64 from the same bf16
values.  Bound per element: 3e-4 sum |o w| for the f32 accumulation, 2^-8 of the
partial sums for a bf16 z (it is rounded after each pass)."""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def geom(H, G, d_c, d_r, d_model, n_pg, rotary=False):
    return SimpleNamespace(n_heads=H, n_groups=G, d_latent=d_c, d_rope=d_r, d_model=d_model, n_proj_groups=n_pg,
                           softmax_scale=1.0, rope_base=10000.0, value_rope=rotary)


def tile(g, p):
    """(rows, channels, rounds over the 256 workgroups) of the tile the device rule takes for p protected rows."""
    cw = g.d_model // g.n_proj_groups
    rounds = {(bm, bn): -(-(-(-p // bm) * -(-cw // bn) * g.n_proj_groups) // 256) for bm, bn in WEIGHT}
    bm, bn = min(WEIGHT, key=lambda t: rounds[t] * WEIGHT[t])
    return bm, bn, rounds[bm, bn]


WEIGHT = {(256, 256): 33, (128, 256): 21, (64, 256): 15, (64, 128): 9, (32, 128): 8}   # cost of a round, in the rule's order

# geometry, rows, protected rows; the tile and its rounds over the workgroups
CASES = {
    "height32_one_row": (geom(64, 8, 512, 64, 4096, 8), 300, 1, (32, 128, 1)),
    "height32": (geom(64, 8, 512, 64, 4096, 8), 300, 255, (32, 128, 1)),
    "height64_narrow": (geom(64, 8, 512, 64, 4096, 8), 700, 511, (64, 128, 1)),
    "height64_narrow_edge": (geom(64, 8, 512, 64, 4096, 8), 700, 257, (64, 128, 1)),
    "height64": (geom(64, 8, 512, 64, 4096, 8), 1100, 1023, (64, 256, 1)),
    "height128": (geom(64, 8, 512, 64, 4096, 8), 2100, 1030, (128, 256, 1)),
    "height256": (geom(64, 8, 512, 64, 4096, 8), 2500, 2400, (256, 256, 1)),
    "ragged_columns": (geom(32, 4, 512, 64, 4 * 448, 4), 400, 333, (32, 128, 1)),
    "narrow_groups": (geom(12, 4, 64, 16, 4 * 96, 4), 500, 97, (32, 128, 1)),
    "dense": (geom(16, 2, 512, 64, 1024, 1), 260, 70, (32, 128, 1)),
    "rotary": (geom(16, 2, 512, 64, 512, 2, rotary=True), 200, 65, (32, 128, 1)),
    # more tiles than workgroups: a workgroup walks several
    "height128_three_rounds": (geom(64, 8, 512, 64, 4096, 8), 4300, 4203, (128, 256, 3)),
    "height64_narrow_two_rounds": (geom(8, 1, 64, 16, 128, 1), 17000, 16501, (64, 128, 2)),
    "height256_three_rounds": (geom(16, 4, 64, 16, 8 * 512, 4), 11000, 10800, (256, 256, 3)),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("z_dtype", ["float32", "bfloat16"])
def test_local_pass(name, z_dtype):
    import torch
    from paper_2609_07008_amd import mla
    g, n, p, shape = CASES[name]
    assert tile(g, p) == shape
    hpg, dv, cw = g.n_heads // g.n_groups, mla.head_width(g), g.d_model // g.n_proj_groups
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11 * n + p)
    draw = lambda shape, std: torch.empty(shape, device="cuda").normal_(0, std, generator=gen).to(torch.bfloat16)  # noqa: E731
    o_glob, o_loc = draw((n, g.n_groups, dv), 1.0), draw((n, g.n_groups, hpg - 1, dv), 1.0)
    w_o = draw((g.n_proj_groups, g.n_heads // g.n_proj_groups * dv, cw), 0.02)
    z_off = draw((n, g.d_model), 1.0)
    rng = np.random.default_rng(n)
    rows = np.sort(rng.choice(n, size=p, replace=False)).astype(np.int32)
    glob_head = rng.integers(0, hpg, size=g.n_groups).astype(np.int32)
    prot = torch.from_numpy(np.concatenate([rows, np.full(n - p, 2 ** 30, np.int32)])).cuda()
    count = torch.tensor([p], dtype=torch.int32, device="cuda")
    segs = [[0, n, 0]]
    plan = torch.empty((int(mla.plan_query(g, segs, n, n).plan_bytes),), dtype=torch.uint8, device="cuda")
    info = mla.online_plan(g, segs, n, n, plan)
    z = torch.full((n, g.d_model), float("nan"), dtype=getattr(torch, z_dtype), device="cuda")
    mla.sliced_oproj_add_planned(g, info, o_glob, o_loc, glob_head, prot, count, w_o, z_off, z)
    torch.cuda.synchronize()

    gpp = g.n_groups // g.n_proj_groups
    w = w_o.double().view(g.n_proj_groups, gpp, hpg, dv, cw)
    idx = torch.from_numpy(rows.astype(np.int64)).cuda()
    ref, mag, part = z_off.double(), torch.zeros((n, g.d_model), dtype=torch.float64, device="cuda"), None
    ref[idx] = 0.0
    part = torch.zeros_like(ref)   # the Global sums, which a bf16 z holds rounded between the passes
    for grp in range(g.n_groups):
        pg, gi, gh = grp // gpp, grp % gpp, int(glob_head[grp])
        cols = slice(pg * cw, (pg + 1) * cw)
        og, wg = o_glob[:, grp].double(), w[pg, gi, gh]
        part[:, cols] += og @ wg
        mag[:, cols] += og.abs() @ wg.abs()
        loc = [j for j in range(hpg) if j != gh]
        ol, wl = o_loc[:p, grp].reshape(p, -1).double(), w[pg, gi][loc].reshape(-1, cw)
        ref[idx, cols] += ol @ wl
        mag[idx, cols] += ol.abs() @ wl.abs()
    ref += part
    bound = 3e-4 * mag + 1e-6
    if z_dtype == "bfloat16":
        bound = bound + 2.0 ** -8 * (ref.abs() + part.abs())
    assert bool(((z.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("name", ["height64_narrow", "narrow_groups", "dense", "rotary"])
def test_no_artifact_when_every_row_is_protected(name):
    """z_off may be absent when P == N: the same bits as with an artifact, which is
    not read for a protected row."""
    import torch
    from paper_2609_07008_amd import mla
    g, n = CASES[name][:2]
    hpg, dv, cw = g.n_heads // g.n_groups, mla.head_width(g), g.d_model // g.n_proj_groups
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    draw = lambda shape, std: torch.empty(shape, device="cuda").normal_(0, std, generator=gen).to(torch.bfloat16)  # noqa: E731
    o_glob, o_loc = draw((n, g.n_groups, dv), 1.0), draw((n, g.n_groups, hpg - 1, dv), 1.0)
    w_o = draw((g.n_proj_groups, g.n_heads // g.n_proj_groups * dv, cw), 0.02)
    glob_head = np.zeros(g.n_groups, np.int32)
    rows = torch.arange(n, dtype=torch.int32, device="cuda")
    z = [torch.full((n, g.d_model), float("nan"), device="cuda") for _ in range(2)]
    mla.sliced_oproj_add(g, n, o_glob, o_loc, glob_head, rows, n, w_o, draw((n, g.d_model), 1.0), z[0])
    mla.sliced_oproj_add(g, n, o_glob, o_loc, glob_head, rows, n, w_o, None, z[1])
    torch.cuda.synchronize()
    assert bool(torch.isfinite(z[0]).all())
    assert torch.equal(z[0], z[1])
