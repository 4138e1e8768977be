"""W_b at the edges of its launch rules: every tile (picked by how the rows
fill the compute units), the K pipelines' lengths (fewer slices than
buffers, as many, more), the few-row kernel's row blocks and its boundary with the
tiles, and outputs whose rows are not a whole number of 16-byte chunks.  Against
the fp64 oracle, each element also held to 3e-4 sum |w z| (+ 2^-8 |y| for bf16
output); rows sampled where there are many, the first and last among them."""
import numpy as np
import pytest

from workloads import wb_inputs

from test_gpu_wb import check_wb, gpu_wb

pytestmark = pytest.mark.gpu


def tile(rows, d_out):
    """(height / 32, channels) of the tile the launch rule takes."""
    def rounds(mi, bn):
        return -(-(-(-rows // (32 * mi)) * -(-d_out // bn)) // 256)
    cost = {(mi, 256): rounds(mi, 256) * 3 * (mi + 3) for mi in range(8, 1, -1)}
    cost.update({(mi, 128): rounds(mi, 128) * (mi + 7) for mi in range(4, 0, -1)})
    return min(cost, key=cost.get)


# tile: rows, channels
TILES = {(1, 128): (250, 4090), (2, 128): (500, 4090), (3, 128): (767, 4090), (4, 128): (1021, 4090),
         (2, 256): (190, 21750), (3, 256): (1535, 4090), (4, 256): (2047, 4090), (5, 256): (2100, 4090),
         (6, 256): (3071, 4090), (7, 256): (3577, 4090), (8, 256): (4090, 4090)}


@pytest.mark.parametrize("mi,bn", sorted(TILES))
@pytest.mark.parametrize("d_in,out", [(64, "f32"), (320, "bf16"), (512, "bf16")])
def test_tiles(mi, bn, d_in, out):
    n, d_out = TILES[mi, bn]
    assert tile(n, d_out) == (mi, bn)
    z, w = wb_inputs(n, d_in, d_out, seed=300 + mi + bn, z_std=1.0, w_std=d_in ** -0.5)
    got = gpu_wb(z, w, out)
    assert np.isfinite(got).all()
    rows = np.unique(np.concatenate([[0, 15, 16, 31, min(32 * mi, n) - 1, min(32 * mi, n - 1), n - 1], np.arange(0, n, 97)]))
    check_wb(got[rows], z, w, out, rows=rows)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 32, 33, 48, 63, 64, 65])
@pytest.mark.parametrize("d_in,d_out,out", [(64, 16, "f32"), (448, 37, "bf16"), (2048, 130, "f32"), (4160, 19, "bf16")])
def test_few_rows(n, d_in, d_out, out):
    z, w = wb_inputs(n, d_in, d_out, seed=500 + n, z_std=1.0, w_std=d_in ** -0.5)
    check_wb(gpu_wb(z, w, out), z, w, out)


@pytest.mark.parametrize("d_in,d_out,out", [(64, 16, "f32"), (448, 37, "bf16"), (576, 1024, "f32"), (1600, 130, "f32"), (4160, 19, "bf16"),
                                            (128, 8192, "bf16"), (128, 8193, "f32")])
def test_a_row_does_not_depend_on_the_number_of_rows(d_in, d_out, out):
    """Every launch rule adds an element's products in the same order: the first rows
    of any request have the bits they have in a larger one."""
    import torch
    from paper_2609_07008_amd import mla
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d_in)
    z = torch.empty((2100, d_in), device="cuda").normal_(0, 1, generator=gen).bfloat16()
    w = torch.empty((d_out, d_in), device="cuda").normal_(0, d_in ** -0.5, generator=gen).bfloat16()
    dtype = torch.bfloat16 if out == "bf16" else torch.float32
    whole = torch.empty((2100, d_out), dtype=dtype, device="cuda")
    mla.shared_wb(z, w, whole)
    for n in (1, 7, 16, 17, 32, 33, 65, 300, 700, 1100):
        y = torch.full((n, d_out), float("nan"), dtype=dtype, device="cuda")
        mla.shared_wb(z[:n].contiguous(), w, y)
        assert torch.equal(y, whole[:n]), n
