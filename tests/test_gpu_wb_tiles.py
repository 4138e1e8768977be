"""W_b at the edges of its launch rules: every tile height (picked by how the
rows fill the compute units), the K pipelines' lengths (fewer slices than
buffers, as many, more), the few-row kernel's row blocks and its boundary with the
tiles, and outputs whose rows are not a whole number of 16-byte chunks.  Against
the fp64 oracle, each element also held to 3e-4 sum |w z| (+ 2^-8 |y| for bf16
output); rows sampled where there are many, the first and last among them."""
import numpy as np
import pytest

from workloads import wb_inputs

from test_gpu_wb import check_wb, gpu_wb

pytestmark = pytest.mark.gpu


def tile_height(rows, d_out):
    n_tiles = -(-d_out // 256)
    cost = {mi: -(-(-(-rows // (32 * mi)) * n_tiles) // 256) * (mi + 3) for mi in range(8, 0, -1)}
    return min(cost, key=cost.get)


HEIGHTS = {1: 500, 2: 1021, 3: 1535, 4: 2047, 5: 2100, 6: 3071, 7: 3577, 8: 4090}


@pytest.mark.parametrize("mi", sorted(HEIGHTS))
@pytest.mark.parametrize("d_in,out", [(64, "f32"), (320, "bf16")])
def test_tile_heights(mi, d_in, out):
    n, d_out = HEIGHTS[mi], 4090
    assert tile_height(n, d_out) == mi
    z, w = wb_inputs(n, d_in, d_out, seed=300 + mi, z_std=1.0, w_std=d_in ** -0.5)
    got = gpu_wb(z, w, out)
    assert np.isfinite(got).all()
    rows = np.unique(np.concatenate([[0, 15, 16, 31, 32 * mi - 1, 32 * mi, n - 1], np.arange(0, n, 97)]))
    check_wb(got[rows], z, w, out, rows=rows)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 32, 33, 48, 63, 64, 65])
@pytest.mark.parametrize("d_in,d_out,out", [(64, 16, "f32"), (448, 37, "bf16"), (2048, 130, "f32"), (4160, 19, "bf16")])
def test_few_rows(n, d_in, d_out, out):
    z, w = wb_inputs(n, d_in, d_out, seed=500 + n, z_std=1.0, w_std=d_in ** -0.5)
    check_wb(gpu_wb(z, w, out), z, w, out)
