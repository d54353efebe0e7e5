"""The forms of the U-matrix kernel against the oracle, on both sides of the lines between them (gpu tests, through the C ABI)."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("map_type,grid", [("planar", "square"), ("toroid", "hexagonal")])
@pytest.mark.parametrize("rows,cols,dim", [
    (5, 7, 1), (5, 7, 3), (6, 4, 384), (6, 4, 385),        # rows one feature a lane, and sixteen bytes a lane
    (3, 5, 767), (3, 5, 4095), (3, 5, 4096), (3, 5, 4099),  # ... and a node by four wavefronts
    (32, 32, 4097), (25, 41, 4098),                         # ... up to 1,024 nodes
    (80, 77, 5), (72, 85, 6),                              # one neighbour at a time from there on
    (64, 64, 128), (64, 65, 128), (64, 65, 129), (96, 64, 129), (96, 65, 129),      # ... with rows of up to 128, and of more
    (1, 1, 4100), (1, 2, 400), (2, 2, 4100), (3, 3, 390),   # few or aliased neighbours
])
def test_forms(oracle, map_type, grid, rows, cols, dim):
    from paper_1305_1422_amd import Som
    if grid == "hexagonal" and map_type == "toroid" and rows % 2:
        map_type = "planar"
    W = np.random.default_rng(rows * cols + dim).standard_normal((rows * cols, dim)).astype(np.float32)
    som = Som(rows, cols, dim, map_type, grid, codebook=torch.from_numpy(W))
    got = som.umatrix().cpu().numpy().reshape(-1)
    want = np.asarray(oracle.umatrix(W, rows, cols, P.MAP[map_type], P.GRID[grid])).reshape(-1)
    # fp64 sums in another order, then one rounding to fp32
    assert np.abs(got - want).max() <= 2.0 ** -23 * max(1.0, np.abs(want).max())
    som.close()
