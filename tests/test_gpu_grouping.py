"""Per-node sums and smoothing of the update alone, for given BMUs, through every way the instances are grouped by node
(a workgroup per node, one workgroup's counting sort, the tiled one, maps whose counters leave room for one or two
wavefronts only, the radix sort where they leave none or the tiled form's table would be too large) and the one-launch smoothing of small maps, against the oracle: skewed, uniform and single-node
assignments, sizes at the edges of the tiles."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,rows,cols,dim,grid,map_type", [
    (1, 1, 1, 1, "square", "planar"), (63, 3, 5, 7, "hexagonal", "toroid"), (512, 20, 20, 10, "square", "planar"),
    (513, 1, 70, 33, "hexagonal", "planar"), (8192, 9, 7, 32, "hexagonal", "toroid"), (8193, 9, 7, 5, "square", "toroid"),
    (4097, 37, 29, 63, "hexagonal", "planar"), (3000, 12, 11, 300, "square", "toroid"),      # a workgroup per node
    (16384, 21, 19, 40, "square", "planar"), (16385, 21, 19, 40, "hexagonal", "toroid"),      # one workgroup, tiles
    (65536, 30, 30, 4, "square", "planar"), (131073, 50, 50, 3, "hexagonal", "toroid"),       # tiles of four, eight wavefronts ...
    (262145, 50, 51, 2, "square", "planar"), (524289, 50, 50, 2, "square", "toroid"),          # ... sixteen, and more keys for each
    (250000, 100, 100, 3, "square", "planar"), (300000, 200, 201, 2, "square", "planar"),      # tables at their finest and coarser
    (40001, 70, 70, 6, "square", "toroid"), (20000, 140, 150, 5, "hexagonal", "planar"),      # fewer counters per wavefront
    (9000, 230, 231, 3, "square", "planar"), (5000, 288, 282, 3, "square", "toroid"),          # one wavefront's counters (up to 81,408 nodes)
    (825000, 285, 285, 2, "square", "planar"), (850001, 285, 285, 2, "hexagonal", "toroid"),  # the largest table; radix sort beyond
    (5000, 289, 282, 3, "square", "planar"), (40000, 300, 301, 3, "hexagonal", "toroid"),     # no room for counters: radix sort
])
@pytest.mark.parametrize("spread", ["skewed", "uniform", "one"])
def test_update_for_given_bmus(oracle, n, rows, cols, dim, grid, map_type, spread):
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(6100 + n + dim)
    k = rows * cols
    X = rng.normal(0, 1, (n, dim)).astype(np.float32)
    W = rng.random((k, dim)).astype(np.float32)
    if spread == "uniform":
        b = rng.integers(0, k, n)
    elif spread == "skewed":
        b = np.minimum(rng.integers(0, k, n), rng.integers(0, k, n) // 7)
        b[rng.random(n) < 0.4] = k - 1
    else:
        b = np.full(n, k // 2)
    b = b.astype(np.int32)
    radius = max(1.0, min(rows, cols) / 4)
    S, C = oracle.accumulate_dense(X, b, k)
    new = []
    for _ in range(2):
        som = Som(rows, cols, dim, map_type, grid, codebook=torch.from_numpy(W))
        som.update(P.to_dev(X), P.to_dev(b), radius)
        new.append(som.codebook.cpu().numpy())
        som.close()
    assert np.array_equal(new[0], new[1])                    # the order of the additions is fixed
    nodes = None if k < 60000 else np.unique(np.concatenate([np.arange(0, k, 97), [k // 2, k - 1]]))
    P.check_codebook(oracle, S, C, W, new[0], rows, cols, P.MAP[map_type], P.GRID[grid], radius, nodes=nodes)


@pytest.mark.parametrize("rows,cols", [(288, 282), (289, 282)])
def test_search_order_beside_the_counters_limit(oracle, rows, cols):
    """The two-level search puts its instances in order with the same grouping: on either side of 81,408 nodes."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(6200 + rows)
    W = rng.random((rows * cols, 5)).astype(np.float32)
    X = rng.random((2500, 5)).astype(np.float32)
    som = Som(rows, cols, 5, codebook=torch.from_numpy(W), filter="two_level")
    b = som.bmus(P.to_dev(X)).cpu().numpy()
    assert som.two_level_stats()[1] > 0
    som.close()
    P.check_bmus_dense(oracle, X, W, b)
