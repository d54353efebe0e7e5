"""Epochs whose neighbourhood tables are written by the launch that adds up the nodes' instances (few instances on few
nodes: no launch of their own): every epoch of a schedule against the oracle, for each kind of table, and single epochs
with changing radii and given choices on the same context."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("name,compact,function", [("gaussian", False, 0), ("gaussian", True, 0), ("bubble", False, 1)])
@pytest.mark.parametrize("rows,cols,dim,n,map_type,grid_type", [
    (1, 1, 3, 5, "planar", "square"),               # one node, one workgroup of tables
    (12, 19, 10, 600, "toroid", "hexagonal"),       # the two factor tables alone
    (70, 40, 12, 900, "planar", "hexagonal"),       # coefficient matrices (or a wide weight table): many workgroups
    (64, 33, 300, 40, "toroid", "square"),          # two column blocks of sums: the tables once
])
def test_every_epoch_of_a_schedule(oracle, rows, cols, dim, n, map_type, grid_type, name, compact, function):
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(rows * cols + n)
    k = rows * cols
    X = rng.random((n, dim), dtype=np.float32)
    W = rng.random((k, dim), dtype=np.float32)
    som = Som(rows, cols, dim, map_type, grid_type, codebook=torch.from_numpy(W))
    som.set_neighborhood(name, compact)
    Xd = P.to_dev(X)
    bmus, _, books, chosen = som.train_snapshots(Xd, 4, snapshots=2, radius0=4.0, radiusN=1.0)
    torch.cuda.synchronize()
    books, chosen = books.cpu().numpy(), chosen.cpu().numpy()
    before = W
    for e in range(4):
        radius = oracle.cool(4.0, 1.0, 4, e, oracle.LINEAR)
        P.check_bmus_dense(oracle, X, before, chosen[e])
        S, C = oracle.accumulate_dense(X, chosen[e], k)
        P.check_codebook(oracle, S, C, before, books[e], rows, cols, P.MAP[map_type], P.GRID[grid_type], radius,
                         function=function, compact=compact)
        before = books[e]
    S, C = oracle.accumulate_dense(X, chosen[3], k)
    for radius in (2.0, 5.0):
        W_in = som.codebook.cpu().numpy().copy()
        som.update(Xd, bmus, radius)
        torch.cuda.synchronize()
        P.check_codebook(oracle, S, C, W_in, som.codebook.cpu().numpy(), rows, cols, P.MAP[map_type], P.GRID[grid_type], radius,
                         function=function, compact=compact)
    som.close()
