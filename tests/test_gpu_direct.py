"""The small-problem search in double precision (the default filter below its size limit) against the oracle:
every way it shares out the work, rows that end inside a step of 16 features, copies of nodes (ties go to the lowest
index, more of them than a list holds), coincident instances, non-finite input, a bubble's masked copies."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _bmus(W, X, rows, cols, **kw):
    from paper_1305_1422_amd import Som
    som = Som(rows, cols, W.shape[1], codebook=torch.from_numpy(W), filter="auto")
    if kw.get("bubble"):
        som.set_neighborhood("bubble")
    b = som.bmus(P.to_dev(X)).cpu().numpy()
    assert som.stats() == (0, 0, 0) and som.two_level_stats() == (0, 0)      # no filter pass, no exact stage
    som.close()
    return b


@pytest.mark.parametrize("n,rows,cols,dim", [
    (1, 1, 1, 1), (5, 1, 3, 2), (17, 4, 4, 3), (16, 4, 4, 4), (15, 5, 13, 5),       # rows shorter than a load
    (40, 9, 9, 15), (300, 20, 20, 16), (1000, 20, 20, 17), (700, 33, 31, 33), (65, 20, 13, 64),
    (4097, 37, 29, 49), (900, 17, 8, 65), (33, 40, 40, 130),                        # the nodes over the wavefronts / groups
    (7, 50, 50, 511), (64, 30, 30, 513), (3, 40, 50, 1000),                         # the features over the wavefronts
    (512, 40, 50, 520), (513, 40, 50, 520), (1537, 30, 40, 100), (4200, 40, 25, 100), (8200, 100, 25, 20),   # 1 .. 16 instances merged by a workgroup
    (11000, 20, 20, 64), (12001, 31, 31, 33),                                       # ... in tiles of 64 nodes
    (64, 5, 8, 700), (8000, 5, 8, 200), (20000, 10, 10, 64),                        # one group of nodes: no merge
    (3, 250, 250, 3), (9, 70, 300, 2),                                              # groups, rows shorter than a load
    (70000, 3, 7, 6), (66001, 10, 12, 18), (66000, 4, 4, 9), (66000, 6, 10, 80),    # a wavefront per 16 instances
])
def test_matches_the_oracle(oracle, n, rows, cols, dim):
    rng = np.random.default_rng(5100 + n + dim)
    k = rows * cols
    W = (rng.random((k, dim)) - 0.3).astype(np.float32)
    X = rng.random((n, dim)).astype(np.float32)
    if k > 8:
        W[k - 1] = W[k // 3] = W[1]                       # copies: the lowest index wins
        X[0] = W[k - 1]
        W[k // 2] = W[2]
        W[k // 2, 0] = np.nextafter(W[2, 0], np.float32(9))      # one rounding away from node 2
        X[n // 2] = W[k // 2]
    m = min(n, 3000)
    b = _bmus(W, X, rows, cols)
    P.check_bmus_dense(oracle, X[:m], W, b[:m])
    P.check_bmus_dense(oracle, X[n - m:], W, b[n - m:])
    if k > 8 and n > 1:
        assert b[0] == 1 and b[n // 2] == k // 2


@pytest.mark.parametrize("n,dim,bubble", [(50, 40, False), (50, 600, False), (70000, 4, False), (50, 40, True), (1200, 200, False),
                                          (1200, 200, True), (3000, 13, False), (800, 1000, False)])
def test_more_copies_than_a_list_holds(oracle, n, dim, bubble):
    rng = np.random.default_rng(5200 + dim)
    rows, cols = 20, 15
    W = (rng.random((rows * cols, dim)) + 3.0).astype(np.float32)
    W[37:237] = rng.random((1, dim)).astype(np.float32)
    X = rng.random((n, dim)).astype(np.float32)
    assert np.all(_bmus(W, X, rows, cols, bubble=bubble) == 37)


def test_non_finite_rows():
    rng = np.random.default_rng(5300)
    for n, rows, cols, dim in ((40, 12, 12, 20), (20, 40, 40, 700), (66000, 4, 5, 5)):
        W = rng.random((rows * cols, dim)).astype(np.float32)
        X = rng.random((n, dim)).astype(np.float32)
        want = _bmus(W, X, rows, cols)
        hit = int(np.bincount(want).argmax())
        X[3, 1], X[5, 0], X[6, 2] = np.nan, np.inf, -np.inf
        b = _bmus(W, X, rows, cols)
        keep = np.setdiff1d(np.arange(n), [3, 5, 6])
        assert np.all(b[[3, 5, 6]] == 0) and np.array_equal(b[keep], want[keep])      # no finite distance: node 0
        W[hit, 0] = np.nan
        W[(hit + 1) % len(W), 2] = np.inf
        b = _bmus(W, X, rows, cols)
        assert np.all(b[[3, 5, 6]] == 0) and not np.isin(b[keep], [hit, (hit + 1) % len(W)]).any()
        same = keep[~np.isin(want[keep], [hit, (hit + 1) % len(W)])]
        assert np.array_equal(b[same], want[same])


@pytest.mark.parametrize("filt", ["auto", "split_f16", "two_level", "fp32"])
@pytest.mark.parametrize("n,rows,cols,dim", [(40, 12, 12, 20), (66000, 4, 5, 5), (20, 40, 40, 700), (64, 5, 8, 700)])
def test_no_finite_distance_gives_node_0(oracle, filt, n, rows, cols, dim):
    """An instance with an infinite component is at no finite distance of any node, whatever node 0 holds: a NaN or an
    infinity of its own makes its distance a NaN while the others are at +inf.  The answer is node 0 all the same, by
    every filter and by the direct search in one kernel (wavefronts that share the nodes or own an instance tile), with
    shared features, and merged from groups."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(5400 + n)
    X = rng.random((n, dim)).astype(np.float32)
    X[3, 1], X[5, 0], X[6, 2] = np.inf, -np.inf, np.nan
    for bad in (np.nan, np.inf):
        W = rng.random((rows * cols, dim)).astype(np.float32)
        W[0, :3] = bad
        som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter=filt)
        b = som.bmus(P.to_dev(X)).cpu().numpy()
        som.close()
        m = min(n, 500)
        assert np.array_equal(b[[3, 5, 6]], oracle.bmu_dense(X[[3, 5, 6]], W))
        assert np.all(b[[3, 5, 6]] == 0)
        keep = np.setdiff1d(np.arange(m), [3, 5, 6])
        P.check_bmus_dense(oracle, X[keep], W, b[keep])
