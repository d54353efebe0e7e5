"""Collected lists compared sixteen at a time (as one matrix product over the union of their nodes) against the oracle:
maps full of near-copies and of exact copies, at the edges of the tiles and of the union's room, with instances that coincide
with nodes, short rows, and non-finite ones."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _search(W, X, rows, cols, filt):
    from paper_1305_1422_amd import Som
    som = Som(rows, cols, W.shape[1], codebook=torch.from_numpy(W), filter=filt)
    b = som.bmus(P.to_dev(X)).cpu().numpy()
    stats = som.stats()
    som.close()
    return b, stats


@pytest.mark.parametrize("n,rows,cols,dim,groups,filt", [
    (4097, 20, 30, 40, 30, "two_level"),       # unions of some 20 nodes, a last tile of one list
    (5000, 25, 30, 130, 3, "two_level"),       # 250 near-copies each: unions near their room
    (5000, 30, 30, 33, 2, "split_f16"),        # ... and lists beyond their own
    (4500, 20, 25, 3, 25, "split_f16"),        # rows of three features, lists in any order
    (6000, 16, 20, 17, 40, "split_f16"),
])
def test_near_copies(oracle, n, rows, cols, dim, groups, filt):
    rng = np.random.default_rng(8500 + n + dim)
    k = rows * cols
    base = rng.random((groups, dim)).astype(np.float32)
    W = base[np.arange(k) * groups // k].copy()
    W += (rng.integers(-2, 3, size=W.shape) * np.float32(2.0 ** -22)).astype(np.float32)
    W[k - 7] = W[3]                                              # exact copies: the lowest index wins
    X = (base[rng.integers(groups, size=n)] + rng.normal(0, 0.05, size=(n, dim))).astype(np.float32)
    X[::17] = W[rng.integers(0, k, X[::17].shape[0])]            # instances on nodes, next to nodes an ulp away
    X[-1] = W[k - 7]
    b, (refined, collected, rescanned) = _search(W, X, rows, cols, filt)
    assert collected >= 4096
    P.check_bmus_dense(oracle, X, W, b)
    assert b[-1] == np.nonzero((W == W[k - 7]).all(1))[0][0]


def test_non_finite_among_the_lists(oracle):
    """Instances and a node with infinities or NaN do not disturb the others of their tile."""
    rng = np.random.default_rng(8600)
    rows, cols, dim, n = 20, 30, 24, 5000
    k = rows * cols
    base = rng.random((20, dim)).astype(np.float32)
    W = base[np.arange(k) * 20 // k] + (rng.integers(-2, 3, size=(k, dim)) * np.float32(2.0 ** -22)).astype(np.float32)
    X = (base[rng.integers(20, size=n)] + rng.normal(0, 0.05, size=(n, dim))).astype(np.float32)
    good = np.ones(n, dtype=bool)
    good[7::501] = False
    clean, _ = _search(W, X, rows, cols, "split_f16")
    X[7::1002] = np.nan
    X[508::1002, 5] = np.inf
    b, stats = _search(W, X, rows, cols, "split_f16")
    assert np.array_equal(b[good], clean[good]) and np.all(b[~good] == 0)


@pytest.mark.parametrize("n,rows,cols,dim,groups,filt", [
    (5000, 30, 30, 33, 2, "two_level"),        # the shapes above in the order that the union takes them in
    (4500, 20, 25, 3, 25, "two_level"),
    (6000, 16, 20, 17, 40, "two_level"),
    (5000, 25, 30, 130, 3, "split_f16"),       # ... and a list at a time, in any order
    (4097, 20, 30, 40, 30, "fp32"),
])
def test_near_copies_in_and_out_of_order(oracle, n, rows, cols, dim, groups, filt):
    test_near_copies(oracle, n, rows, cols, dim, groups, filt)


@pytest.mark.parametrize("n,rows,cols,dim,groups", [
    (8191, 20, 30, 40, 30),        # one list too few for the union
    (8192, 20, 30, 40, 30),
    (8209, 25, 30, 130, 3),        # 250 near-copies each: unions near their room
    (9000, 30, 30, 33, 2),         # lists beyond their own room, all of them scanned
    (8300, 20, 30, 50, 60),        # tiles whose lists have little in common: left, a list at a time
    (8500, 40, 30, 7, 90),
    (8400, 20, 25, 3, 25),         # rows of three features
])
def test_near_copies_by_the_union(oracle, n, rows, cols, dim, groups):
    test_near_copies(oracle, n, rows, cols, dim, groups, "two_level")


@pytest.mark.parametrize("groups", [20, 60])
def test_non_finite_among_the_unions(oracle, groups):
    """The same in the order that the union takes them in, also where tiles are left to be compared list by list."""
    rng = np.random.default_rng(8650)
    rows, cols, dim, n = 20, 30, 24, 9000
    k = rows * cols
    base = rng.random((groups, dim)).astype(np.float32)
    W = base[np.arange(k) * groups // k] + (rng.integers(-2, 3, size=(k, dim)) * np.float32(2.0 ** -22)).astype(np.float32)
    X = (base[rng.integers(groups, size=n)] + rng.normal(0, 0.05, size=(n, dim))).astype(np.float32)
    good = np.ones(n, dtype=bool)
    good[7::501] = False
    X[7::1002] = np.nan
    X[508::1002, 5] = np.inf
    b, (refined, collected, rescanned) = _search(W, X, rows, cols, "two_level")
    assert collected >= 8192
    assert np.array_equal(b[good], oracle.bmu_dense(X[good], W)) and np.all(b[~good] == 0)
