"""Exact stage with nodes that are copies of one another to the bit, at the lengths where its lists are taken in groups: the lowest
index wins, whichever group a copy falls into (gpu tests, through the C ABI)."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("copies", [63, 64, 65, 128, 129, 150])
def test_copies_left_by_the_union(oracle, copies):
    """Two groups of nodes with so many copies each: the product over the union cannot tell copies apart, so all of them are left
    to the plain sums, from one wavefront's width of them to more than two."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8700 + copies)
    rows, cols, dim, n = 20, 25, 40, 8500
    k = rows * cols
    base = rng.random((2, dim)).astype(np.float32)
    W = (rng.random((k, dim)) + 3.0).astype(np.float32)          # the others: far from everything
    order = rng.permutation(k)
    of = np.full(k, -1)
    of[order[:copies]], of[order[copies:2 * copies]] = 0, 1
    W[of >= 0] = base[of[of >= 0]]
    near = order[2 * copies:2 * copies + 10]                     # ... and ten a little farther away than the copies
    W[near] = base[np.arange(10) % 2] * np.float32(1 + 2.0 ** -14)
    which = rng.integers(2, size=n)
    X = (base[which] * rng.uniform(0.8, 0.95, size=(n, 1))).astype(np.float32)
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level")
    b = som.bmus(P.to_dev(X)).cpu().numpy()
    refined, collected, rescanned = som.stats()
    som.close()
    assert collected >= 8192 and rescanned < n // 2
    lowest = np.array([np.nonzero(of == g)[0][0] for g in (0, 1)])
    assert np.array_equal(oracle.bmu_dense(X[:50], W), lowest[which[:50]])
    assert np.array_equal(b, lowest[which])


def _groups_of_pairs(rng, dim, longest):
    """Nodes in groups of 2 .. longest: two of a group, at every pair of places, are copies; the others are a little farther from
    what lies on the line from the origin to them.  Returns (nodes, row of every group's copies, lower index of the pair)."""
    nodes, rows, lowest = [], [], []
    for size in range(2, longest + 1):
        for p in range(size):
            for q in range(p + 1, size):
                base = rng.random(dim) + 0.05
                base = (8.0 * base / np.linalg.norm(base)).astype(np.float32)
                at = len(nodes)
                for t in range(size):
                    nodes.append(base if t in (p, q) else base * np.float32(1 + 2.0 ** -18))
                rows.append(base)
                lowest.append(at + p)
    return np.stack(nodes), np.stack(rows), np.array(lowest)


@pytest.mark.parametrize("filt", ["split_f16", "two_level", "fp32"])
def test_pairs_of_copies_in_short_lists_dense(oracle, filt):
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8800)
    W, rows, lowest = _groups_of_pairs(rng, 70, 9)
    X = np.concatenate([rows * np.float32(s) for s in (0.9, 0.95, 1.0)])
    som = Som(1, len(W), 70, codebook=torch.from_numpy(W), filter=filt)
    b = som.bmus(P.to_dev(X)).cpu().numpy()
    refined, collected, _ = som.stats()
    som.close()
    assert refined + collected >= len(X) // 2 and collected > 0
    assert np.array_equal(oracle.bmu_dense(X, W), np.tile(lowest, 3))
    assert np.array_equal(b, np.tile(lowest, 3))


@pytest.mark.parametrize("entries", [1, 63, 64, 65, 128, 129, 300])
def test_pairs_of_copies_in_short_lists_sparse(oracle, entries):
    """Rows on both sides of the 64 and 128 entries that a wavefront has on the way at a time."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8900 + entries)
    dim = 310
    W, rows, lowest = _groups_of_pairs(rng, dim, 8)
    n = len(rows)
    columns = [np.sort(rng.choice(dim, size=entries, replace=False)) for _ in range(n)]
    indptr = np.arange(n + 1, dtype=np.int64) * entries
    indices = np.concatenate(columns).astype(np.int32)
    values = np.concatenate([rows[j][columns[j]] for j in range(n)])
    values *= np.repeat([0.8 * 64.0 / np.square(rows[j][columns[j]]).sum() for j in range(n)], entries)      # x.w = 0.8 |w|^2
    values = values.astype(np.float32)
    csr = (indptr, indices, values)
    som = Som(1, len(W), dim, codebook=torch.from_numpy(W))
    b = som.bmus(P.csr_to_dev(csr)).cpu().numpy()
    refined, collected, _ = som.stats()
    som.close()
    want = oracle.bmu_csr(csr, dim, W)
    P.check_bmus_csr(oracle, csr, dim, W, b)
    first = np.array([np.nonzero((W == W[i]).all(1))[0][0] for i in b])
    assert np.array_equal(b, first)                              # never the higher of two copies
    if entries >= 63:                                            # long enough to point at its group, nearly always
        assert refined + collected >= n // 2 and collected > 0
        assert np.array_equal(b, want) and np.mean(want == lowest) > 0.9
