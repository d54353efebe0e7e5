"""Per-node sums of sparse rows at the edges of their tiles and chunks (gpu tests, through the C ABI)."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim", [5, 1000, 13055, 13056, 13057, 26112, 26113, 40004])
@pytest.mark.parametrize("per_node", [2, 3])
def test_sums_at_the_edges_of_tiles_and_chunks(oracle, dim, per_node):
    """One tile of columns, its largest, one column more, several; rows of no, one, 64, 128, 129 and 300 entries; nodes with none, one,
    64 (a chunk), 65 and 130 instances; on both sides of the line where long rows leave the atomics.  The sums are exact: small whole
    numbers, so any order of the additions gives the same."""
    from paper_1305_1422_amd import Som
    rows, cols = 10, 12
    k, n = rows * cols, rows * cols * per_node - (per_node == 2)
    rng = np.random.default_rng(dim + per_node)
    bmus = np.full(n, 7, dtype=np.int32)
    bmus[:64], bmus[64:129], bmus[129:130] = 3, k - 1, 11
    if per_node == 3:
        bmus[130:260] = 0
    rng.shuffle(bmus)
    lengths = np.minimum(rng.choice([0, 1, 64, 65, 128, 129, 300], size=n), dim)
    indptr = np.zeros(n + 1, dtype=np.int64)
    indptr[1:] = np.cumsum(lengths)
    indices = np.concatenate([np.sort(rng.choice(dim, size=m, replace=False)) for m in lengths]).astype(np.int32)
    values = rng.integers(1, 9, size=indptr[-1]).astype(np.float32)
    W = rng.random((k, dim)).astype(np.float32)
    som = Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W))
    som.set_neighborhood("bubble")                       # radius below 1: every node is the mean of its own instances
    som.update(P.csr_to_dev((indptr, indices, values)), P.to_dev(bmus), 0.5)
    torch.cuda.synchronize()
    S, C = np.zeros((k, dim)), np.bincount(bmus, minlength=k)
    np.add.at(S, (np.repeat(bmus, lengths), indices), values)
    want = np.where(C[:, None] > 0, S / np.maximum(C, 1)[:, None], W)
    got = som.codebook.cpu().numpy()
    assert np.abs(got - want).max() <= 2.0 ** -22 * np.abs(want).max()      # one division, its operands exact: an ulp or two
    som.close()


@pytest.mark.parametrize("dim", [26113, 104448, 417792, 417793])
@pytest.mark.parametrize("n", [12, 200])
def test_sums_of_long_rows_and_many_tiles(dim, n):
    """Three, eight and 32 tiles of columns shared out to several workgroups, and the first row length that goes by atomics; rows at the
    edges of what a lane keeps (128 entries) and of the pieces of 256 beyond it, one of thousands among short ones; nodes of one chunk and of
    several.  Small whole numbers: any order of the additions gives the same."""
    from paper_1305_1422_amd import Som
    k = 6
    rng = np.random.default_rng(dim + n)
    bmus = rng.integers(0, k - 1, size=n).astype(np.int32)      # (the last node has none)
    bmus[n // 3:] = 2
    lengths = rng.choice([0, 1, 127, 128, 129, 384, 385, 2176, 2177, 6000], size=n)
    indptr = np.zeros(n + 1, dtype=np.int64)
    indptr[1:] = np.cumsum(lengths)
    indices = np.concatenate([np.sort(rng.choice(dim, size=m, replace=False)) for m in lengths]).astype(np.int32)
    if lengths[-1]:
        indices[-1] = dim - 1                            # the last column of the last tile
    values = rng.integers(1, 9, size=indptr[-1]).astype(np.float32)
    W = rng.random((k, dim)).astype(np.float32)
    som = Som(2, 3, dim, "planar", "square", codebook=torch.from_numpy(W))
    som.set_neighborhood("bubble")
    csr = P.csr_to_dev((indptr, indices, values))
    som.update(csr, P.to_dev(bmus), 0.5)
    torch.cuda.synchronize()
    S, C = np.zeros((k, dim)), np.bincount(bmus, minlength=k)
    np.add.at(S, (np.repeat(bmus, lengths), indices), values)
    want = np.where(C[:, None] > 0, S / np.maximum(C, 1)[:, None], W)
    assert np.abs(som.codebook.cpu().numpy() - want).max() <= 2.0 ** -22 * np.abs(want).max()      # as above
    som.close()


def _check_sums(rows, cols, dim, bmus, lengths, rng):
    """Bubble below radius 1: every node the mean of its own instances, whose entries are small whole numbers (any order adds up the same)."""
    from paper_1305_1422_amd import Som
    k, n = rows * cols, len(bmus)
    indptr = np.zeros(n + 1, dtype=np.int64)
    indptr[1:] = np.cumsum(lengths)
    first = rng.integers(0, dim, size=n)
    step = np.arange(indptr[-1]) - np.repeat(indptr[:-1], lengths)
    column = (np.repeat(first, lengths) + step) % dim    # consecutive columns, wrapped: put in order row by row
    row = np.repeat(np.arange(n), lengths)
    indices = column[np.lexsort((column, row))].astype(np.int32)
    values = rng.integers(1, 9, size=indptr[-1]).astype(np.float32)
    W = rng.random((k, dim)).astype(np.float32)
    som = Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W))
    som.set_neighborhood("bubble")
    som.update(P.csr_to_dev((indptr, indices, values)), P.to_dev(bmus.astype(np.int32)), 0.5)
    torch.cuda.synchronize()
    C = np.bincount(bmus, minlength=k)
    S = np.bincount(bmus[row].astype(np.int64) * dim + indices, weights=values, minlength=k * dim).reshape(k, dim)
    want = np.where(C[:, None] > 0, S / np.maximum(C, 1)[:, None], W)
    assert np.abs(som.codebook.cpu().numpy() - want).max() <= 2.0 ** -22 * np.abs(want).max()      # one division, as above
    som.close()


@pytest.mark.parametrize("dim,more", [(7, 0), (500, 0), (500, 1), (501, 0), (13056, 0), (13056, 1), (13053, 0)])
@pytest.mark.parametrize("rows,cols", [(10, 12), (16, 17)])
def test_sums_of_nodes_with_few_entries(rows, cols, dim, more):
    """Both sides of 768 entries per node (rows of seven columns never reach it), on maps of fewer nodes than the chip has CUs and of more: nodes of
    0, 1, 15, 16, 17, 63, 64, 65 and 130 instances."""
    rng = np.random.default_rng(dim + more)
    k = rows * cols
    sizes = np.array([0, 1, 15, 16, 17, 63, 64, 65, 130, 0] + [2] * (k - 10))
    bmus = np.repeat(np.arange(k), sizes)
    rng.shuffle(bmus)
    n, nnz = len(bmus), 768 * k - 1 + more
    lengths = np.minimum(np.full(n, nnz // n), dim)
    if lengths[0] < dim:
        lengths[:nnz - lengths.sum()] += 1
        assert lengths.sum() == nnz
    _check_sums(rows, cols, dim, bmus, lengths, rng)


@pytest.mark.parametrize("dim", [30, 31, 6528, 6529])
@pytest.mark.parametrize("n", [48 * 256 - 1, 48 * 256, 100 * 256, 100 * 256 + 1])
def test_sums_of_about_a_hundred_instances_a_node(dim, n):
    """Chunks of 128 rows in two copies of the row, and the sizes on both sides of them: a node of none, of 1, 31 .. 33, 63 .. 65, 127 .. 129, 256 and 257
    instances, the others share the rest."""
    rng = np.random.default_rng(dim + n)
    sizes = np.zeros(256, dtype=np.int64)
    sizes[:14] = [0, 1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 256, 257, 8]
    sizes[14:] = (n - sizes.sum()) // 242
    sizes[255] += n - sizes.sum()
    bmus = np.repeat(np.arange(256), sizes)
    rng.shuffle(bmus)
    _check_sums(16, 16, dim, bmus, rng.choice([20, 25, 30], size=n), rng)
