"""The sparse search on the coordinates of a smooth code book against the oracle: whole epochs on planar maps, at ragged sizes,
with empty and long rows, where the coordinates do and where they do not carry the code book, recorded into a graph, and what
goes past it."""
import numpy as np
import pytest

from gen import sparse_zipf_csr
from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _always(som):
    """These sets are far below those that try the coordinates by themselves."""
    from paper_1305_1422_amd import capi
    capi.som_debug_subspace_always(som.ctx, True)
    return som


def _smooth_book(rng, rows, cols, dim, radius, csr):
    """What a batch update of that radius leaves: Gaussian means of rows placed at random nodes."""
    indptr, indices, values = csr
    n = indptr.size - 1
    at = rng.integers(0, rows * cols, n)
    S = np.zeros((rows * cols, dim))
    np.add.at(S, (np.repeat(at, np.diff(indptr)), indices), values)
    C = np.bincount(at, minlength=rows * cols).astype(np.float64)
    y, x = np.divmod(np.arange(rows * cols), cols)
    H = np.exp(-((y[:, None] - y) ** 2 + (x[:, None] - x) ** 2) / (2.0 * radius * radius))
    return ((H @ S) / (H @ C)[:, None]).astype(np.float32)


def _edge_rows(csr, dim):
    """The same set with an empty row, a row of one nonzero, and one of a thousand."""
    indptr, indices, values = csr
    n = indptr.size - 1
    rows = [(indices[indptr[j]:indptr[j + 1]], values[indptr[j]:indptr[j + 1]]) for j in range(n)]
    rows[3] = (np.zeros(0, np.int32), np.zeros(0, np.float32))
    rows[5] = (np.array([dim - 1], np.int32), np.array([0.7], np.float32))
    rows[n - 1] = (np.arange(5, 1005, dtype=np.int32), np.linspace(-0.1, 0.1, 1000).astype(np.float32))
    ptr = np.zeros(n + 1, np.int64)
    ptr[1:] = np.cumsum([r[0].size for r in rows])
    return ptr, np.concatenate([r[0] for r in rows]).astype(np.int32), np.concatenate([r[1] for r in rows]).astype(np.float32)


@pytest.mark.parametrize("rows,cols,dim,n,radius", [(30, 32, 1500, 700, 9.0), (17, 61, 2051, 333, 14.0), (40, 40, 4096, 129, 11.0), (9, 9, 1027, 65, 4.0)])
@pytest.mark.parametrize("registered", [False, True])
def test_epochs_on_the_coordinates(oracle, rows, cols, dim, n, radius, registered):
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(8800 + dim)
    csr = _edge_rows(sparse_zipf_csr(n, dim, 88, mean_len=40.0, max_len=200), dim)
    W = _smooth_book(rng, rows, cols, dim, radius, csr)
    som = _always(Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W), filter="two_level"))
    som.set_sparse_dense_filter(False)         # (short rows of a registered set would go through its planes)
    dev = P.csr_to_dev(csr)
    if registered:
        capi.som_set_data_csr(som.ctx, *dev)
    for _ in range(2):
        mism = P.epoch_parity_csr(oracle, som, csr, dev, dim, radius, P.MAP["planar"], P.GRID["square"])
        assert som.two_level_stats()[0] > 0, "the coordinates were not used"
        assert mism == 0
    P.epoch_parity_csr(oracle, som, csr, dev, dim, 1.5, P.MAP["planar"], P.GRID["square"])       # narrow: not tried
    assert som.two_level_stats() == (0, 0)
    som.close()


def _dense(csr, dim):
    indptr, indices, values = csr
    X = np.zeros((indptr.size - 1, dim))
    X[np.repeat(np.arange(indptr.size - 1), np.diff(indptr)), indices] = values
    return X


@pytest.mark.parametrize("rows,cols,dim,n,radius", [(30, 32, 1500, 300, 9.0), (17, 61, 2051, 333, 14.0), (9, 9, 1027, 65, 4.0),
                                                    (16, 16, 40000, 40, 5.0)])
@pytest.mark.parametrize("data", ["near", "sizes", "rest"])
def test_scores_within_the_margins(rows, cols, dim, n, radius, data):
    """Block minima of the coarse and every score of the fine pass against fp64; among the rows an empty one, one of a thousand
    nonzeros and one that is full.  "rest": nodes that lie outside by a share of what may be left, and by several
    times that once the basis has been disturbed by it."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(8850 + dim)
    k = rows * cols
    csr = _edge_rows(sparse_zipf_csr(n, dim, 88, mean_len=40.0, max_len=200), dim)
    W = _smooth_book(rng, rows, cols, dim, radius, csr)
    indptr, indices, values = csr
    full = rng.standard_normal(dim).astype(np.float32) / np.float32(np.sqrt(dim))
    indptr = np.append(indptr, indptr[-1] + dim)
    indices, values = np.concatenate([indices, np.arange(dim, dtype=np.int32)]), np.concatenate([values, full])
    n += 1
    if data == "rest":
        e = rng.standard_normal((k, dim))
        W = (W + e * (2.0 ** -21 * np.linalg.norm(W - W.mean(0), axis=1).max() / np.linalg.norm(e, axis=1))[:, None]).astype(np.float32)
    if data == "sizes":
        values = values * np.repeat(np.exp2(rng.integers(-18, 18, n)), np.diff(indptr)).astype(np.float32)
    som = Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W), filter="two_level")
    dev = P.csr_to_dev((indptr, indices, values))
    m = torch.empty(((k + 127) // 128, n), dtype=torch.float32, device="cuda")
    scores = torch.empty((n, k), dtype=torch.float32, device="cuda")
    select, margin = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2))
    node_of = torch.empty(k, dtype=torch.int32, device="cuda")
    mu = torch.empty(dim, dtype=torch.float32, device="cuda")
    used = torch.empty(2, dtype=torch.int32, device="cuda")
    capi.som_debug_subspace_csr(som.ctx, *dev, som.codebook, m, select, node_of, scores, margin, mu, used)
    m, scores, select, margin, node_of, mu, used = (t.cpu().numpy() for t in (m, scores, select, margin, node_of, mu, used))
    som.close()
    assert used[0] > 0 and used[1] == 1
    X = _dense((indptr, indices, values), dim)
    wc = (W - mu).astype(np.float32).astype(np.float64)
    c = (wc ** 2).sum(1) + 2.0 * wc @ mu.astype(np.float64)
    exact = c[None, :] - 2.0 * X @ wc.T
    err = np.abs(scores.astype(np.float64) - exact).max(1)
    assert np.all(err <= 0.5 * margin), (2 * err / margin).max()
    ordered = exact[:, node_of]
    want_m = np.stack([ordered[:, b:b + 128].min(1) for b in range(0, k, 128)])
    err_m = np.abs(m.astype(np.float64) - want_m).max(0)
    assert np.all(err_m <= 0.5 * select), (2 * err_m / select).max()
    print(f"used {used}, worst error / half the margin: fine {(2 * err / margin).max():.3f}, coarse {(2 * err_m / select).max():.3f}")


def test_an_epoch_by_default(oracle):
    """Large enough to try the coordinates by itself."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(8860)
    rows, cols, dim, n = 45, 45, 1100, 120_000
    csr = sparse_zipf_csr(n, dim, 86, mean_len=60.0, max_len=120)
    few = (csr[0][:4001], csr[1][:csr[0][4000]], csr[2][:csr[0][4000]])
    W = _smooth_book(rng, rows, cols, dim, 14.0, few)
    som = Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W))
    b = som.train_epoch(P.csr_to_dev(csr), 14.0).cpu().numpy()
    assert capi.som_debug_subspace_used(som.ctx)[0::2] == (1, 1)
    som.close()
    P.check_bmus_csr(oracle, few, dim, W, b[:4000])


@pytest.mark.parametrize("book", ["random", "nan", "inf", "constant"])
def test_code_books_it_is_not_for(oracle, book):
    """Full rank, non-finite, and equal rows: the same nodes as a search that does not try the coordinates."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8900)
    rows, cols, dim, n = 25, 40, 1300, 300
    csr = sparse_zipf_csr(n, dim, 89, mean_len=30.0, max_len=100)
    W = rng.random((rows * cols, dim)).astype(np.float32) * np.float32(0.01)
    if book == "constant":
        W[:] = W[:1]
    elif book != "random":
        W = _smooth_book(rng, rows, cols, dim, 11.0, csr)
        W[77, 5] = np.nan if book == "nan" else np.inf
    dev = P.csr_to_dev(csr)
    som = Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W), filter="two_level")
    want = som.bmus(dev).cpu().numpy()
    got = som.train_epoch(dev, 11.0).cpu().numpy()           # a small set: not tried by itself
    assert som.two_level_stats() == (0, 0) and np.array_equal(got, want)
    som.codebook.copy_(torch.from_numpy(W))
    got = _always(som).train_epoch(dev, 11.0).cpu().numpy()
    if book == "random":
        assert som.two_level_stats()[0] == 0
    som.close()
    assert np.array_equal(got, want)
    if book == "constant":
        assert np.all(got == 0)


def test_ties_and_near_copies(oracle):
    """Copies of smooth nodes elsewhere on the map (the lowest index wins), rows that coincide with a node's weights."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(9000)
    rows, cols, dim, n = 32, 32, 1100, 400
    csr = sparse_zipf_csr(n, dim, 90, mean_len=40.0, max_len=200)
    W = _smooth_book(rng, rows, cols, dim, 12.0, csr)
    W[700:1000] = W[100:400]
    dev = P.csr_to_dev(csr)
    som = _always(Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W), filter="two_level"))
    b = som.train_epoch(dev, 12.0).cpu().numpy()
    assert som.two_level_stats()[0] > 0
    som.close()
    P.check_bmus_csr(oracle, csr, dim, W, b)
    assert np.all((b < 700) | (b >= 1000))


def test_recorded_epochs(oracle):
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(9100)
    rows, cols, dim, n = 30, 35, 1200, 500
    csr = sparse_zipf_csr(n, dim, 91, mean_len=40.0, max_len=200)
    books = [_smooth_book(rng, rows, cols, dim, 11.0, csr), (rng.random((rows * cols, dim)) * 0.01).astype(np.float32)]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        dev = P.csr_to_dev(csr)
        som = _always(Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(books[0]), filter="two_level"))
        start = P.to_dev(books[0])
        b = torch.empty(n, dtype=torch.int32, device="cuda")

        def epoch():
            som.codebook.copy_(start)
            som.train_epoch(dev, 11.0, bmus=b)

        epoch()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            epoch()
        for W in books + books:
            start.copy_(P.to_dev(W))
            epoch()
            eager = b.cpu().numpy()
            P.check_bmus_csr(oracle, csr, dim, W, eager)
            b.fill_(-1)
            graph.replay()
            assert np.array_equal(b.cpu().numpy(), eager)
        stream.synchronize()
        som.close()


def _held(call):
    """Device memory that the call leaves allocated, besides torch's."""
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()
    call()
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0] - torch.cuda.memory_reserved()


def test_only_epochs_hold_memory_for_it(oracle):
    """Searches of their own and the other neighbourhoods never try the coordinates: 396 bytes an instance that they do not hold."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(9200)
    rows, cols, dim, n = 20, 20, 1100, 60_000
    csr = sparse_zipf_csr(n, dim, 92, mean_len=5.0, max_len=20)
    W = _smooth_book(rng, rows, cols, dim, 8.0, csr)
    dev = P.csr_to_dev(csr)
    b = torch.empty(n, dtype=torch.int32, device="cuda")
    room = n * 396

    def context(function="gaussian", compact=False):
        som = _always(Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W), filter="two_level"))
        som.set_neighborhood(function, compact)
        return som

    som = context()
    own = _held(lambda: som.bmus(dev, b))
    want = b.cpu().numpy()
    epoch = _held(lambda: som.train_epoch(dev, 8.0, bmus=b))
    assert capi.som_debug_subspace_used(som.ctx)[1] > 0 and np.array_equal(b.cpu().numpy(), want)
    assert epoch >= room
    som.close()
    for kind in (("bubble", False), ("gaussian", True)):
        som = context(*kind)
        held = _held(lambda: som.train_epoch(dev, 8.0, bmus=b))
        assert capi.som_debug_subspace_used(som.ctx)[0] == 0
        assert held <= own + room // 4, (held, own, room)
        som.close()


def test_an_epoch_recorded_before_any_other(oracle):
    """What a search needs came with a search of its own; the coordinates did not, and nothing can be allocated while recording:
    the epoch is recorded without them."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(9300)
    rows, cols, dim, n = 20, 30, 1100, 900
    csr = sparse_zipf_csr(n, dim, 93, mean_len=30.0, max_len=100)
    W = _smooth_book(rng, rows, cols, dim, 9.0, csr)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        dev = P.csr_to_dev(csr)
        other = _always(Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W), filter="two_level"))
        eager = other.train_epoch(dev, 9.0).cpu().numpy()          # (loads the kernels)
        assert capi.som_debug_subspace_used(other.ctx)[1] > 0
        som = _always(Som(rows, cols, dim, "planar", "square", codebook=torch.from_numpy(W), filter="two_level"))
        start = P.to_dev(W)
        b = torch.empty(n, dtype=torch.int32, device="cuda")
        som.bmus(dev, b)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            som.codebook.copy_(start)
            som.train_epoch(dev, 9.0, bmus=b)
        for _ in range(3):
            b.fill_(-1)
            graph.replay()
            assert np.array_equal(b.cpu().numpy(), eager)
            np.testing.assert_allclose(som.codebook.cpu().numpy(), other.codebook.cpu().numpy(), rtol=0, atol=1e-5 * np.abs(W).max())
            other.codebook.copy_(start)
            assert np.array_equal(other.train_epoch(dev, 9.0).cpu().numpy(), eager)
        assert capi.som_debug_subspace_used(som.ctx)[0] == 0
        stream.synchronize()
        som.close()
        other.close()
