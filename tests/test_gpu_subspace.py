"""The coarse pass of the two-level search in the subspace of a smooth code book: its block minima against fp64 scores and
the margin of the block selection, at the ranks where the device's choice of the coordinates changes and at the edges of
its tiles; whole epochs against the oracle; what is left out of it (code books of full rank, non-finite rows)."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _book(rng, k, dim, rank, scale=1.0):
    """k rows in `rank` directions (of sizes that fall off a hundredfold), plus a common row; rank 0: any rows."""
    if rank == 0:
        return rng.random((k, dim)).astype(np.float32) * np.float32(scale)
    a = rng.standard_normal((k, rank)) * np.logspace(0, -2, rank)
    b = np.linalg.qr(rng.standard_normal((dim, rank)))[0].T
    return (scale * (rng.random(dim) + a @ b)).astype(np.float32)


def _always(som):
    """These shapes are far below those that try the subspace by themselves."""
    from paper_1305_1422_amd import capi
    capi.som_debug_subspace_always(som.ctx, True)
    return som


def _used(som):
    from paper_1305_1422_amd import capi
    return capi.som_debug_subspace_used(som.ctx)


def _minima(W, X, rows, cols):
    """Block minima, margins, order of the nodes, centring vector, coordinates used [2], losses [2]."""
    from paper_1305_1422_amd import Som, capi
    k, dim = W.shape
    n = X.shape[0]
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level")
    m = torch.empty(((k + 127) // 128, n), dtype=torch.float32, device="cuda")
    margin = torch.empty(n, dtype=torch.float64, device="cuda")
    node_of = torch.empty(k, dtype=torch.int32, device="cuda")
    mu = torch.empty(dim, dtype=torch.float32, device="cuda")
    used = torch.empty(2, dtype=torch.int32, device="cuda")
    loss = torch.empty(2, dtype=torch.float32, device="cuda")
    capi.som_debug_subspace(som.ctx, P.to_dev(X), som.codebook, m, margin, node_of, mu, used, loss)
    out = m.cpu().numpy(), margin.cpu().numpy(), node_of.cpu().numpy(), mu.cpu().numpy(), used.cpu().numpy(), loss.cpu().numpy()
    som.close()
    return out


@pytest.mark.parametrize("rows,cols,dim,n,rank,want", [
    (12, 25, 65, 300, 7, 1), (1, 33, 128, 1, 28, 1), (16, 16, 255, 257, 30, 2), (37, 7, 256, 255, 60, 2), (23, 45, 1000, 520, 12, 1),
    (40, 13, 2048, 64, 45, 2), (9, 57, 97, 1000, 90, 0), (20, 20, 300, 129, 0, 0), (5, 5, 70, 33, 3, 1)])
@pytest.mark.parametrize("data", ["near", "offset", "sizes"])
def test_block_minima_within_the_margin(rows, cols, dim, n, rank, want, data):
    rng = np.random.default_rng(8000 + dim + n)
    k = rows * cols
    W = _book(rng, k, dim, rank)
    X = W[rng.integers(0, k, n)] + 0.2 * rng.standard_normal((n, dim)).astype(np.float32)
    if data == "offset":                       # data and code book far from the origin
        W, X = W + np.float32(300), X + np.float32(300)
    if data == "sizes":                        # instances of very different norms, one at the centre
        X = X * np.exp2(rng.integers(-18, 18, (n, 1))).astype(np.float32)
        X[0] = 0.0
    m, margin, node_of, mu, (used, _), _ = _minima(W, X, rows, cols)
    if data == "near":
        assert used == want
    assert np.array_equal(np.sort(node_of), np.arange(k))
    xc = (X - mu).astype(np.float32).astype(np.float64)
    wc = (W - mu).astype(np.float32).astype(np.float64)[node_of]
    exact = (wc ** 2).sum(1)[None, :] - 2.0 * xc @ wc.T
    want_m = np.stack([exact[:, b:b + 128].min(1) for b in range(0, k, 128)])
    err = np.abs(m.astype(np.float64) - want_m).max(0)
    assert np.all(err <= 0.5 * margin), (2 * err / margin).max()
    print(f"used {used}, worst error / half the margin {(2 * err / margin).max():.3f}, margin {margin.mean():.2e}")


@pytest.mark.parametrize("rows,cols,dim", [(30, 40, 200), (50, 50, 300)])
@pytest.mark.parametrize("fall,want", [(0.14, 2), (0.1, 0), (0.08, 0), (0.0, 0)])
def test_too_many_directions_end_the_attempt_early(rows, cols, dim, fall, want):
    """150 directions of sizes exp(-fall j).  What 61 of them leave of the largest node (0.3, 2.5, 7.5 and many times what may be
    left) shows in the last pivots already: the nodes' coordinates are not even computed where it is too much."""
    rng = np.random.default_rng(8050)
    k = rows * cols
    a = rng.standard_normal((k, 150)) * np.exp(-fall * np.arange(150))
    b = np.linalg.qr(rng.standard_normal((dim, 150)))[0].T
    W = (rng.random(dim) + a @ b).astype(np.float32)
    X = W[rng.integers(0, k, 100)] + np.float32(0.01) * rng.standard_normal((100, dim)).astype(np.float32)
    _, _, _, _, (used, fine), loss = _minima(W, X, rows, cols)
    assert used == want and fine == 0
    if want:
        assert 0.0 < loss[1] < loss[0]
    else:
        assert np.all(loss == -1.0)


@pytest.mark.parametrize("rows,cols,dim,n,rank", [(12, 25, 256, 300, 7), (16, 16, 257, 257, 30), (37, 7, 320, 255, 55), (23, 45, 1000, 520, 12),
                                                  (40, 13, 2048, 64, 45), (1, 33, 1001, 129, 20)])
@pytest.mark.parametrize("data", ["near", "offset", "sizes", "rest"])
def test_fine_scores_within_the_margin(rows, cols, dim, n, rank, data):
    """Every score of the fine pass on the coordinates against fp64.  "rest": nodes that lie outside by an eighth of what the fine pass
    may leave (2^-14 of the largest), and by several times that once the basis has been disturbed by it."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(8060 + dim + n)
    k = rows * cols
    W = _book(rng, k, dim, rank)
    if data == "rest":
        e = rng.standard_normal((k, dim))
        W = (W + e * (2.0 ** -17 * np.linalg.norm(W - W.mean(0), axis=1).max() / np.linalg.norm(e, axis=1))[:, None]).astype(np.float32)
    X = W[rng.integers(0, k, n)] + 0.2 * rng.standard_normal((n, dim)).astype(np.float32)
    if data == "offset":
        W, X = W + np.float32(3), X + np.float32(3)
    if data == "sizes":
        X = X * np.exp2(rng.integers(-18, 18, (n, 1))).astype(np.float32)
        X[0] = 0.0
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level")
    scores = torch.empty((n, k), dtype=torch.float32, device="cuda")
    margin = torch.empty(n, dtype=torch.float64, device="cuda")
    mu = torch.empty(dim, dtype=torch.float32, device="cuda")
    used = torch.empty(2, dtype=torch.int32, device="cuda")
    capi.som_debug_subspace_fine(som.ctx, P.to_dev(X), som.codebook, scores, mu, margin, used)
    s, margin, mu, used = scores.cpu().numpy(), margin.cpu().numpy(), mu.cpu().numpy(), used.cpu().numpy()
    som.close()
    if data != "sizes":
        assert used[1] == 1
    if not used[1]:                            # (a centring vector far from the nodes: the largest |w'| is its length then)
        return
    xc = (X - mu).astype(np.float32).astype(np.float64)
    wc = (W - mu).astype(np.float32).astype(np.float64)
    err = np.abs(s.astype(np.float64) - ((wc ** 2).sum(1)[None, :] - 2.0 * xc @ wc.T)).max(1)
    assert np.all(err <= 0.5 * margin), (2 * err / margin).max()
    print(f"used {used}, worst error / half the margin {(2 * err / margin).max():.3f}, margin {margin.mean():.2e}")


def test_what_the_fine_pass_may_leave():
    """A remainder between what the coarse and what the fine pass may leave: the coarse pass alone runs on the coordinates."""
    rng = np.random.default_rng(8070)
    rows, cols, dim = 30, 40, 300
    k = rows * cols
    base = _book(rng, k, dim, 20)
    e = rng.standard_normal((k, dim))
    e *= np.linalg.norm(base - base.mean(0), axis=1).max() / np.linalg.norm(e, axis=1)[:, None]
    for share, coarse, fine in ((2.0 ** -17, True, 1), (2.0 ** -13, True, 0), (2.0 ** -11, True, 0), (2.0 ** -6, False, 0)):
        W = (base + share * e).astype(np.float32)
        X = W[rng.integers(0, k, 200)]
        _, _, _, _, used, loss = _minima(W, X, rows, cols)
        assert (used[0] > 0) == coarse and used[1] == fine, (share, used, loss)


@pytest.mark.parametrize("rows,cols,dim,n,map_type,grid", [(30, 36, 96, 3000, "toroid", "square"), (33, 35, 200, 1999, "planar", "hexagonal"),
                                                           (40, 29, 1030, 700, "planar", "square")])
def test_epochs_of_a_schedule(oracle, rows, cols, dim, n, map_type, grid):
    """From a random code book (full rank) over wide radii (few directions) to a narrow one: registered and not."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(8100 + dim)
    means = rng.random((11, dim))
    X = (means[rng.integers(11, size=n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    som = _always(Som(rows, cols, dim, map_type, grid, codebook=torch.from_numpy(rng.random((rows * cols, dim)).astype(np.float32)),
                      filter="two_level"))
    Xd = P.to_dev(X)
    capi.som_set_data_dense(som.ctx, Xd)
    for radius, want in ((15.0, 0), (11.0, 1), (7.0, 1), (4.0, 1), (1.0, None)):      # (the first code book is random)
        P.epoch_parity_dense(oracle, som, X, Xd, radius, P.MAP[map_type], P.GRID[grid])
        tried, use, _ = _used(som)
        assert not tried if want is None else tried and (use > 0) == (want > 0)
        P.epoch_parity_dense(oracle, som, X[:501], Xd[:501].clone(), radius, P.MAP[map_type], P.GRID[grid])
    som.close()


def test_equal_rows_and_copies(oracle):
    """A code book of equal rows (no direction at all), and one whose instances' nearest nodes have copies in other blocks:
    the lowest index wins."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8200)
    rows, cols, dim, n = 40, 30, 130, 400
    k = rows * cols
    W = np.tile(rng.random((1, dim)).astype(np.float32), (k, 1))
    X = rng.random((n, dim)).astype(np.float32)
    som = _always(Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level"))
    assert np.all(som.train_epoch(P.to_dev(X), 20.0).cpu().numpy() == 0)
    W = _book(rng, k, dim, 9)
    W[600:1100] = W[50:550]
    som.codebook.copy_(P.to_dev(W))
    X = (W[rng.integers(600, 1100, n)] + 0.001 * rng.standard_normal((n, dim))).astype(np.float32)
    assert np.array_equal(som.train_epoch(P.to_dev(X), 20.0).cpu().numpy(), oracle.bmu_dense(X, W))
    assert _used(som)[:2] == (1, 1)
    som.close()


def test_non_finite_rows_go_the_general_way(oracle):
    """Infinities and NaN among the instances and the nodes: the same nodes as a search that does not try the subspace."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8300)
    rows, cols, dim, n = 36, 30, 100, 600
    k = rows * cols
    W = _book(rng, k, dim, 8)
    X = (W[rng.integers(0, k, n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    X[5, 3] = np.inf
    X[77, 99] = np.nan
    X[300] = -np.inf
    for spoil in (None, np.inf, np.nan):
        V = W.copy()
        if spoil is not None:
            V[41, 7] = spoil
        som = Som(rows, cols, dim, codebook=torch.from_numpy(V), filter="two_level")
        want = som.bmus(P.to_dev(X)).cpu().numpy()
        assert _used(som)[0] == 0
        got = _always(som).train_epoch(P.to_dev(X), 20.0).cpu().numpy()
        assert _used(som)[:2] == (1, 0)          # (the centring vector is the mean of these instances, and not finite)
        som.close()
        assert np.array_equal(got, want)


@pytest.mark.parametrize("dim", [100, 300])
def test_non_finite_instances_on_the_coordinates(oracle, dim):
    """The same among more instances than the centring vector is a sample of, which does not hold them: the others stay on the
    coordinates, and they themselves, at no finite distance from any node, get the first."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8350)
    rows, cols, n = 20, 30, 16401
    W = _book(rng, rows * cols, dim, 8)
    X = (W[rng.integers(0, rows * cols, n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    good = np.ones(n, dtype=bool)
    good[1::1202] = False                      # (every second row is in the sample)
    X[1::2404, 3] = np.inf
    X[1203::2404, 99] = np.nan
    som = _always(Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level"))
    b = som.train_epoch(P.to_dev(X), 20.0).cpu().numpy()
    assert _used(som) == (1, 1, int(dim >= 256))
    som.close()
    assert np.all(b[~good] == 0) and np.array_equal(b[good], oracle.bmu_dense(X[good], W))


def test_recorded_epochs(oracle):
    """Epochs recorded into a graph: the choice of the coordinates is made again in every replay."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(8400)
    rows, cols, dim, n = 30, 40, 150, 900
    k = rows * cols
    books = [_book(rng, k, dim, r) for r in (10, 50, 0)]
    X = (books[0][rng.integers(0, k, n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        Xd = P.to_dev(X)
        som = _always(Som(rows, cols, dim, codebook=torch.from_numpy(books[0]), filter="two_level"))
        capi.som_set_data_dense(som.ctx, Xd)
        start = P.to_dev(books[0])
        b = torch.empty(n, dtype=torch.int32, device="cuda")

        def epoch():
            som.codebook.copy_(start)
            som.train_epoch(Xd, 18.0, bmus=b)

        epoch()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            epoch()
        for W in books + books[:1]:
            start.copy_(P.to_dev(W))
            epoch()
            eager = b.cpu().numpy()
            P.check_bmus_dense(oracle, X, W, eager)
            b.fill_(-1)
            graph.replay()
            assert np.array_equal(b.cpu().numpy(), eager)
        stream.synchronize()
        som.close()


@pytest.mark.parametrize("dim,rank", [(256, 20), (300, 50), (1000, 12), (2048, 40)])
@pytest.mark.parametrize("data", ["near", "sizes", "copies"])
def test_whole_search_on_the_coordinates(oracle, dim, rank, data):
    """Code books that lie in the coordinates to rounding: the fine and the collect pass run on them too."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8700 + dim)
    rows, cols, n = 33, 37, 1100
    k = rows * cols
    W = _book(rng, k, dim, rank)
    if data == "copies":                       # near-copies that only exact distances tell apart, and exact ones
        W = W[np.arange(k) // 40 * 40]
        W += (rng.integers(-1, 2, size=W.shape) * np.float32(2.0 ** -24)).astype(np.float32)
        W[k // 2:k // 2 + 100] = W[:100]
    X = (W[rng.integers(0, k, n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    if data == "sizes":
        X = (X * np.exp2(rng.integers(-12, 12, (n, 1)))).astype(np.float32)
    som = _always(Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level"))
    b = som.bmus(P.to_dev(X)).cpu().numpy()
    tried, use, fine = _used(som)
    assert tried and use and fine
    som.close()
    P.check_bmus_dense(oracle, X, W, b)
    assert np.array_equal(b, oracle.bmu_dense(X, W))


@pytest.mark.parametrize("rows,cols,dim,n", [(20, 20, 100, 5000), (40, 40, 200, 2000)])
@pytest.mark.parametrize("filt", ["two_level", "auto"])
def test_small_searches_do_not_try_it(oracle, rows, cols, dim, n, filt):
    """By whatever name: the basis alone would cost a small search more than the coordinates save."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8800 + dim)
    W = _book(rng, rows * cols, dim, 9)
    X = (W[rng.integers(0, rows * cols, n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter=filt)
    want = oracle.bmu_dense(X, W)
    assert np.array_equal(som.bmus(P.to_dev(X)).cpu().numpy(), want) and _used(som)[0] == 0
    assert np.array_equal(som.train_epoch(P.to_dev(X), 20.0).cpu().numpy(), want) and _used(som)[0] == 0
    som.close()


def test_only_the_gaussian_neighbourhood_holds_memory_for_it():
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8900)
    rows, cols, dim, n = 20, 25, 260, 60_000
    W = _book(rng, rows * cols, dim, 9)
    Xd = P.to_dev((W[rng.integers(0, rows * cols, n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32))
    b = torch.empty(n, dtype=torch.int32, device="cuda")
    held = {}
    kinds = (("gaussian", False), ("gaussian", True), ("bubble", False))
    for function, compact in kinds + kinds:    # (the second time nothing is left to load)
        som = _always(Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level"))
        som.set_neighborhood(function, compact)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        som.train_epoch(Xd, 8.0, bmus=b)
        torch.cuda.synchronize()
        held[function, compact] = before - torch.cuda.mem_get_info()[0]
        assert _used(som)[0] == int((function, compact) == ("gaussian", False))
        som.close()
    room = n * 396
    assert held["gaussian", False] >= held["gaussian", True] + 3 * room // 4
    assert held["gaussian", False] >= held["bubble", False] + 3 * room // 4


def test_a_search_by_default(oracle):
    """Large enough to try the subspace by itself: an epoch, and a search of its own, which takes twice the work."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(8950)
    rows, cols, dim, n = 40, 50, 320, 280_000
    k = rows * cols
    W = _book(rng, k, dim, 9)
    Xd = torch.from_numpy(W).cuda()[torch.from_numpy(rng.integers(0, k, n)).cuda()] + 0.05 * torch.randn((n, dim), device="cuda")
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W))
    b = som.bmus(Xd).cpu().numpy()
    assert _used(som) == (1, 1, 1)
    few = slice(0, 20_011)
    assert np.array_equal(b[few], oracle.bmu_dense(Xd[few].cpu().numpy(), W))
    assert np.array_equal(som.train_epoch(Xd, 20.0).cpu().numpy(), b) and _used(som) == (1, 1, 1)
    som.codebook.copy_(torch.from_numpy(W))
    half = Xd[: n // 2].contiguous()
    assert np.array_equal(som.bmus(half).cpu().numpy(), b[: n // 2]) and _used(som)[0] == 0
    assert np.array_equal(som.train_epoch(half, 20.0).cpu().numpy(), b[: n // 2]) and _used(som) == (1, 1, 1)
    som.close()
