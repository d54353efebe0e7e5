"""Calls recorded into a HIP graph: every call clears the counters and lists that its own search appends to, so that a
recorded search does not build on what another call did, or was only recorded to do."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("filt", ["split_f16", "two_level", "fp32"])
def test_filtered_search_beside_a_direct_epoch(oracle, filt):
    """A map full of near-copies (every list of the exact stage is in use).  A small epoch, searched without a filter
    pass, and a filtered search are recorded one after the other; an eager filtered search runs while the recorded epoch
    has not, and between the replays."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(9100)
    rows, cols, dim, n = 24, 25, 40, 1500
    means = rng.random((12, dim))
    W = (means[rng.integers(0, 12, rows * cols)] + 1e-7 * rng.standard_normal((rows * cols, dim))).astype(np.float32)
    X = (means[rng.integers(0, 12, n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    small = rng.random((30, dim)).astype(np.float32)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        Xd, Sd, Wd = P.to_dev(X), P.to_dev(small), P.to_dev(W)
        som = Som(rows, cols, dim, codebook=torch.from_numpy(W))
        b_small = torch.empty(30, dtype=torch.int32, device="cuda")
        b, b_eager = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")

        def both():
            som.codebook.copy_(Wd)
            som.set_filter("auto")
            som.train_epoch(Sd, 1.0, bmus=b_small)
            som.codebook.copy_(Wd)
            som.set_filter(filt)
            som.bmus(Xd, b)

        both()                                    # allocates what the recorded calls need
        want_small, want = b_small.cpu().numpy(), b.cpu().numpy()
        stats = som.stats()
        assert stats[1] > 0                       # the lists are in use
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            both()
        som.bmus(Xd, b_eager)
        assert np.array_equal(b_eager.cpu().numpy(), want) and som.stats() == stats
        for _ in range(4):
            b.fill_(-1)
            b_small.fill_(-1)
            graph.replay()
            assert np.array_equal(b.cpu().numpy(), want) and np.array_equal(b_small.cpu().numpy(), want_small)
            assert som.stats() == stats
            som.bmus(Xd, b_eager)
            assert np.array_equal(b_eager.cpu().numpy(), want)
        stream.synchronize()
        som.close()
    P.check_bmus_dense(oracle, X, W, want)


def test_stats_are_those_of_the_search_that_ran_last():
    """The counters belong to the search that the GPU ran last, whether it was called or replayed: a search without a
    filter pass leaves zeros, a replayed filtered one its own figures."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(9200)
    rows, cols, dim, n = 20, 20, 30, 900
    means = rng.random((10, dim))
    W = (means[rng.integers(0, 10, rows * cols)] + 1e-7 * rng.standard_normal((rows * cols, dim))).astype(np.float32)
    X = (means[rng.integers(0, 10, n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        Xd = P.to_dev(X)
        b = torch.empty(n, dtype=torch.int32, device="cuda")
        som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="split_f16")
        som.bmus(Xd, b)
        stats = som.stats()
        assert stats[1] > 0
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            som.bmus(Xd, b)
        som.set_filter("auto")
        for _ in range(3):
            som.bmus(Xd, b)
            assert som.stats() == (0, 0, 0)
            graph.replay()
            assert som.stats() == stats
        som.close()


def test_smaller_calls_need_no_more_scratch(oracle):
    """A context that has served a large set serves any smaller one without growing: it can be recorded, which rules out
    an allocation and a wait.  (The other context sees to it that the kernels have been loaded.)"""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(9300)
    rows, cols, dim = 50, 50, 100
    W = rng.random((rows * cols, dim)).astype(np.float32)
    X = rng.random((20000, dim)).astype(np.float32)
    sizes = (1500, 4000, 700, 64, 3)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        Xd = P.to_dev(X)
        b = torch.empty(len(X), dtype=torch.int32, device="cuda")
        other = Som(rows, cols, dim, codebook=torch.from_numpy(W))
        want = {}
        for n in sizes:
            want[n] = other.bmus(Xd[:n]).cpu().numpy()
            assert other.stats() == (0, 0, 0)            # searched without a filter pass
        som = Som(rows, cols, dim, codebook=torch.from_numpy(W))
        som.bmus(Xd, b)
        stream.synchronize()
        for n in sizes:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                som.bmus(Xd[:n], b[:n])
            for _ in range(3):
                b.fill_(-1)
                graph.replay()
                assert np.array_equal(b[:n].cpu().numpy(), want[n]) and int(b[n]) == -1
        stream.synchronize()
        som.close()
        other.close()
    P.check_bmus_dense(oracle, X[:1500], W, want[1500])


def test_recorded_searches_of_changing_sparse_rows(oracle):
    """A search of few unregistered rows writes only the columns they meet and marks them with a number of its own, which a
    replay uses again: its rows and the code book change in place, and plain searches of other rows come between."""
    from gen import sparse_zipf_csr
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(9400)
    rows, cols, dim, n, m = 24, 26, 1500, 60, 40          # 2,400 nonzeros on 1,500 columns
    stream = torch.cuda.Stream()

    def draw(low):                                         # columns of one half, or anywhere
        columns = [np.sort(rng.choice(dim // 2, size=m, replace=False)) + low for _ in range(n)]
        return (np.arange(n + 1, dtype=np.int64) * m, np.concatenate(columns).astype(np.int32),
                (rng.random(n * m) + 0.1).astype(np.float32))

    with torch.cuda.stream(stream):
        csr = draw(0)
        csr_d = P.csr_to_dev(csr)
        W = rng.random((rows * cols, dim)).astype(np.float32)
        som = Som(rows, cols, dim, codebook=torch.from_numpy(W))
        b = torch.empty(n, dtype=torch.int32, device="cuda")
        som.bmus(csr_d, b)                                 # allocates what the recorded call needs
        other = sparse_zipf_csr(30, dim, 9401, mean_len=20.0, max_len=60)
        other_d = P.csr_to_dev(other)
        b_other = torch.empty(30, dtype=torch.int32, device="cuda")
        som.bmus(other_d, b_other)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            som.bmus(csr_d, b)
        for low in (0, dim // 2, dim // 4, 0, dim // 2):
            csr = draw(low)
            for dst, src in zip(csr_d, csr):
                dst.copy_(torch.from_numpy(src))
            W = rng.random((rows * cols, dim)).astype(np.float32)
            som.codebook.copy_(torch.from_numpy(W))
            som.bmus(other_d, b_other)
            b.fill_(-1)
            graph.replay()
            P.check_bmus_csr(oracle, csr, dim, W, b.cpu().numpy())
            P.check_bmus_csr(oracle, other, dim, W, b_other.cpu().numpy())
        stream.synchronize()
        som.close()


@pytest.mark.parametrize("dim,n", [(300, 90), (300, 3000), (300, 18000), (30000, 900)])
def test_recorded_updates_of_changing_sparse_rows(oracle, dim, n):
    """The sums of sparse rows by four and by eight wavefronts a node, in two copies and in several tiles, recorded once; the rows and their nodes
    change in place between the replays."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(9500 + n)
    rows, cols, m = 16, 18, 20
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        csr_d = (torch.arange(n + 1, dtype=torch.int64, device="cuda") * m, torch.zeros(n * m, dtype=torch.int32, device="cuda"),
                 torch.zeros(n * m, dtype=torch.float32, device="cuda"))
        b = torch.zeros(n, dtype=torch.int32, device="cuda")
        W = rng.random((rows * cols, dim)).astype(np.float32)
        som = Som(rows, cols, dim, codebook=torch.from_numpy(W))
        som.update(csr_d, b, 1.5)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            som.update(csr_d, b, 1.5)
        for turn in range(4):
            start = rng.integers(dim - m, size=(n, 1))
            csr = (csr_d[0].cpu().numpy(), (start + np.arange(m)).reshape(-1).astype(np.int32), rng.random(n * m).astype(np.float32))
            bmus = (rng.random(n) ** (1 + turn) * rows * cols).astype(np.int32)
            csr_d[1].copy_(torch.from_numpy(csr[1]))
            csr_d[2].copy_(torch.from_numpy(csr[2]))
            b.copy_(torch.from_numpy(bmus))
            som.codebook.copy_(torch.from_numpy(W))
            graph.replay()
            got = som.codebook.cpu().numpy()
            S, C = oracle.accumulate_csr(csr, dim, bmus, rows * cols)
            P.check_codebook(oracle, S, C, W, got, rows, cols, oracle.PLANAR, oracle.SQUARE, 1.5)
        stream.synchronize()
        som.close()
