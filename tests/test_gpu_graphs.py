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
