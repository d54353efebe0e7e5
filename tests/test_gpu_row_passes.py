"""The passes over whole rows (planes and norms of a dense search, distances to the best matching units) at the row
lengths where their loads end: shorter than one load, at and around the 256 features a wavefront takes at once, at and
past the longest row it holds in registers."""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DIMS = [1, 2, 3, 4, 5, 31, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 1023, 1025, 2047, 2048, 2049]


@pytest.mark.parametrize("filter", ["split_f16", "two_level"])
@pytest.mark.parametrize("dim", DIMS)
def test_planes_of_any_row_length(oracle, filter, dim):
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(6100 + dim)
    rows, cols, n = 12, 13, 203
    W = (3.0 + rng.random((rows * cols, dim))).astype(np.float32)
    X = (3.0 + rng.random((n, dim))).astype(np.float32)
    X[0] = W[7]
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter=filter)
    P.check_bmus_dense(oracle, X, W, som.bmus(P.to_dev(X)).cpu().numpy())
    som.close()


@pytest.mark.parametrize("n", [1, 7, 2051, 9001])
@pytest.mark.parametrize("dim", [1, 3, 4, 6, 64, 65, 128, 129, 256, 257, 513, 1023, 1024, 1025, 2050])
def test_distances_of_any_row_length(n, dim):
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(6200 + n + dim)
    rows, cols = 5, 9
    k = rows * cols
    W = rng.random((k, dim)).astype(np.float32)
    X = (rng.random((n, dim)) * (rng.random((n, dim)) < 0.3)).astype(np.float32)
    b = rng.integers(0, k - 3, n).astype(np.int32)          # some nodes nobody asks for
    want = np.sqrt(((X.astype(np.float64) - W[b].astype(np.float64)) ** 2).sum(1))
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W))
    csr = torch.from_numpy(X).to_sparse_csr()
    sparse = (csr.crow_indices().cuda(), csr.col_indices().to(torch.int32).cuda(), csr.values().cuda())
    for data in (P.to_dev(X), sparse, sparse):
        d, q = som.bmu_distances(data, P.to_dev(b))
        np.testing.assert_allclose(d.cpu().numpy(), want, rtol=2e-7)
        assert abs(float(q) - want.mean()) <= 2e-7 * want.mean()
    som.close()


@pytest.mark.parametrize("rows,cols", [(5, 9), (120, 130)])
def test_sparse_distances_call_after_call(rows, cols):
    """Calls of many and of few instances on one context, the code book changed in between: what an earlier call left
    behind about a node is not taken for this call's."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(6300 + rows)
    k, dim = rows * cols, 70
    som = Som(rows, cols, dim, codebook=torch.from_numpy(rng.random((k, dim)).astype(np.float32)))
    for n in (3000, 20, 44, 45, 46, 3000, 1, 20000, 700):
        W = rng.random((k, dim)).astype(np.float32)
        som.codebook.copy_(torch.from_numpy(W))
        X = (rng.random((n, dim)) * (rng.random((n, dim)) < 0.2)).astype(np.float32)
        b = (rng.integers(0, k, n) // int(rng.integers(1, 4))).astype(np.int32)
        if n > 1:
            b[n // 2] = -1                                   # no node: a NaN of its own, nothing else changes
        csr = torch.from_numpy(X).to_sparse_csr()
        sparse = (csr.crow_indices().cuda(), csr.col_indices().to(torch.int32).cuda(), csr.values().cuda())
        d, _ = som.bmu_distances(sparse, P.to_dev(b))
        want = np.sqrt(((X.astype(np.float64) - W[b].astype(np.float64)) ** 2).sum(1))
        want[b < 0] = np.nan
        np.testing.assert_allclose(d.cpu().numpy(), want, rtol=2e-7)
    som.close()
