"""The two-level dense BMU search (coarse one-product pass, block selection, sorted tiles, split-fp16 pass
over the listed blocks) against the oracle, on the cases its block selection could get wrong: maps of many
node blocks, equal and nearly equal nodes in different blocks (ties go to the lowest index, so the block of
the lower copy must stay in), code books of equal rows (every block listed), sizes that leave ragged tiles
and blocks, tiles whose lists are shorter than the number of workgroups that share them.
"""
import numpy as np
import pytest

from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _bmus(W, X, rows, cols, filter="two_level"):
    from paper_1305_1422_amd import Som
    som = Som(rows, cols, W.shape[1], codebook=torch.from_numpy(W), filter=filter)
    b = som.bmus(P.to_dev(X)).cpu().numpy()
    stats = som.stats()
    som.close()
    return b, stats


def _ordered_map(rng, rows, cols, dim, clusters):
    """A code book that looks like a trained map: smooth over the grid, so that the nodes near an instance's BMU
    sit in a few node blocks, and the other blocks are far away."""
    anchors = rng.random((clusters, dim))
    gy, gx = np.divmod(np.arange(rows * cols), cols)
    u = np.stack([gy / max(rows - 1, 1), gx / max(cols - 1, 1)], 1)
    cpos = rng.random((clusters, 2))
    d2 = ((u[:, None, :] - cpos[None, :, :]) ** 2).sum(-1)
    wgt = np.exp(-d2 / 0.01)
    wgt /= wgt.sum(1, keepdims=True)
    return (wgt @ anchors).astype(np.float32), anchors


@pytest.mark.parametrize("n,rows,cols,dim", [(3000, 40, 45, 96), (129, 1, 129, 40), (1, 30, 50, 7), (2500, 64, 64, 200)])
def test_ordered_map_matches_the_oracle(oracle, n, rows, cols, dim):
    rng = np.random.default_rng(4100 + n)
    W, anchors = _ordered_map(rng, rows, cols, dim, 12)
    X = (anchors[rng.integers(12, size=n)] + 0.03 * rng.standard_normal((n, dim))).astype(np.float32)
    b, _ = _bmus(W, X, rows, cols)
    P.check_bmus_dense(oracle, X, W, b)
    b1, _ = _bmus(W, X, rows, cols, "split_f16")
    assert np.array_equal(b, b1)


def test_random_code_book_lists_many_blocks(oracle):
    """Unordered nodes: the candidates of a tile are spread over all blocks, the fine pass runs nearly everywhere."""
    rng = np.random.default_rng(4200)
    rows, cols, dim, n = 37, 41, 64, 2000
    W = rng.random((rows * cols, dim)).astype(np.float32)
    X = rng.random((n, dim)).astype(np.float32)
    b, _ = _bmus(W, X, rows, cols)
    P.check_bmus_dense(oracle, X, W, b)


def test_copies_of_the_best_node_in_other_blocks(oracle):
    """Every instance's nearest node has an exact copy 5 blocks further up and one a block further down: the
    lowest of the three must win, i.e. the coarse selection keeps all three blocks (equal rows have equal coarse
    scores) and the order of the listed blocks is ascending."""
    rng = np.random.default_rng(4300)
    rows, cols, dim, n = 30, 64, 48, 1500                       # 1,920 nodes = 15 blocks
    k = rows * cols
    W = rng.random((k, dim)).astype(np.float32)
    src = rng.integers(640, 1152, size=n)                        # blocks 5 .. 8
    X = (W[src] + 0.001 * rng.standard_normal((n, dim))).astype(np.float32)
    lower = src - 128 * rng.integers(1, 6, size=n)               # a copy 1 .. 5 blocks below
    upper = src + 128 * rng.integers(1, 6, size=n)
    Wc = W.copy()
    for s, lo, up in zip(src, lower, upper):
        Wc[lo] = W[s]
        Wc[up] = W[s]
    W = Wc
    b, _ = _bmus(W, X, rows, cols)
    want = oracle.bmu_dense(X, W)
    assert np.array_equal(b, want)                               # exact ties: no band, the lowest index


def test_equal_rows_everywhere(oracle):
    """All nodes equal: every block is a candidate for every instance, and node 0 wins."""
    rows, cols, dim, n = 40, 40, 33, 700
    rng = np.random.default_rng(4400)
    W = np.tile(rng.random((1, dim)).astype(np.float32), (rows * cols, 1))
    X = rng.random((n, dim)).astype(np.float32)
    b, _ = _bmus(W, X, rows, cols)
    assert np.all(b == 0)


def test_near_copies_across_blocks_are_decided_exactly(oracle):
    """Nodes that differ by a few ulps and lie in different blocks: neither pass can separate them, the exact
    stage must see all of them."""
    rng = np.random.default_rng(4500)
    rows, cols, dim, n = 25, 52, 128, 600                       # 1,300 nodes, 11 blocks (the last one ragged)
    base = rng.random((5, dim)).astype(np.float32)
    W = base[rng.integers(5, size=rows * cols)].copy()
    W += (rng.integers(-2, 3, size=W.shape) * np.float32(2.0 ** -22)).astype(np.float32)
    X = (base[rng.integers(5, size=n)] + rng.normal(0, 0.05, size=(n, dim))).astype(np.float32)
    b, (refined, collected, rescanned) = _bmus(W, X, rows, cols)
    P.check_bmus_dense(oracle, X, W, b)
    assert collected + rescanned > 0


def test_epochs_with_the_two_level_search(oracle):
    """Whole epochs (search + update) from a random code book down to a small radius, registered data: the
    order of the instances and the block lists change every epoch."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(4600)
    rows, cols, dim, n = 36, 36, 50, 4000
    means = rng.random((9, dim))
    X = (means[rng.integers(9, size=n)] + 0.05 * rng.standard_normal((n, dim))).astype(np.float32)
    W = rng.random((rows * cols, dim)).astype(np.float32)
    som = Som(rows, cols, dim, "toroid", "square", codebook=torch.from_numpy(W), filter="two_level")
    Xd = P.to_dev(X)
    capi.som_set_data_dense(som.ctx, Xd)
    for radius in (18.0, 9.0, 4.0, 2.0, 1.0):
        P.epoch_parity_dense(oracle, som, X, Xd, radius, P.MAP["toroid"], P.GRID["square"])
    som.close()


def test_default_filter_is_two_level_on_large_maps_only(oracle):
    """The default picks the two-level search from 1,024 nodes on; results are the same either way."""
    rng = np.random.default_rng(4700)
    for rows, cols in [(20, 20), (32, 40)]:
        dim, n = 24, 900
        W = rng.random((rows * cols, dim)).astype(np.float32)
        X = rng.random((n, dim)).astype(np.float32)
        b_auto, _ = _bmus(W, X, rows, cols, "auto")
        b_split, _ = _bmus(W, X, rows, cols, "split_f16")
        assert np.array_equal(b_auto, b_split)
        P.check_bmus_dense(oracle, X, W, b_auto)


def test_statistics_of_the_second_pass(oracle):
    """som_two_level_stats: the pairs the second pass worked on, out of all (tile, block) pairs; an ordered map
    lists a small share, a code book of equal rows all of them, a one-level search reports (0, 0)."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(4800)
    rows, cols, dim, n = 48, 48, 40, 3000                        # 2,304 nodes = 18 blocks, 24 tiles
    W, anchors = _ordered_map(rng, rows, cols, dim, 10)
    X = (anchors[rng.integers(10, size=n)] + 0.02 * rng.standard_normal((n, dim))).astype(np.float32)
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level")
    assert som.two_level_stats() == (0, 0)                       # no search yet
    som.bmus(P.to_dev(X))
    listed, pairs = som.two_level_stats()
    assert pairs == 24 * 18 and 24 <= listed < pairs // 2, (listed, pairs)
    som.set_filter("split_f16")
    som.bmus(P.to_dev(X))
    assert som.two_level_stats() == (0, 0)
    som.close()
    W_eq = np.tile(W[:1], (rows * cols, 1))
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W_eq), filter="two_level")
    som.bmus(P.to_dev(X))
    assert som.two_level_stats() == (pairs, pairs)
    som.close()


@pytest.mark.parametrize("rows,cols,dim", [(1, 1500, 20), (1500, 1, 20), (5, 300, 33), (300, 5, 33), (13, 100, 64), (17, 77, 65),
                                           (18, 64, 2100), (41, 29, 7)])
def test_node_patches_of_any_map_shape(oracle, rows, cols, dim):
    """The planes hold the nodes by bands of map rows: bands of one row, of all rows, of unequal heights, maps narrower
    than a block, rows too long for registers; copies of nodes in different bands (the lowest index wins), also where a
    bubble neighbourhood masks them."""
    from paper_1305_1422_amd import Som
    rng = np.random.default_rng(7000 + rows + dim)
    k, n = rows * cols, 700
    W, _ = _ordered_map(rng, rows, cols, dim, 9)
    W += 0.02 * rng.random((k, dim)).astype(np.float32)
    W[k - 1] = W[k // 2] = W[3]
    X = (W[rng.integers(0, k, n)] + 0.03 * rng.standard_normal((n, dim))).astype(np.float32)
    X[:3] = W[k - 1]
    b, _ = _bmus(W, X, rows, cols)
    P.check_bmus_dense(oracle, X, W, b)
    assert np.all(b[:3] == 3)
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level")
    som.set_neighborhood("bubble")
    assert np.array_equal(som.bmus(P.to_dev(X)).cpu().numpy(), b)
    csr = torch.from_numpy(X).to_sparse_csr()
    dev = (csr.crow_indices().cuda(), csr.col_indices().to(torch.int32).cuda(), csr.values().cuda())
    som.close()
    som = Som(rows, cols, dim, codebook=torch.from_numpy(W), filter="two_level")
    from paper_1305_1422_amd import capi
    capi.som_set_data_csr(som.ctx, *dev)
    P.check_bmus_dense(oracle, X, W, som.bmus(dev).cpu().numpy())
    som.close()


@pytest.mark.parametrize("case", ["uniform", "offset_mixture", "heavy_tail", "tiny_and_huge_rows", "ragged_dim", "odd_dim",
                                  "long_rows"])
def test_selection_margin_covers_the_coarse_scores(case):
    """The block selection's margin, made of the residuals of the rows at hand, against fp64 scores of the same centred
    rows: no coarse score is off by more than half of it, and it stays below the bound for any rows."""
    from paper_1305_1422_amd import Som, capi
    from tests.test_gpu_filter_bound import _dense_case
    rng = np.random.default_rng(7200)
    rows, cols = 12, 25
    if case == "long_rows":
        x, w = rng.random((60, 2500)).astype(np.float32), rng.random((rows * cols, 2500)).astype(np.float32)
    else:
        x, w = _dense_case(case, rng, rows, cols)
    n, dim = x.shape
    som = Som(rows, cols, dim, codebook=torch.from_numpy(w), filter="two_level")
    scores = torch.empty((n, rows * cols), dtype=torch.float32, device="cuda")
    mu = torch.empty(dim, dtype=torch.float32, device="cuda")
    any_rows = torch.empty(n, dtype=torch.float64, device="cuda")
    margin = torch.empty(n, dtype=torch.float64, device="cuda")
    capi.som_debug_scores_dense(som.ctx, P.to_dev(x), som.codebook, scores, mu, any_rows)
    capi.som_debug_select_margins(som.ctx, margin)
    with pytest.raises(Exception):
        capi.som_debug_select_margins(som.ctx, margin[:-1])
    m = mu.cpu().numpy()
    xc, wc = (x - m).astype(np.float32).astype(np.float64), (w - m).astype(np.float32).astype(np.float64)
    exact = (wc ** 2).sum(1)[None, :] - 2.0 * xc @ wc.T
    err = np.abs(scores.cpu().numpy().astype(np.float64) - exact).max(1)
    margin, any_rows = margin.cpu().numpy(), any_rows.cpu().numpy()
    som.close()
    assert np.all(err <= 0.5 * margin), (err / margin).max()
    assert np.all(margin <= any_rows)
    print(f"{case}: worst error / half the margin {(2 * err / margin).max():.3f}, margin / bound for any rows {(margin / any_rows).mean():.3f}")


@pytest.mark.parametrize("blocks", [1, 3, 4, 5, 16, 17, 31, 32, 33, 127, 128, 129, 255, 256, 257, 300, 512, 513])
def test_block_selection_at_every_number_of_blocks(oracle, blocks):
    """The selection reads the block minima in runs of four per thread, keeps 128 or 256 blocks in registers and joins mask
    words of 32: best nodes with copies in every other block, in one and in the last, ragged block and instance tile included."""
    rng = np.random.default_rng(4400 + blocks)
    rows = 1 if blocks <= 512 else 3                             # (a side has at most 65,535 nodes)
    cols, dim, n = (128 * blocks - 5) // rows, 12, 65
    k = rows * cols
    W = rng.random((k, dim)).astype(np.float32)
    src = rng.integers(0, 120, size=n)                           # first block
    src[::3] = k - 1 - rng.integers(0, 120, size=len(src[::3]))  # last block
    X = (W[src] + 1e-3 * rng.standard_normal((n, dim))).astype(np.float32)
    for i in range(0, n, 5):
        copies = (src[i] % 120 + 128 * np.arange(0, blocks, 1 + i % 2))
        W[copies] = W[src[i]]                                    # exact copies: the lowest index wins
    b, _ = _bmus(W, X, rows, cols)
    assert np.array_equal(b, oracle.bmu_dense(X, W))
