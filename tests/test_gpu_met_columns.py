"""Searches of few sparse instances write only the columns of the transposed code book that they meet (gpu tests, through the C ABI)."""
import numpy as np
import pytest

from gen import sparse_zipf_csr
from tests import parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim,rows,cols", [(2000, 9, 11), (1999, 40, 70), (257, 24, 22)])
def test_searches_of_changing_columns_and_code_books(oracle, dim, rows, cols):
    """One context: other columns, other code books, sets on both sides of four nonzeros per column, a registered set, empty rows."""
    from paper_1305_1422_amd import Som, capi
    rng = np.random.default_rng(dim)
    som = Som(rows, cols, dim, "planar", "square", codebook=torch.zeros(rows * cols, dim))
    registered = sparse_zipf_csr(70, dim, 7, mean_len=12.0, max_len=40)
    registered_d = P.csr_to_dev(registered)
    capi.som_set_data_csr(som.ctx, *registered_d)
    for turn, n in enumerate([3, 90, dim // 3, 5, 40, 0, 60]):
        W = rng.random((rows * cols, dim)).astype(np.float32)
        som.codebook.copy_(torch.from_numpy(W))
        if turn == 4:
            csr, csr_d = registered, registered_d
        elif n == 0:                                         # nothing but empty rows
            csr = (np.zeros(6, dtype=np.int64), np.zeros(0, dtype=np.int32), np.zeros(0, dtype=np.float32))
            csr_d = P.csr_to_dev(csr)
        else:
            csr = sparse_zipf_csr(n, dim, 100 + turn, mean_len=15.0, max_len=50)
            if turn % 2:                                     # mirrored: the columns that the others hardly meet
                cols_of = [np.sort(dim - 1 - csr[1][csr[0][j]:csr[0][j + 1]]) for j in range(n)]
                csr = (csr[0], np.concatenate(cols_of).astype(np.int32), csr[2])
            csr_d = P.csr_to_dev(csr)
        b = som.bmus(csr_d).cpu().numpy()
        P.check_bmus_csr(oracle, csr, dim, W, b)
    som.close()
