"""The index of patterns by column is made in parts of as many entries: orders where the parts come out uneven, against the oracle's."""
import numpy as np
import pytest

import paper_2408_11551_amd as S
from oracle import cref


# (rows, columns, entries of the short rows, long rows and their entries): one pattern longer than a part; more long patterns than parts; patterns of one
# length; hardly more patterns than are indexed in parts at all
@pytest.mark.parametrize("M,K,short,n_long,long", [(3000, 8000, 1, 1, 7000), (4000, 16000, 2, 40, 4000), (2500, 4096, 3, 0, 0), (1040, 6000, 2, 3, 5000)])
def test_order_with_uneven_patterns(M, K, short, n_long, long):
    rng = np.random.default_rng(M)
    rows = [np.unique(rng.integers(0, K, short)) for _ in range(M)]
    for r in rng.choice(M, n_long, replace=False):
        rows[r] = np.unique(rng.integers(0, K, long))
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum([x.size for x in rows], out=row_ptr[1:])
    col_idx = np.concatenate(rows).astype(np.int32)
    pp, pi = cref.block_pattern_csr(M, K, row_ptr, col_idx)
    perm, n_blocks, _, _ = cref.choose_perm_c(M, pp, pi, (K + 15) // 16, 700)
    h = S.smat_preprocess(M, K, row_ptr, col_idx, np.ones(col_idx.size, np.uint16), "f16")
    assert np.array_equal(S.smat_export_perm(h, M), perm) and S.smat_get_info(h)["n_blocks"] == n_blocks
    S.smat_destroy(h)
