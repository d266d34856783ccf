"""The clustering once its scan has asked for the partners of all patterns (preprocess.cpp): matrices whose counting is
long enough for that, with repeated patterns, empty rows and short rows among long ones, against the C oracle."""
import numpy as np
import pytest

import paper_2408_11551_amd as S
from oracle import cref


def _matrix(M, K, per_row, seed):
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 2 * per_row + 1, size=M)
    deg[rng.random(M) < 0.2] = rng.integers(0, 4)                    # short and empty rows
    rows = np.repeat(np.arange(M), deg)
    keys = np.unique(rows * K + rng.integers(0, K, rows.size))
    r, c = keys // K, keys % K
    lists = [c[s:e] for s, e in zip(np.searchsorted(r, np.arange(M)), np.searchsorted(r, np.arange(M), side="right"))]
    for i in rng.integers(1, M, M // 8):                               # some rows repeat an earlier one, whole or in part
        src = lists[rng.integers(0, i)]
        lists[i] = src if rng.random() < 0.5 else src[rng.random(src.size) < 0.7]
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum([x.size for x in lists], out=row_ptr[1:])
    return row_ptr, np.concatenate(lists).astype(np.int32)


@pytest.mark.parametrize("tau", [0, 300, 700, 900, 1000])
@pytest.mark.parametrize("shape", [(6001, 2000, 12), (3000, 20000, 300)], ids=["short", "long"])
def test_permutation_with_partners(shape, tau):
    M, K, per_row = shape
    row_ptr, col_idx = _matrix(M, K, per_row, seed=tau + M)
    h = S.smat_preprocess(M, K, row_ptr, col_idx, np.ones(col_idx.size, np.uint16), "f16", tau_permille=tau)
    pp, pi = cref.block_pattern_csr(M, K, row_ptr, col_idx)
    perm, n_e, n_id, used = cref.choose_perm_c(M, pp, pi, (K + 15) // 16, tau)
    info = S.smat_get_info(h)
    assert np.array_equal(S.smat_export_perm(h, M), perm)
    assert (info["n_blocks"], info["n_blocks_identity"], info["used_identity"]) == (n_e, n_id, bool(used))
    S.smat_destroy(h)
