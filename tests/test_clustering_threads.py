"""The clustering once its scan has asked for the partners of all patterns (preprocess.cpp): matrices whose counting is
long enough for that, with repeated patterns, empty rows and short rows among long ones, against the C oracle."""
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2408_11551_amd as S
from oracle import cref

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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


def _hub_matrix(M, K, hubs, seed, plain):
    """Rows of one of `hubs` shared columns and one or two of their own, among them `plain` rows of twelve random columns, some of
    which repeat."""
    rng = np.random.default_rng(seed)
    lists = []
    for i in range(M):
        if i % M < plain and rng.random() < 0.3 and lists:
            lists.append(lists[rng.integers(0, len(lists))])
        elif rng.random() < plain / M:
            lists.append(np.unique(rng.integers(0, K, 12)))
        else:
            lists.append(np.unique(np.concatenate([16 * rng.integers(0, hubs, 1), rng.integers(16 * hubs, K, rng.integers(1, 3))])))
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum([x.size for x in lists], out=row_ptr[1:])
    return row_ptr, np.concatenate(lists).astype(np.int32)


@pytest.mark.parametrize("tau", [300, 700, 900, 1000])
@pytest.mark.parametrize("hubs,plain", [(1, 0), (1, 1500), (40, 600), (300, 2000)])
def test_permutation_with_more_partners_than_are_listed(hubs, plain, tau):
    """Rows that share a column have thousands of partners, which are not listed, beside rows with a few, which are -- some of them
    only among the former."""
    M, K = 4000, 100000
    row_ptr, col_idx = _hub_matrix(M, K, hubs, seed=hubs + tau, plain=plain)
    h = S.smat_preprocess(M, K, row_ptr, col_idx, np.ones(col_idx.size, np.uint16), "f16", tau_permille=tau)
    pp, pi = cref.block_pattern_csr(M, K, row_ptr, col_idx)
    perm, n_e, _, _ = cref.choose_perm_c(M, pp, pi, (K + 15) // 16, tau)
    assert np.array_equal(S.smat_export_perm(h, M), perm) and S.smat_get_info(h)["n_blocks"] == n_e
    S.smat_destroy(h)


def test_a_shared_column_takes_no_quadratic_memory():
    """20 000 rows {one column of all, one of its own} make 200 M pairs: 1.2 GB listed, against a few MB of tables."""
    program = """
import resource
import numpy as np
import paper_2408_11551_amd as S
M, K = 20000, 320000
col_idx = np.stack([np.zeros(M, np.int32), 16 + np.random.default_rng(1).permutation(K - 16)[:M].astype(np.int32)], 1).reshape(-1)
row_ptr = np.arange(M + 1, dtype=np.int64) * 2
before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
S.smat_destroy(S.smat_preprocess(M, K, row_ptr, col_idx, np.ones(2 * M, np.uint16), "f16"))
print((resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before) // 1024)
"""
    out = subprocess.run([sys.executable, "-c", program], cwd=ROOT, stdout=subprocess.PIPE, text=True, timeout=100, check=True)
    assert int(out.stdout.split()[-1]) < 100, out.stdout
