"""Few columns on the list of stored entries (kernels_entries.hip): every number of lanes to a row, of columns in LDS and of rounds of a workgroup, rows of every
length, B from every address.  Small integers: every result is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2408_11551_amd as S            # noqa: E402
from oracle import smat_ref as R            # noqa: E402

HOLE = {"f16": 0x7E00, "bf16": 0x7FC0, "e4m3": 0x7F, "e5m2": 0x7F, "i8": 0x7F}
INF = {"f16": 0x7C00, "bf16": 0x7F80, "e5m2": 0x7C}
SMALL = {"f16": [0x3C00, 0x4000, 0x4200, 0xBC00, 0xC000, 0xC200], "bf16": [0x3F80, 0x4000, 0x4040, 0xBF80, 0xC000, 0xC040],
         "e4m3": [0x38, 0x40, 0x44, 0xB8, 0xC0, 0xC4], "e5m2": [0x3C, 0x40, 0x42, 0xBC, 0xC0, 0xC2], "i8": [1, 2, 3, 0xFF, 0xFE, 0xFD]}


def _matrix(M, K, per_row, dtype, seed):
    """Rows of per_row entries on average, among them empty ones, full ones and those of one to nine entries."""
    rng = np.random.default_rng(seed)
    lens = np.clip(rng.binomial(K, per_row / K, M), 1, K)
    lens[rng.integers(0, M, 12)] = np.r_[0, 0, np.arange(1, 10), 0]
    lens[[0, M // 2, M - 1]] = K, 0, K
    cols = [np.sort(rng.permutation(K)[:n]) if n < K else np.arange(K) for n in lens]
    word = np.uint16 if dtype in ("f16", "bf16") else np.uint8
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum(lens, out=row_ptr[1:])
    return row_ptr, np.concatenate(cols).astype(np.int32), rng.choice(np.array(SMALL[dtype], word), int(row_ptr[-1])), rng


def _product(matrix, M, K, N, dtype, ldb, ldc, shift, oracle_c):
    m, (row_ptr, cols, vals, rng) = matrix
    word = vals.dtype
    b_bits = rng.choice(np.array(SMALL[dtype], word), (K, N))
    # the rows of B end with the buffer, and what is not B is not a number
    flat = np.full(shift + (K - 1) * ldb + N, HOLE[dtype], word)
    for n in range(N):
        flat[shift + n:shift + n + (K - 1) * ldb + 1:ldb] = b_bits[:, n]
    flat = torch.from_numpy(flat.view(np.int16 if word.itemsize == 2 else np.int8)).cuda()
    b = torch.as_strided(flat, (K, N), (ldb, 1), shift)
    integer = dtype == "i8"
    c = torch.full((M, ldc), -77 if integer else float("nan"), dtype=torch.int32 if integer else torch.float32, device="cuda")
    S.smat_spmm(m.handle, b, c, N)
    got = c.cpu().numpy()
    name, launches = S.smat_last_kernel(), S.smat_last_launches()
    assert (got[:, N:] == -77).all() if integer else np.isnan(got[:, N:]).all()
    ref, _ = oracle_c.spmm_ref_c(M, K, N, row_ptr, cols, R.decode_bits(vals, dtype), R.decode_bits(b_bits, dtype))
    assert np.array_equal(got[:, :N].astype(np.float64), ref), (name, N, ldb, ldc, shift)
    if "entries" in name:
        assert launches == ("entries", 0.0)
    return name


# 64, 32 and 16 lanes to a row, one and several rows to each of them; a workgroup's row of B of 1 ... 32 bytes
@pytest.mark.parametrize("shape", [(1100, 9001, 500, 64), (9001, 1500, 100, 32), (26001, 1111, 80, 16), (40007, 700, 60, 16)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", ["f16", "bf16", "e4m3", "e5m2", "i8"])
def test_products_on_the_entry_list(dtype, shape, oracle_c):
    M, K, per_row, lanes = shape
    matrix = _matrix(M, K, per_row, dtype, seed=M)
    m = S.SmatMatrix(M, K, *matrix[:3], dtype, reorder=0)
    names = set()
    for N in (1, 2, 3, 4, 5, 8, 11, 16):
        for ldb, ldc, shift in {(N, N, 0), (N + 1, N + 2, 1), (-(-N // 4) * 4, N, 0), (16 if N > 8 else 8, N + 1, 3)}:
            names.add(_product((m, matrix), M, K, N, dtype, max(ldb, N), ldc, shift, oracle_c))
    m.close()
    assert any("entries" in n and n.endswith(f"x{lanes}") for n in names), names


@pytest.mark.parametrize("dtype", list(INF))
def test_infinities_reach_the_rows_that_store_their_column(dtype):
    """Also row 0 of B, and the list's entries that stand for none."""
    M, K, N = 1100, 9001, 3
    row_ptr, cols, vals, rng = _matrix(M, K, 501, dtype, seed=5)
    m = S.SmatMatrix(M, K, row_ptr, cols, vals, dtype, reorder=0)
    b = torch.zeros((K, N), dtype=torch.int16 if vals.itemsize == 2 else torch.int8, device="cuda")
    spots = [(0, 0), (K // 2, 1), (K - 1, 2)]
    for k, n in spots:
        b[k, n] = INF[dtype]
    got = m.spmm(b).cpu().numpy()
    assert "entries" in S.smat_last_kernel()
    m.close()
    rows = np.repeat(np.arange(M), np.diff(row_ptr))
    a = R.decode_bits(vals, dtype)
    want = np.zeros((M, N))
    for k, n in spots:
        want[rows[cols == k], n] = np.sign(a[cols == k]) * np.inf
    assert np.array_equal(got, want)
