"""How far an infinity or a NaN in B reaches (include/smat.h, smat_spmm): the rows that store its column, where on tiles
and quads an infinity stays one, as NaN perhaps the rest of their group, and nothing else.  Small integers: whatever it does not reach is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2408_11551_amd as S                # noqa: E402
from oracle import smat_ref as R                # noqa: E402
from workloads import random_csr, recast        # noqa: E402

INF = {"f16": 0x7C00, "bf16": 0x7F80, "e5m2": 0x7C}
NAN = {"f16": 0x7E00, "bf16": 0x7FC0, "e5m2": 0x7E, "e4m3": 0x7F}


def _check(dtype, bits, shape, dense_tiles, oracle_c):
    M, K, N, density = shape
    w = random_csr(M, K, N, density, seed=M + N, values="smallint", b_dist="smallint")
    w = w if dtype == "f16" else recast(w, dtype)
    # one in a column that few rows store, one in the last row of B
    spots = [(K // 3, N // 2), (K - 1, N - 1)]
    b = w.b_bits.reshape(K, N).copy()
    for k, n in spots:
        b[k, n] = bits
    m = S.SmatMatrix(M, K, w.row_ptr, w.col_idx, w.a_bits, dtype, reorder=0, dense_tiles=dense_tiles)
    c = m.spmm(torch.from_numpy(b.view(np.int16 if b.itemsize == 2 else np.uint8)).cuda())
    torch.cuda.synchronize()
    name = S.smat_last_launches()[0]
    m.close()
    got = c.cpu().numpy().astype(np.float64)
    ref, _ = oracle_c.spmm_ref_c(M, K, N, w.row_ptr, w.col_idx, R.decode_bits(w.a_bits, dtype), R.decode_bits(w.b_bits, dtype))
    group = 16 if dense_tiles < 0 else 256
    rows = np.repeat(np.arange(M), np.diff(w.row_ptr))
    may = np.zeros((M, N), bool)
    for k, n in spots:
        needs = w.col_idx == k if dense_tiles < 0 else w.col_idx // 16 == k // 16
        groups = np.unique(rows[needs] // group)
        may[:, n] |= np.isin(np.arange(M) // group, groups)
        a = R.decode_bits(w.a_bits, dtype)
        stored = (w.col_idx == k) & (a != 0)
        assert stored.any(), name
        if bits in NAN.values():
            assert np.isnan(got[rows[stored], n]).all(), name
        elif name == "rows":                                                    # (a block row kept by entry multiplies a column once per entry)
            assert not np.isfinite(got[rows[stored], n]).any(), name
        else:                                                                   # infinity times what is stored, sign and all
            assert np.array_equal(got[rows[stored], n], np.sign(a[stored]) * np.inf), name
    assert (~may).any(axis=1).any()
    assert np.array_equal(got[~may], ref[~may]), name                          # not reached: exact
    reached = may & (got != ref)                                               # reached without storing the column: NaN
    for k, n in spots:
        reached[rows[w.col_idx == k], n] = False
    assert np.isnan(got[reached]).all(), name
    return name


# the kernel for few columns, tiles on quads, tiles without, and block rows by themselves
@pytest.mark.parametrize("dtype,bits", [(d, b) for kind in (INF, NAN) for d, b in kind.items()])
def test_nonfinite_elements_of_b(dtype, bits, oracle_c):
    es = 2 if dtype in ("f16", "bf16") else 1
    few = _check(dtype, bits, (4100, 4096, 8, 0.11) if es == 2 else (2600, 4110, 8, 0.11), 0, oracle_c)
    assert "quad_rows" in few, few
    tiles = _check(dtype, bits, (1024, 2100, 144, 0.1), 1, oracle_c)
    assert "quad_tiles" in tiles, tiles
    short = _check(dtype, bits, (1024, 512, 144, 0.12), 1, oracle_c)            # one group of waves, without quads
    assert short.split("+")[-1] in ("tiles", "sum_tiles"), short
    for shape in ((300, 700, 33, 0.02), (1024, 2100, 144, 0.1), (150, 170, 5, 0.08)):
        rows = _check(dtype, bits, shape, -1, oracle_c)
        assert rows == "rows", rows
