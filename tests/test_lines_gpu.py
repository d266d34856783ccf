"""The per-row kernel that gathers rows of B through LDS (kernels_lines.hip): widths around its slabs of a line and of half a line, all row classes, rows
split over one to eight waves, rows of B that begin anywhere; nothing outside the N columns is read into a result or written."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2408_11551_amd as S                                        # noqa: E402
from workloads import OCCUPANCY_SPEC, occupancy_csr, random_csr, recast  # noqa: E402
from test_off_width_gpu import _exact                                   # noqa: E402


@pytest.mark.parametrize("dtype", ["f16", "bf16", "e4m3", "e5m2", "i8"])
@pytest.mark.parametrize("part", [0.55, 0.98, 1.0])
def test_one_slab_every_class_and_split(dtype, part, oracle_c):
    es = 2 if dtype in ("f16", "bf16") else 1
    N, ldb = int(128 // es * part), 128 // es
    names = set()
    for w in (random_csr(1030, 1700, N, 0.008, seed=1, values="smallint", b_dist="smallint"),          # by entry, short rows
              random_csr(1024, 3000, N, 0.009, seed=2, values="smallint", b_dist="smallint"),           # longer ones
              random_csr(1024, 12000, N, 0.013, seed=3, values="smallint", b_dist="smallint"),
              random_csr(1040, 3000, N, 0.1, seed=4, values="smallint", b_dist="smallint"),             # by column
              occupancy_csr(OCCUPANCY_SPEC * 9, K=16 * 64 + 5, N=N, seed=5)):                             # all classes
        w = w if dtype == "f16" else recast(w, dtype)
        for wide, ldc in ((ldb, N), (2 * ldb, N + 1)):
            names.add(_exact(w, oracle_c, wide, ldc, 0))
    assert all("_lds_l8" in name for name in names), names
    assert {name.split("_")[2][2:4] for name in names} >= {"k1", "k4", "k8"}, names


@pytest.mark.parametrize("dtype", ["f16", "e4m3", "i8"])
@pytest.mark.parametrize("extra", [1, 30, 64, 250])
def test_several_slabs(dtype, extra, oracle_c):
    es = 2 if dtype == "f16" else 1
    N = 128 // es + extra
    ldb = (N * es + 127) // 128 * 128 // es
    # by entry, short rows; by column, few packs
    for w in (random_csr(1100, 20000, N, 0.00064, seed=extra, values="smallint", b_dist="smallint"),
              random_csr(1030, 300, N, 0.3, seed=extra, values="smallint", b_dist="smallint"),
              occupancy_csr(OCCUPANCY_SPEC * 9, K=16 * 64 + 5, N=N, seed=extra)):
        near = w.K == 16 * 64 + 5                  # (rows of B from a part of them: another kernel's in 16 bits)
        w = w if dtype == "f16" else recast(w, dtype)
        name = _exact(w, oracle_c, ldb, N + 3, 0)
        assert "_lds_l8" in name or near and dtype == "f16", name


@pytest.mark.parametrize("dtype", ["f16", "bf16", "e4m3", "e5m2", "i8"])
@pytest.mark.parametrize("slab", [64, 128])
@pytest.mark.parametrize("widest", [False, True])
def test_rows_that_begin_anywhere(dtype, slab, widest, oracle_c):
    """On dwords only, and off them by every number of places: the NaN around a row and in the rows next to it (whose columns come with the
    slab) reach no result."""
    es = 2 if dtype in ("f16", "bf16") else 1
    names = set()
    for ldb_off, shift in ((0, 0), (4 // es, 0), (8 // es, 4 // es), (1, 0), (0, 1), (2, 1), (3, 2), (1, 3), (5, 3)):
        on_dwords = ldb_off * es % 4 == 0 and shift * es % 4 == 0
        N = (slab - (0 if on_dwords else 4 - es)) // es if widest else slab // 2 // es + 1
        ldb = (N * es + 3) // 4 * 4 // es + ldb_off
        for w in (random_csr(1030, 1700, N, 0.008, seed=1, values="smallint", b_dist="smallint"),
                  random_csr(1610, 1500, N, 0.1, seed=4, values="smallint", b_dist="smallint"),
                  occupancy_csr(OCCUPANCY_SPEC * 9, K=16 * 64 + 5, N=N, seed=5)):
            w = w if dtype == "f16" else recast(w, dtype)
            name = _exact(w, oracle_c, ldb, N + 1, shift)
            assert name.endswith("_lds_l8" if on_dwords else "_ldso_l8"), (name, N, ldb, shift)
            names.add(name)
    assert len({name.split("_")[2][:2] for name in names}) == 1 and len(names) > 2, names


@pytest.mark.parametrize("dtype", ["f16", "e4m3", "i8"])
@pytest.mark.parametrize("more", [1, 30, 127])
def test_several_slabs_that_begin_anywhere(dtype, more, oracle_c):
    """Off the dwords a slab has as many columns fewer as a row may be shifted by."""
    es = 2 if dtype == "f16" else 1
    N = 120 // es + more
    for ldb_off, shift in ((0, 0), (4 // es, 4 // es), (1, 0), (0, 1), (3, 2)):
        ldb = (N * es + 3) // 4 * 4 // es + ldb_off
        for w in (random_csr(1030, 1700, N, 0.008, seed=more, values="smallint", b_dist="smallint"),
                  random_csr(1024, 400, N, 0.1, seed=more, values="smallint", b_dist="smallint")):
            w = w if dtype == "f16" else recast(w, dtype)
            name = _exact(w, oracle_c, ldb, N + 1, shift)
            assert "_lds" in name, (name, N, ldb, shift)


def test_columns_of_infinities_stay_in_their_columns(oracle_c):
    """A column of infinities or NaN in B off the dwords: its own column of C alone, though it lies in the place of the next one's."""
    w = random_csr(1030, 1700, 51, 0.008, seed=7, values="smallint", b_dist="smallint")
    b = torch.from_numpy(w.b_bits.view(np.int16)).view(torch.float16).cuda()
    b[:, 17], b[:, 34], b[:, 50] = float("inf"), float("nan"), float("inf")
    m = S.SmatMatrix(w.M, w.K, w.row_ptr, w.col_idx, w.a_bits, "f16", reorder=0)
    out = []
    for x in (b, torch.nan_to_num(b, nan=0.0, posinf=0.0)):
        c = torch.empty((w.M, w.N), dtype=torch.float32, device="cuda")
        S.smat_spmm(m.handle, x.view(torch.int16), c, w.N)
        torch.cuda.synchronize()
        assert "_ldso_" in S.smat_last_kernel()
        out.append(c.cpu())
    m.close()
    others = [j for j in range(w.N) if j not in (17, 34, 50)]
    assert torch.equal(out[0][:, others], out[1][:, others])
    assert not torch.isfinite(out[0][:, [17, 34, 50]]).all()
