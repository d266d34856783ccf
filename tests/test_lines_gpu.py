"""The per-row kernel for rows of B on whole cache lines (kernels_lines.hip): widths around its slabs of one line, all row classes, rows split over
one to eight waves; nothing outside the N columns is read into a result or written."""
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
    # by entry, B long enough for narrow slabs to pay; by column, few packs
    for w in (random_csr(1100, 16000, N, 0.0008, seed=extra, values="smallint", b_dist="smallint"),
              random_csr(1030, 300, N, 0.3, seed=extra, values="smallint", b_dist="smallint"),
              occupancy_csr(OCCUPANCY_SPEC * 9, K=16 * 64 + 5, N=N, seed=extra)):
        w = w if dtype == "f16" else recast(w, dtype)
        name = _exact(w, oracle_c, ldb, N + 3, 0)
        assert "_lds_l8" in name, name
