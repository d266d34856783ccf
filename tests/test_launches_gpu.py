"""smat_last_launches names what a product enqueued, and the kernels that other tests no longer reach by size alone: the tile kernel
of two wave groups without quads, which takes fills that quads do not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2408_11551_amd as S                # noqa: E402
from oracle import smat_ref as R                # noqa: E402
from workloads import random_csr, recast        # noqa: E402


@pytest.mark.parametrize("steps", [64, 65, 66, 67, 68, 69])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "e4m3", "e5m2", "i8"])
def test_tile_kernel_without_quads_every_tail_of_its_step_loop(dtype, steps, oracle_c):
    """Tiles of 64 ... 69 steps at 60 % fill, once with the steps split over workgroups (the stream with the area) and once unsplit: ten
    or eleven passes of the three-step loop body per wave group and zero, one or two steps behind the loop."""
    es = 2 if dtype in ("f16", "bf16") else 1
    M, K, N = 512, 64 // es * steps, 144
    w = random_csr(M, K, N, 0.6, seed=300 + steps, values="smallint", b_dist="smallint")
    w = w if dtype == "f16" else recast(w, dtype)
    m = S.SmatMatrix(M, K, w.row_ptr, w.col_idx, w.a_bits, dtype, reorder=0, dense_tiles=1, concurrent_streams=1)
    b = torch.from_numpy(w.b_bits.view(np.int16 if es == 2 else np.uint8).reshape(K, N)).cuda()
    ref, _ = oracle_c.spmm_ref_c(M, K, N, w.row_ptr, w.col_idx, R.decode_bits(w.a_bits, dtype), R.decode_bits(w.b_bits, dtype))
    flop = 2.0 * 16 * 16 * (32 if es == 2 else 64) * 16 * 16 * 2 * steps         # two super rows, two slabs of 128 columns
    for stream, expect in ((None, "tiles+sum_tiles"), (torch.cuda.Stream(), "tiles")):
        c = torch.full((M, N), -1, dtype=torch.int32 if dtype == "i8" else torch.float32, device="cuda")
        torch.cuda.synchronize()
        S.smat_spmm(m.handle, b, c, N, stream)
        torch.cuda.synchronize()
        assert S.smat_last_launches() == (expect, flop)
        assert np.array_equal(c.cpu().numpy().astype(np.float64), ref)
    m.close()


@pytest.mark.parametrize("dtype", ["f16", "e4m3", "i8"])
@pytest.mark.parametrize("case", [(2304, 6000, 1152), (1792, 6000, 896)], ids=str)
def test_long_tiles_that_are_split_go_before_rows(case, dtype):
    """81 and 49 tiles of 94 ... 188 steps at 50 % fill, in as many parts as an XCD's compute units take at a time: 31 ... 45 us, block rows 43 ... 70."""
    M, K, N = case
    w = random_csr(M, K, 8, 0.5, seed=M, values="ones")
    w = w if dtype == "f16" else recast(w, dtype)
    m = S.SmatMatrix(w.M, w.K, w.row_ptr, w.col_idx, w.a_bits, dtype, reorder=0)
    m.spmm(torch.zeros((K, N), dtype=torch.int16 if dtype == "f16" else torch.uint8, device="cuda"))
    assert S.smat_last_launches()[0] == "tiles+sum_tiles"
    m.close()


def test_launches_of_other_products():
    w = random_csr(300, 700, 33, 0.02, seed=1, dtype="bf16")
    m = S.SmatMatrix(w.M, w.K, w.row_ptr, w.col_idx, w.a_bits, w.dtype)
    b = torch.from_numpy(w.b_bits.view(np.int16).reshape(w.K, w.N)).cuda()
    m.spmm(b)
    assert S.smat_last_launches() == ("rows", 2.0 * 16 * 16 * 32 * S.smat_get_layout_info(m.handle)["n_packs"] * 3)
    m.spmm(b[:, :0])
    assert S.smat_last_launches() == ("", 0.0)
    m.close()
    # few columns and tiles on quads; the 8-bit floats go over a step twice
    for dtype, per_step in (("bf16", 32), ("i8", 64), ("e4m3", 128)):
        w = recast(random_csr(4096, 4096, 128, 0.1, seed=2, values="smallint", b_dist="smallint"), dtype)
        m = S.SmatMatrix(w.M, w.K, w.row_ptr, w.col_idx, w.a_bits, dtype, reorder=0)
        b = torch.from_numpy(w.b_bits.view(np.int16 if dtype == "bf16" else np.uint8).reshape(w.K, w.N)).cuda()
        m.spmm(b[:, :4].contiguous())
        names, few = S.smat_last_launches()
        assert names == "quad_rows" and few % (2.0 * 16 * 16 * 16 * per_step) == 0
        m.close()
        m = S.SmatMatrix(w.M, w.K, w.row_ptr, w.col_idx, w.a_bits, dtype, reorder=0, dense_tiles=1)
        m.spmm(b)
        names, tiles = S.smat_last_launches()
        assert names.split("+")[0] == "quad_tiles" and tiles == 8 * few          # one slab of eight times sixteen columns
        m.close()
