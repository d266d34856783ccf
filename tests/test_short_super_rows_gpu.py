"""Super rows of few steps on quads (K of a few hundred to 2000), chosen by estimate: against float64 on integer values, exact; the same call with the static area, and
what tiles that are asked for run on."""
import numpy as np
import pytest
import torch

import paper_2408_11551_amd as S

pytestmark = pytest.mark.gpu
TYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2, "i8": torch.int8}


def _matrix(M, K, dtype, fill, seed, **kw):
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    mask = torch.rand((M, K), device="cuda:0", generator=gen) < fill
    A = torch.randint(-2, 3, (M, K), device="cuda:0", generator=gen) * mask
    rows, cols = mask.nonzero(as_tuple=True)
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum(mask.sum(1).cpu().numpy(), out=row_ptr[1:])
    bits = torch.int16 if TYPES[dtype].itemsize == 2 else torch.uint8
    vals = A[rows, cols].to(TYPES[dtype]).view(bits).cpu().numpy().view(np.uint16 if bits == torch.int16 else np.uint8)
    return A, S.SmatMatrix(M, K, row_ptr, cols.to(torch.int32).cpu().numpy(), vals, dtype, device="cuda:0", **kw)


def _check(A, m, N, ldb, seed):
    dtype = TYPES[m.dtype]
    B = torch.randint(-2, 3, (m.K, ldb), device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(seed))
    bits = B.to(dtype).view(torch.int16 if dtype.itemsize == 2 else torch.uint8)[:, :N]
    want = A.double() @ B[:, :N].double()
    assert torch.equal(m.spmm(bits).double(), want), S.smat_last_kernel()
    launches = S.smat_last_launches()[0]
    C = torch.empty((m.M, N), dtype=torch.int32 if m.dtype == "i8" else torch.float32, device="cuda:0")
    try:
        S.smat_spmm_static(m.handle, bits, C)
        assert torch.equal(C.double(), want), S.smat_last_kernel()
    except S.SmatError as e:          # its partial tiles exceed the static area (smat.h)
        assert e.status_name == "SMAT_ERR_UNSUPPORTED"
    return launches


@pytest.mark.parametrize("dtype", list(TYPES))
@pytest.mark.parametrize("K", [270, 513, 800, 1024, 1500, 2000])
def test_products(K, dtype):
    taken = set()
    for M, fill in ((4003, 0.1), (2570, 0.2)):
        A, m = _matrix(M, K, dtype, fill, K + M)
        for N, ldb in ((33, 33), (160, 160), (333, 334), (640, 640), (1200, 1201)):
            taken.update(_check(A, m, N, ldb, N).split("+"))
        m.close()
    assert "quad_tiles" in taken, taken


@pytest.mark.parametrize("dtype", ["f16", "e4m3", "i8"])
def test_tiles_that_are_asked_for_stay_without_quads(dtype):
    A, m = _matrix(1000, 700, dtype, 0.1, 1, dense_tiles=1)
    assert "tiles" in _check(A, m, 128, 128, 2).split("+")
    m.close()


@pytest.mark.parametrize("dtype,M,K,fill,N", [("e5m2", 6298, 1353, 0.2, 794), ("e4m3", 4997, 528, 0.05, 1184), ("f16", 8083, 853, 0.2, 751), ("i8", 6486, 973, 0.2, 736)])
def test_the_static_call_takes_the_shape_of_any_other(dtype, M, K, fill, N):
    A, m = _matrix(M, K, dtype, fill, M)
    _check(A, m, N, N, N)
    with_static_area = S.smat_last_kernel()
    m.spmm(torch.zeros((K, N), dtype=torch.int16 if TYPES[dtype].itemsize == 2 else torch.uint8, device="cuda:0"))
    # (not 256 x 128 in two groups, whose name has no shape in it)
    assert with_static_area == S.smat_last_kernel() and "x" in with_static_area, with_static_area
    m.close()
