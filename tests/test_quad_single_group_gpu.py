"""Tiles on quads with one group of waves per workgroup (wide products: more tiles than compute units), against float64 on integer values, exact: the types that have them,
the three shapes, ragged last tiles and super rows, walks of any remainder of the ring's three steps."""
import numpy as np
import pytest
import torch

import paper_2408_11551_amd as S

pytestmark = pytest.mark.gpu
TYPES = {"e4m3": torch.float8_e4m3fn, "i8": torch.int8}


def _product(M, K, N, dtype, fill, seed):
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    mask = torch.rand((M, K), device="cuda:0", generator=gen) < fill
    A = torch.randint(-2, 3, (M, K), device="cuda:0", generator=gen) * mask
    B = torch.randint(-2, 3, (K, N), device="cuda:0", generator=gen)
    rows, cols = mask.nonzero(as_tuple=True)
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum(mask.sum(1).cpu().numpy(), out=row_ptr[1:])
    bits = torch.int16 if TYPES[dtype].itemsize == 2 else torch.uint8
    vals = A[rows, cols].to(TYPES[dtype]).view(bits).cpu().numpy()
    m = S.SmatMatrix(M, K, row_ptr, cols.to(torch.int32).cpu().numpy(), vals.view(np.uint16 if bits == torch.int16 else np.uint8), dtype, device="cuda:0")
    C = m.spmm(B.to(TYPES[dtype]).view(bits))
    name = S.smat_last_kernel()
    assert torch.equal(C.double(), A.double() @ B.double()), name
    m.close()
    return name


# (dtype, columns of a tile, M, K, N): by what the estimates choose
CASES = [("e4m3", 128, 3484, 3387, 3561), ("e4m3", 96, 3075, 2477, 2912), ("i8", 128, 4378, 4422, 3295), ("i8", 128, 3247, 2257, 2816),
         ("i8", 128, 4696, 3919, 2371), ("i8", 64, 6012, 1316, 883)]


@pytest.mark.parametrize("dtype,columns,M,K,N", CASES)
def test_wide_products(dtype, columns, M, K, N):
    name = _product(M, K, N, dtype, 0.1, M + N)
    assert name.replace("_staged", "") == f"spmm_dense_{dtype}_g1_256x{columns}", name


@pytest.mark.parametrize("dtype", ["e4m3", "i8"])
@pytest.mark.parametrize("K", [2050, 2180, 2300, 2450, 2600, 2700])
def test_every_remainder_of_the_ring(dtype, K):
    assert "_g1" in _product(4500, K, 2500 + K % 7, dtype, 0.1, K)
