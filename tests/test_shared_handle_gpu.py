"""One handle shared by threads, streams and graphs on products that copy B first or keep partial tiles: every product reads its own
B.  Small integers: all results are exact and compared bit for bit."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2408_11551_amd as S            # noqa: E402
from workloads import random_csr            # noqa: E402

# the per-row kernel and the tile kernel on a copy of B (rows of B off the cache lines, off 16-byte pieces); split tiles
CASES = {"rows": (2048, 8200, 519, 0.02, -1), "tiles": (512, 4112, 1101, 0.12, 1), "split": (512, 1100, 264, 0.12, 1)}


def _case(kind, streams=2):
    M, K, N, density, dense_tiles = CASES[kind]
    w = random_csr(M, K, N, density, seed=M, values="smallint", b_dist="smallint")
    m = S.SmatMatrix(w.M, w.K, w.row_ptr, w.col_idx, w.a_bits, w.dtype, reorder=0, dense_tiles=dense_tiles, concurrent_streams=streams)
    one = torch.from_numpy(w.b_bits.view(np.int16).reshape(K, N)).cuda()
    bs = [one, one.flip(0).contiguous()]
    a = torch.zeros((M, K), dtype=torch.float64, device="cuda")
    a[torch.repeat_interleave(torch.arange(M), torch.from_numpy(np.diff(w.row_ptr))).cuda(), torch.from_numpy(w.col_idx).long().cuda()] = \
        torch.from_numpy(w.a_bits.view(np.float16).astype(np.float64)).cuda()
    refs = [(a @ b.view(torch.float16).double()).float() for b in bs]
    torch.cuda.synchronize()
    return m, bs, refs


@pytest.mark.parametrize("kind", list(CASES))
def test_two_threads_on_one_stream(kind):
    m, bs, refs = _case(kind)
    cs = [[torch.full_like(refs[t], float("nan")) for _ in range(20)] for t in range(2)]
    start = threading.Barrier(2)

    def work(t):
        start.wait()
        for c in cs[t]:
            S.smat_spmm(m.handle, bs[t], c)
    threads = [threading.Thread(target=work, args=(t,)) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for t in range(2):
        for c in cs[t]:
            assert torch.equal(c, refs[t])
    m.close()


@pytest.mark.parametrize("kind", list(CASES))
def test_per_thread_stream_goes_without_an_area(kind):
    m, bs, refs = _case(kind)
    c = torch.full_like(refs[0], float("nan"))
    torch.cuda.synchronize()
    S.smat_spmm(m.handle, bs[0], c, None, 2)                     # hipStreamPerThread
    name = S.smat_last_kernel()
    torch.cuda.synchronize()
    assert "_staged" not in name and not name.split("+")[0].endswith(("k2", "k4", "k8")), name
    assert torch.equal(c, refs[0])
    m.close()


@pytest.mark.parametrize("kind", list(CASES))
def test_graphs_of_one_stream_replayed_on_others(kind):
    """Two graphs captured on one stream run at the same time on two streams, beside calls on a third: three areas for the default
    stream and the two captures."""
    m, bs, refs = _case(kind, streams=3)
    cs = [torch.full_like(refs[t], float("nan")) for t in range(2)]
    eager = torch.full_like(refs[0], float("nan"))
    S.smat_spmm(m.handle, bs[0], eager)
    name = S.smat_last_kernel()
    torch.cuda.synchronize()
    side, graphs = torch.cuda.Stream(), []
    for t in range(2):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            S.smat_spmm(m.handle, bs[t], cs[t])
        assert S.smat_last_kernel() == name
        graphs.append(g)
    others = [torch.cuda.Stream() for _ in range(2)]
    for rep in range(5):
        for c in (*cs, eager):
            c.fill_(float("nan"))
        torch.cuda.synchronize()
        for t in range(2):
            with torch.cuda.stream(others[t]):
                graphs[t].replay()
        S.smat_spmm(m.handle, bs[1], eager)
        torch.cuda.synchronize()
        assert torch.equal(cs[0], refs[0]) and torch.equal(cs[1], refs[1]) and torch.equal(eager, refs[1]), rep
    m.close()
