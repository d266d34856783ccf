"""What a user of this library has it do, as cases that can be timed.

Two kinds of work.  "spmm": a matrix has been preprocessed and bound once, and C = A B is called
again and again with dense operands that change (`SmatMatrix.spmm`).  "set_up": a matrix is new --
a sampled subgraph, weights pruned anew -- so preprocessing, bind and the first product are what
the user waits for.

The sparse matrices are those of the library's workloads: uniformly random, a power-law graph, a
band, dense 16 x 16 blocks hidden by row and column permutations, and a pruned weight matrix.  They
are generated here on the GPU from the seed alone, so that a new one is quick to make.

    family        parameters
    uniform       M = K, `per_row` entries per row on average
    powerlaw      M = K, row degrees d with P(d) ~ d^-1.2 and mean `per_row`, random columns
    banded        M = K, entry (i, j) with |i - j| <= `half` stored with probability `fill`, diagonal always
    hidden        M = K = 16 * `grid`, each 16 x 16 block stored with probability `fill`, then scrambled
    pruned        M x K, each entry stored with probability `fill`
"""
import math

import numpy as np
import torch

import paper_2408_11551_amd as smat

DEVICE = "cuda:0"
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2}
BYTES = {"f16": 2, "bf16": 2, "e4m3": 1, "e5m2": 1, "i8": 1}


def _case(name, family, dtype, N, **kw):
    case = {"name": name, "kind": "spmm", "family": family, "dtype": dtype, "N": N, "ldb": N, "reorder": 1, "per_row": 0.0,
            "half": 0, "fill": 0.0, "grid": 0, "M": 0, "K": 0}
    case.update(kw)
    if family == "hidden":
        case["M"] = 16 * case["grid"]
    case["K"] = case["K"] or case["M"]
    return case


def listed():
    return [
        # the smallest call: a product inside somebody's inner loop, latency and host path only
        _case("tiny", "pruned", "f16", 64, M=1024, fill=0.01),
        # one layer of a graph network on a random graph: features of 128
        _case("uniform_n128", "uniform", "f16", 128, M=16384, per_row=16.4),
        # a large graph with few vectors (ranking, label propagation); nothing to regroup in it, so reordering is off
        _case("powerlaw_n8", "powerlaw", "f16", 8, M=262144, per_row=16.0, reorder=0),
        # the same kind of graph with input features of a length that is nobody's power of two
        _case("powerlaw_n100", "powerlaw", "bf16", 100, M=100003, per_row=16.0),
        # a discretised operator applied to a wide block of vectors
        _case("banded_n256", "banded", "f16", 256, M=65536, half=64, fill=0.3),
        # the same with an odd number of right-hand sides and an odd size
        _case("banded_n33", "banded", "bf16", 33, M=50021, half=32, fill=0.6),
        # block structure hidden by permutations, which the row reordering finds (the benchmark's default workload)
        _case("hidden_n256", "hidden", "f16", 256, grid=2048, fill=0.02),
        # and the widest B the method is usually quoted with, whose rows do not fill cache lines: the largest case
        _case("hidden_n1000", "hidden", "f16", 1000, grid=2048, fill=0.02),
        # pruned weights: a long prompt (prefill), a batch of four tokens (decode), a ragged batch in 8-bit floats
        _case("pruned_n2048", "pruned", "bf16", 2048, M=4096, fill=0.1),
        _case("pruned_n4", "pruned", "i8", 4, M=8192, K=4096, fill=0.1),
        _case("pruned_n777", "pruned", "e4m3", 777, M=6000, K=4096, fill=0.1),
        # a graph seen for the first time: clustering, layout, upload and one product
        _case("set_up", "powerlaw", "f16", 64, kind="set_up", M=65536, per_row=16.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["uniform", "powerlaw", "banded", "hidden", "pruned", "pruned"])
    dtype = rng.choice(["f16", "f16", "f16", "bf16", "bf16", "e4m3", "e4m3", "e5m2", "i8", "i8"])
    kind = "set_up" if rng.random() < 0.1 else "spmm"
    small = kind == "set_up"                       # a set-up stays below the listed one's cost
    kw = {"kind": kind}
    if family == "uniform":
        kw.update(M=_log_int(rng, 1024, 16384 if small else 65536), per_row=round(math.exp(rng.uniform(math.log(4), math.log(64))), 1))
        nnz = kw["M"] * kw["per_row"]
    elif family == "powerlaw":
        kw.update(M=_log_int(rng, 16384, 65536 if small else 262144), per_row=16.0)
        kw["reorder"] = 0 if kw["M"] > 131072 else rng.choice([0, 1, 1])
        nnz = kw["M"] * kw["per_row"]
    elif family == "banded":
        kw.update(M=_log_int(rng, 4096, 16384 if small else 65536), half=_log_int(rng, 8, 128), fill=rng.choice([0.3, 0.6, 1.0]))
        nnz = kw["M"] * (2 * kw["half"] + 1) * kw["fill"]
    elif family == "hidden":
        kw.update(grid=_log_int(rng, 128, 512 if small else 2048), fill=0.02)
        nnz = 256.0 * kw["fill"] * kw["grid"] ** 2
        kw["M"] = 16 * kw["grid"]
    else:
        top = 3000 if small else 8192
        kw.update(M=_log_int(rng, 1000, top), K=_log_int(rng, 1000, top), fill=rng.choice([0.05, 0.1, 0.2]))
        nnz = kw["M"] * kw["K"] * kw["fill"]
    # one column to thousands, within the largest listed product and the largest listed B and C together
    most = min(4096.0, 2.1e10 / nnz, 2.1e8 / (6.0 * max(kw["M"], kw.get("K", 0))))
    N = _log_int(rng, 1, max(1.0, most))
    step = rng.choice([1, 1, 8, 32])               # half of the widths as they come, half rounded as users pad them
    N = max(1, N // step * step)
    case = _case("", family, dtype, N, **kw)
    if rng.random() < 0.15:
        case["ldb"] = N + rng.choice([1, 8, 24])   # B is a slice of a wider array
    del case["name"]
    return case


def _degrees(M, mean, gen):
    """Degrees d = 1 .. d_max with P(d) ~ d^-1.2, d_max the first for which the mean is reached."""
    d = torch.arange(1, 4097, dtype=torch.float64)
    p = d ** -1.2
    means = torch.cumsum(d * p, 0) / torch.cumsum(p, 0)
    top = int(torch.nonzero(means >= mean)[0]) + 1
    cdf = torch.cumsum(p[:top], 0)
    cdf = (cdf / cdf[-1]).to(DEVICE)
    u = torch.rand(M, dtype=torch.float64, device=DEVICE, generator=gen)
    return torch.searchsorted(cdf, u).clamp_(max=top - 1) + 1


def _pattern(case, gen):
    """(rows, columns) of the stored entries, by row and then by column (int64, on the GPU)."""
    M, K, family = case["M"], case["K"], case["family"]
    if family == "pruned":
        mask = torch.rand((M, K), device=DEVICE, generator=gen) < case["fill"]
        return mask.nonzero(as_tuple=True)
    if family == "banded":
        half = case["half"]
        mask = torch.rand((M, 2 * half + 1), device=DEVICE, generator=gen) < case["fill"]
        mask[:, half] = True
        i, d = mask.nonzero(as_tuple=True)
        j = i + d - half
        ok = (j >= 0) & (j < K)
        return i[ok], j[ok]
    if family == "uniform":
        keys = torch.randint(0, M * K, (int(round(M * case["per_row"])),), device=DEVICE, generator=gen)
    elif family == "powerlaw":
        rows = torch.repeat_interleave(torch.arange(M, device=DEVICE), _degrees(M, case["per_row"], gen))
        keys = rows * K + torch.randint(0, K, rows.shape, device=DEVICE, generator=gen)
    else:
        bi, bj = (torch.rand((case["grid"], case["grid"]), device=DEVICE, generator=gen) < case["fill"]).nonzero(as_tuple=True)
        new_row = torch.randperm(M, device=DEVICE, generator=gen)
        new_col = torch.randperm(K, device=DEVICE, generator=gen)
        lane = torch.arange(16, device=DEVICE)
        r, c = new_row[bi[:, None] * 16 + lane], new_col[bj[:, None] * 16 + lane]
        keys = (r[:, :, None] * K + c[:, None, :]).reshape(-1)
    keys = torch.unique(keys)
    return keys // K, keys % K


def _values(shape, dtype, gen, scale):
    """Normal values of the type: activations, weights, features."""
    x = torch.randn(shape, device=DEVICE, generator=gen) * scale
    if dtype == "i8":
        return (x * (40.0 / scale)).round_().clamp_(-127, 127).to(torch.int8)
    return x.to(DTYPES[dtype])


def _bits(t):
    return t.view(torch.int16 if t.element_size() == 2 else torch.uint8)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed) * 1000003 + 17)
    M, K, N, dtype = case["M"], case["K"], case["N"], case["dtype"]
    rows, cols = _pattern(case, gen)
    row_ptr = np.zeros(M + 1, dtype=np.int64)
    np.cumsum(torch.bincount(rows, minlength=M).cpu().numpy(), out=row_ptr[1:])
    vals = _bits(_values(rows.shape, dtype, gen, 0.25)).cpu().numpy()
    vals = vals.view(np.uint16 if vals.itemsize == 2 else np.uint8)
    csr = (M, K, row_ptr, cols.to(torch.int32).cpu().numpy(), vals, dtype)
    B = _bits(_values((K, case["ldb"]), dtype, gen, 1.0))[:, :N]
    if case["kind"] == "set_up":
        return {"csr": csr, "reorder": case["reorder"], "B": B}
    return {"A": smat.SmatMatrix(*csr, reorder=case["reorder"], device=DEVICE), "B": B}


def run(state):
    if "A" in state:
        return state["A"].spmm(state["B"])
    A = smat.SmatMatrix(*state["csr"], reorder=state["reorder"], device=DEVICE)
    C = A.spmm(state["B"])
    order = smat.smat_export_perm(A.handle, A.M)
    # the workspace is given back in stream order, so the product may still be running
    A.close()
    return {"C": C, "order": order}


def _entries(case):
    M, K, family = case["M"], case["K"], case["family"]
    if family in ("uniform", "powerlaw"):
        return M * case["per_row"]
    if family == "banded":
        return M * (2 * case["half"] * case["fill"] + 1)
    if family == "hidden":
        return 256.0 * case["fill"] * case["grid"] ** 2
    return M * K * case["fill"]


def work(case):
    """A once as CSR (values, columns, row offsets), B once, C once; a multiply-add per entry and column."""
    nnz, es, N = _entries(case), BYTES[case["dtype"]], case["N"]
    return {"bytes": nnz * (es + 4) + (case["M"] + 1) * 8 + case["K"] * N * es + case["M"] * N * 4.0, "flops": 2.0 * nnz * N}


def tolerance(case):
    # 8-bit integers are summed in 32-bit integers; the floating types multiply exactly and add in fp32
    return "exact" if case["dtype"] == "i8" else {"rel": 1e-5}
