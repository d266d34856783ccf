"""The search for rows that could start a cluster together, on the device: its pairs against brute force on dense patterns, and the handle that it helps to
make against the one that the host makes alone."""
import numpy as np
import pytest
import torch

import paper_2408_11551_amd as S

pytestmark = pytest.mark.gpu


def _patterns(n, nbc, lengths, seed, families):
    """n distinct patterns in the order of their lengths; `families`: that many of the patterns are others with a few columns changed."""
    rng = np.random.default_rng(seed)
    lists = []
    for i in range(n):
        if lists and rng.random() < families:
            src = lists[rng.integers(0, len(lists))]
            cols = np.union1d(src[rng.random(src.size) < 0.8], rng.integers(0, nbc, 1 + src.size // 8))
        else:
            cols = np.unique(rng.integers(0, nbc, rng.choice(lengths)))
        lists.append(cols)
    lists = sorted({tuple(x) for x in lists if len(x)}, key=lambda x: (len(x), x))
    ptr = np.zeros(len(lists) + 1, np.uint32)
    np.cumsum([len(x) for x in lists], out=ptr[1:])
    return ptr, np.concatenate([np.array(x, np.uint32) for x in lists])


def _brute(ptr, columns, nbc, keep):
    n, lens = ptr.size - 1, np.diff(ptr).astype(np.int64)
    dense = torch.zeros((n, nbc), dtype=torch.float32)
    dense[torch.from_numpy(np.repeat(np.arange(n), lens)), torch.from_numpy(columns.astype(np.int64))] = 1.0
    want = []
    for k0 in range(0, n, 512):
        shared = (dense[k0:k0 + 512] @ dense.t()).numpy().astype(np.int64)         # (counts: exact in fp32)
        union = lens[k0:k0 + 512, None] + lens[None, :] - shared
        a, b = np.nonzero(1000 * shared > keep * union)
        want.append(np.stack([a + k0, b], 1)[a + k0 < b])
    return np.concatenate(want)


# one and two columns; on both sides of the 32 columns up to which a wave takes a pattern, and of the 255 that a byte counts; a column with thousands of
# patterns; more patterns than the counters of a workgroup (65536 bytes, 32768 halves)
@pytest.mark.parametrize("n,nbc,lengths,families", [
    (1, 5, [3], 0), (2, 5, [2], 0), (3000, 4000, [1, 2, 3], 0.2), (3000, 300, [30, 31, 32, 33, 34, 40], 0.3),
    (2000, 4000, [200, 250, 255, 256, 300], 0.5), (1500, 9000, [1, 2, 31, 33, 600, 700], 0.4), (4000, 40, [4, 5], 0.0), (3000, 64, [2, 40], 0.0)])
@pytest.mark.parametrize("keep", [300, 700, 1])
def test_pairs_are_those_of_brute_force(n, nbc, lengths, families, keep):
    ptr, columns = _patterns(n, nbc, lengths, n + nbc, families)
    want = _brute(ptr, columns, nbc, keep)
    scratch = torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0")
    # (what the kernels hold of a pattern that is the shorter one: 128 pairs up to 32 columns, where a wave takes it, else 512)
    partners, lens = np.bincount(want[:, 0], minlength=ptr.size - 1), np.diff(ptr)
    try:
        got = S.smat_pattern_partners(ptr, columns, nbc, keep, scratch, want.shape[0] + 1)
    except S.SmatError as e:
        assert e.status_name == "SMAT_ERR_UNSUPPORTED" and (partners[lens <= 32].max(initial=0) > 128 or partners[lens > 32].max(initial=0) > 512)
        return
    assert partners.max(initial=0) <= 512
    assert got.shape == want.shape and np.array_equal(got[np.lexsort((got[:, 1], got[:, 0]))], want)


# A pattern with as many partners as the kernels hold of one, taken by a wave or a workgroup that holds as many of another already; and one more
@pytest.mark.parametrize("length,together,held,most,keep", [(8, 8192, 63, 128, 850), (40, 768, 255, 512, 960)])
@pytest.mark.parametrize("one_more", [0, 1])
def test_most_partners_of_a_pattern(length, together, held, most, keep, one_more):
    # `together` patterns on, the same wave or workgroup comes by; a partner has the pattern's columns and one more
    partners = np.zeros(together + 8, np.int64)
    partners[:8], partners[together:] = most, held
    partners[3] += one_more
    n_bases, n_more = partners.size, int(partners.sum())
    base = np.arange(n_bases * length).reshape(n_bases, length)
    more = np.concatenate([base[np.repeat(np.arange(n_bases), partners)], n_bases * length + np.arange(n_more)[:, None]], axis=1)
    ptr = np.concatenate([np.arange(n_bases + 1) * length, n_bases * length + (length + 1) * np.arange(1, n_more + 1)]).astype(np.uint32)
    columns = np.concatenate([base.reshape(-1), more.reshape(-1)]).astype(np.uint32)
    want = np.stack([np.repeat(np.arange(n_bases), partners), n_bases + np.arange(n_more)], axis=1)
    scratch = torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0")
    if one_more:
        with pytest.raises(S.SmatError, match="UNSUPPORTED"):
            S.smat_pattern_partners(ptr, columns, n_bases * length + n_more, keep, scratch, n_more)
    else:
        got = S.smat_pattern_partners(ptr, columns, n_bases * length + n_more, keep, scratch, n_more)
        assert np.array_equal(got[np.lexsort((got[:, 1], got[:, 0]))], want)


# Lists so long that many short patterns reach the bound by accident: more counters (keep = 700, and fewer patterns than these), or none but exact ones
@pytest.mark.parametrize("n,nbc,lengths,keep", [(9000, 52, [9, 10, 11], 300), (9000, 52, [9, 10, 11], 700), (8150, 48, [9, 10, 11], 360), (3000, 80, [20, 31, 40], 400)])
def test_pairs_where_columns_have_long_lists(n, nbc, lengths, keep):
    ptr, columns = _patterns(n, nbc, lengths, n + keep, 0.05)
    want = _brute(ptr, columns, nbc, keep)
    got = S.smat_pattern_partners(ptr, columns, nbc, keep, torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0"), want.shape[0] + 1)
    assert got.shape == want.shape and np.array_equal(got[np.lexsort((got[:, 1], got[:, 0]))], want)


@pytest.mark.parametrize("per_row", [34, 300])
def test_more_patterns_than_a_workgroup_counts_at_a_time(per_row):
    """70 000 patterns beyond the short ones, in bytes and in halves; checked on the pairs that were planted, and that every pair found is one."""
    n, nbc = 70000, 1000000
    rng = np.random.default_rng(per_row)
    base = np.sort(rng.integers(0, nbc, (n, per_row)), axis=1)
    base[1::1000] = base[0::1000]                    # a partner for every thousandth ...
    base[1::1000, 0] = rng.integers(0, 1000, n // 1000)      # ... with another first column
    lists = sorted({tuple(np.unique(x)) for x in base}, key=lambda x: (len(x), x))
    ptr = np.zeros(len(lists) + 1, np.uint32)
    np.cumsum([len(x) for x in lists], out=ptr[1:])
    columns = np.concatenate([np.array(x, np.uint32) for x in lists])
    scratch = torch.empty(512 << 20, dtype=torch.uint8, device="cuda:0")
    got = S.smat_pattern_partners(ptr, columns, nbc, 300, scratch, n)
    for a, b in got:
        shared = len(set(lists[a]) & set(lists[b]))
        assert a < b and 1000 * shared > 300 * (len(lists[a]) + len(lists[b]) - shared)
    where = {x: i for i, x in enumerate(lists)}
    planted = {tuple(sorted((where[tuple(np.unique(base[i]))], where[tuple(np.unique(base[i + 1]))]))) for i in range(0, n, 1000)}
    assert {p for p in planted if p[0] != p[1]} <= {tuple(p) for p in got}


def _graph(M, K, per_row, seed):
    rng = np.random.default_rng(seed)
    deg = np.minimum(rng.zipf(1.6, M), 40 * per_row)
    deg = np.maximum(1, (deg * (per_row / deg.mean())).astype(np.int64))
    keys = np.unique(np.repeat(np.arange(M), deg) * K + rng.integers(0, K, deg.sum()))
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum(np.bincount(keys // K, minlength=M), out=row_ptr[1:])
    return row_ptr, (keys % K).astype(np.int32)


def _pattern_table(M, row_ptr, col_idx):
    """What the clustering sends to the device: every row pattern once, by length."""
    rows = np.repeat(np.arange(M), np.diff(row_ptr))
    keys = np.unique(rows * (1 << 24) + col_idx // 16)
    cols = (keys % (1 << 24)).astype(np.uint32)
    ends = np.searchsorted(keys, np.arange(M + 1) * (1 << 24))
    lists = sorted({cols[a:b].tobytes() for a, b in zip(ends[:-1], ends[1:])}, key=len)
    ptr = np.zeros(len(lists) + 1, np.uint32)
    np.cumsum([len(x) // 4 for x in lists], out=ptr[1:])
    return ptr, np.frombuffer(b"".join(lists), np.uint32)


# (searched: on the device with any number of threads; with sixteen the others may be the threads' own)
@pytest.mark.parametrize("M,K,per_row,tau,searched", [(40000, 40000, 12, 700, True), (30001, 9000, 20, 500, True), (60000, 60000, 20, 900, True), (30000, 60000, 40, 700, True),
                                                      (20000, 300000, 30, 900, False), (16000, 16000, 60, 700, False)])
def test_the_handle_is_the_hosts(M, K, per_row, tau, searched):
    row_ptr, col_idx = _graph(M, K, per_row, M + tau)
    args = (M, K, row_ptr, col_idx, np.ones(col_idx.size, np.uint16), "f16")
    alone = S.smat_preprocess(*args, tau_permille=tau)
    before = torch.cuda.memory_stats().get("allocation.all.allocated", 0)
    helped = S.smat_preprocess_on_device(*args, device="cuda:0", tau_permille=tau)
    if searched:
        # it asked for memory, and these patterns are none that the search declines
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before + 1
        ptr, columns = _pattern_table(M, row_ptr, col_idx)
        S.smat_pattern_partners(ptr, columns, (K + 15) // 16, 1000 - tau, torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0"), 4 << 20)
    assert np.array_equal(S.smat_export_perm(alone, M), S.smat_export_perm(helped, M))
    for a, b in zip(S.smat_export_bcsr(alone, with_vals=False)[:2], S.smat_export_bcsr(helped, with_vals=False)[:2]):
        assert np.array_equal(a, b)
    S.smat_destroy(alone)
    S.smat_destroy(helped)


def test_memory_is_asked_for_only_where_the_search_pays():
    """A band's rows join their clusters, so nothing is looked for: its set-up takes no memory of the device."""
    M, half = 20000, 16
    rows = np.repeat(np.arange(M), 2 * half + 1)
    cols = rows + np.tile(np.arange(-half, half + 1), M)
    ok = (cols >= 0) & (cols < M)
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum(np.bincount(rows[ok], minlength=M), out=row_ptr[1:])
    before = torch.cuda.memory_stats().get("allocation.all.allocated", 0)
    band = S.smat_preprocess_on_device(M, M, row_ptr, cols[ok].astype(np.int32), np.ones(ok.sum(), np.uint16), "f16", device="cuda:0")
    assert torch.cuda.memory_stats().get("allocation.all.allocated", 0) == before
    S.smat_destroy(band)
    row_ptr, col_idx = _graph(40000, 40000, 12, 1)
    graph = S.smat_preprocess_on_device(40000, 40000, row_ptr, col_idx, np.ones(col_idx.size, np.uint16), "f16", device="cuda:0")
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before + 1
    S.smat_destroy(graph)
