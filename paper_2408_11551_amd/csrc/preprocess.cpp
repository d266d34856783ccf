// Host-side preprocessing for the blocked SpMM: see preprocess.h.
//
// The clustering follows the greedy procedure of the paper's Preprocessing
// section (open a cluster with an unclustered row; every other unclustered row
// whose Jaccard distance to the cluster's column union is below the threshold
// is merged).  A row can only pass the test if it shares a block column with
// the union as it stands when the row is reached, so instead of looking at
// every row the scan walks an ascending candidate set fed from an inverted
// index (block column -> rows): when a column enters the union, every later
// unclustered row holding it becomes a candidate and its intersection counter
// goes up by one.  The counter a row carries when the scan reaches it is then
// exactly |row n union|, and rows that never became candidates have an empty
// intersection and could not have merged.  The result is the same permutation
// the row-by-row scan gives.  (The index and the counters are kept per distinct
// row pattern, not per row: rows with the same pattern have the same counter.)
//
// Most seeds of a graph or a uniformly random matrix end up alone, and finding that out by counting is nearly all the
// time there is.  Whether a pattern can merge with any other at all is a question about pairs, not about the
// state of the scan, so once the scan has shown that the clusters stay small it is answered for all remaining
// patterns at once, on several threads (partners_of); seeds without a partner are then placed without counting.
#include "preprocess.h"

#include <algorithm>
#include <cmath>
#include <limits>
#include <memory>
#include <numeric>

namespace smat {

// Rows per piece of a loop over rows that costs by the entry: as many as hold some ten thousand, but one piece for every thread (which finds
// what it has read in its caches when it comes to its rows again: 21.5 million entries, 4.0 ms for their patterns, 9.6 in pieces of 25 rows), and not too many.
static int64_t row_grain(int64_t M, int64_t entries, int64_t most, const Workers& workers)
{
    const int64_t share = (M + workers.most() - 1) / workers.most();
    return std::clamp<int64_t>(entries > 0 ? std::max(M * 16384 / entries, share) : most, 1, most);
}

std::string validate_csr(int64_t M, int64_t K, const int64_t* row_ptr, const int32_t* col_idx, Workers& workers)
{
    std::atomic<int64_t> first_bad{M};
    auto fault = [&](int64_t r) -> const char* {
        int64_t prev = -1;
        for (int64_t p = row_ptr[r]; p < row_ptr[r + 1]; ++p) {
            const int64_t c = col_idx[p];
            if (c < 0 || c >= K) return "column out of range in row ";
            if (c <= prev) return "columns not strictly ascending in row ";
            prev = c;
        }
        return nullptr;
    };
    workers.ranges(M, row_grain(M, row_ptr[M], 4096, workers), [&](int64_t r0, int64_t r1, int) {
        for (int64_t r = r0; r < r1; ++r)
            if (fault(r)) {
                int64_t seen = first_bad.load();
                while (r < seen && !first_bad.compare_exchange_weak(seen, r)) {}
                return;
            }
    });
    const int64_t r = first_bad.load();
    return r < M ? fault(r) + std::to_string(r) : std::string();
}

// Prefix sums in place: ptr[0] = 0, ptr[i + 1] holds the count of item i on entry.
template <typename P>
static void prefix_sums(P& ptr)
{
    for (size_t i = 1; i < ptr.size(); ++i) ptr[i] += ptr[i - 1];
}

void block_patterns(const Csr& a, Patterns& pat, Workers& workers)
{
    pat.ptr.resize(static_cast<size_t>(a.M) + 1);
    pat.ptr[0] = 0;
    auto walk = [&](int64_t r, int32_t* out) {
        int32_t last = -1;
        int64_t n = 0;
        for (int64_t p = a.row_ptr[r]; p < a.row_ptr[r + 1]; ++p) {
            const int32_t bc = a.col_idx[p] / kBlock;     // columns ascend, so block columns do too
            if (bc != last) {
                if (out) out[n] = bc;
                ++n;
                last = bc;
            }
        }
        return n;
    };
    const int64_t grain = row_grain(a.M, a.row_ptr[a.M], 2048, workers);
    workers.ranges(a.M, grain, [&](int64_t r0, int64_t r1, int) {
        for (int64_t r = r0; r < r1; ++r) pat.ptr[r + 1] = walk(r, nullptr);
    });
    prefix_sums(pat.ptr);
    pat.idx.resize(static_cast<size_t>(pat.ptr[a.M]));
    workers.ranges(a.M, grain, [&](int64_t r0, int64_t r1, int) {
        for (int64_t r = r0; r < r1; ++r) walk(r, pat.idx.data() + pat.ptr[r]);
    });
}

namespace {

// Set of row indices that supports "insert" and "smallest member >= from", three
// levels of 64-way summary bits.
class AscendingSet {
public:
    explicit AscendingSet(int64_t n) : n_(n)
    {
        n0_ = (n + 63) / 64; n1_ = (n0_ + 63) / 64; n2_ = (n1_ + 63) / 64;
        l0_.assign(n0_ + 1, 0); l1_.assign(n1_ + 1, 0); l2_.assign(n2_ + 1, 0);
    }
    void insert(int64_t i)
    {
        l0_[i >> 6] |= 1ull << (i & 63);
        l1_[i >> 12] |= 1ull << ((i >> 6) & 63);
        l2_[i >> 18] |= 1ull << ((i >> 12) & 63);
    }
    void erase(int64_t i)
    {
        if ((l0_[i >> 6] &= ~(1ull << (i & 63))) == 0)
            if ((l1_[i >> 12] &= ~(1ull << ((i >> 6) & 63))) == 0)
                l2_[i >> 18] &= ~(1ull << ((i >> 12) & 63));
    }
    // smallest member >= from, or -1
    int64_t next(int64_t from) const
    {
        if (from >= n_) return -1;
        int64_t w0 = from >> 6;
        uint64_t bits = l0_[w0] & (~0ull << (from & 63));
        if (bits) return (w0 << 6) + __builtin_ctzll(bits);
        const int64_t i1 = w0 + 1;                       // first level-0 word still to look at
        if (i1 >= n0_) return -1;
        int64_t w1 = i1 >> 6;
        bits = l1_[w1] & (~0ull << (i1 & 63));
        if (!bits) {
            const int64_t i2 = w1 + 1;                   // first level-1 word still to look at
            if (i2 >= n1_) return -1;
            int64_t w2 = i2 >> 6;
            uint64_t b2 = l2_[w2] & (~0ull << (i2 & 63));
            while (!b2) {
                if (++w2 >= n2_) return -1;
                b2 = l2_[w2];
            }
            w1 = (w2 << 6) + __builtin_ctzll(b2);
            bits = l1_[w1];
        }
        w0 = (w1 << 6) + __builtin_ctzll(bits);
        return (w0 << 6) + __builtin_ctzll(l0_[w0]);
    }
private:
    int64_t n_, n0_, n1_, n2_;
    std::vector<uint64_t> l0_, l1_, l2_;
};

}  // namespace

// Rows with the same pattern (the sixteen rows of a dense block row, the degrees of freedom of
// one mesh node) have the same intersection with any union, so the counting is done once per
// distinct pattern ("class"), not once per row: the inverted index lists classes, and a class
// whose count makes it a candidate puts all its unclustered rows ahead of the scan into the
// candidate set.  Classes are numbered by the length of their pattern, then by their first row.
struct PatternClasses {
    Buf<int32_t> class_of;             // [M]
    Buf<int32_t> first_row;            // [n] the first row that carries the class's pattern
    Buf<int32_t> len;                  // [n] length of the pattern
    Buf<int64_t> member_ptr;           // [n+1]
    Buf<int32_t> members;              // rows of every class, ascending
    int64_t size() const { return static_cast<int64_t>(first_row.size()); }
};

static PatternClasses group_equal_patterns(int64_t M, const Patterns& pat, Workers& workers)
{
    auto len_of = [&](int64_t r) { return static_cast<int32_t>(pat.ptr[r + 1] - pat.ptr[r]); };
    Buf<uint64_t> hash(static_cast<size_t>(M));
    workers.ranges(M, row_grain(M, pat.ptr[M], 4096, workers), [&](int64_t r0, int64_t r1, int) {
        for (int64_t r = r0; r < r1; ++r) {
            uint64_t x = 0x9E3779B97F4A7C15ull ^ static_cast<uint64_t>(pat.ptr[r + 1] - pat.ptr[r]);
            for (int64_t q = pat.ptr[r]; q < pat.ptr[r + 1]; ++q) {
                x ^= static_cast<uint64_t>(static_cast<uint32_t>(pat.idx[q])) + 0x9E3779B97F4A7C15ull + (x << 6) + (x >> 2);
                x *= 0xFF51AFD7ED558CCDull;
            }
            hash[r] = x;
        }
    });
    auto same = [&](int32_t a, int32_t b) {
        return hash[a] == hash[b] && len_of(a) == len_of(b) &&
               std::equal(pat.idx.begin() + pat.ptr[a], pat.idx.begin() + pat.ptr[a + 1], pat.idx.begin() + pat.ptr[b]);
    };
    // First row with the same pattern, by open addressing; each piece has the rows of some of the top hash bits, which a counting sort
    // has put together.
    Buf<int32_t> rep(static_cast<size_t>(M)), by_shard(static_cast<size_t>(M));
    const int64_t shards = M < 8192 ? 1 : 64, parts = shards == 1 ? 1 : workers.most();
    auto shard_of = [&](int64_t r) { return shards == 1 ? int64_t{0} : static_cast<int64_t>(hash[r] >> 58); };
    std::vector<int64_t> place(static_cast<size_t>(parts * shards), 0), shard_at(static_cast<size_t>(shards) + 1, 0);
    workers.ranges(parts, 1, [&](int64_t p0, int64_t p1, int) {
        for (int64_t part = p0; part < p1; ++part)
            for (int64_t r = M * part / parts; r < M * (part + 1) / parts; ++r) ++place[part * shards + shard_of(r)];
    });
    for (int64_t shard = 0, at = 0; shard < shards; ++shard) {
        for (int64_t part = 0; part < parts; ++part) {
            const int64_t n = place[part * shards + shard];
            place[part * shards + shard] = at;
            at += n;
        }
        shard_at[shard + 1] = at;
    }
    workers.ranges(parts, 1, [&](int64_t p0, int64_t p1, int) {
        for (int64_t part = p0; part < p1; ++part)
            for (int64_t r = M * part / parts; r < M * (part + 1) / parts; ++r) by_shard[place[part * shards + shard_of(r)]++] = static_cast<int32_t>(r);
    });
    workers.ranges(shards, 1, [&](int64_t s0, int64_t s1, int) {
        std::vector<int32_t> table;
        for (int64_t shard = s0; shard < s1; ++shard) {
            size_t mask = 15;
            while (mask < static_cast<size_t>(2 * (shard_at[shard + 1] - shard_at[shard]))) mask = 2 * mask + 1;
            table.assign(mask + 1, -1);
            for (int64_t x = shard_at[shard]; x < shard_at[shard + 1]; ++x) {
                const int32_t r = by_shard[x];
                size_t at = static_cast<size_t>(hash[r]) & mask;
                while (table[at] >= 0 && !same(table[at], r)) at = (at + 1) & mask;
                if (table[at] < 0) table[at] = r;
                rep[r] = table[at];
            }
        }
    });
    PatternClasses pc;
    std::vector<int64_t> of_len(1, 0);           // by length: how many, then where the next one goes
    int64_t n = 0;
    for (int64_t r = 0; r < M; ++r) {
        if (rep[r] != r) continue;
        const size_t len = static_cast<size_t>(len_of(r));
        if (len + 2 > of_len.size()) of_len.resize(len + 2, 0);
        ++of_len[len + 1];
        ++n;
    }
    prefix_sums(of_len);
    pc.first_row.resize(static_cast<size_t>(n));
    for (int64_t r = 0; r < M; ++r)
        if (rep[r] == r) pc.first_row[of_len[len_of(r)]++] = static_cast<int32_t>(r);
    pc.class_of.resize(static_cast<size_t>(M));
    pc.len.resize(static_cast<size_t>(n));
    pc.member_ptr.assign(static_cast<size_t>(n) + 1, 0);
    pc.members.resize(static_cast<size_t>(M));
    for (int64_t k = 0; k < n; ++k) {
        pc.len[k] = len_of(pc.first_row[k]);
        pc.class_of[pc.first_row[k]] = static_cast<int32_t>(k);
    }
    for (int64_t r = 0; r < M; ++r) ++pc.member_ptr[(pc.class_of[r] = pc.class_of[rep[r]]) + 1];
    prefix_sums(pc.member_ptr);
    std::vector<int64_t> fill(pc.member_ptr.begin(), pc.member_ptr.end() - 1);
    for (int64_t r = 0; r < M; ++r) pc.members[fill[pc.class_of[r]]++] = static_cast<int32_t>(r);
    return pc;
}

// Inverted index: for every block column the classes whose pattern has it, ascending.
struct ColumnIndex {
    Buf<int64_t> ptr;       // [nbc+1]
    Buf<int64_t> len;       // [nbc] classes still listed (the clustering drops those that are used up)
    Buf<int32_t> classes;
    Buf<int32_t> at;        // [patterns] where a class stands in the list of a column of its pattern, as long as nothing has been dropped; for partners_of,
                            // and empty where a search elsewhere may take its place
    bool dropped = false;
};

// wants_at(index): asked once the lists' lengths are known.
template <typename F>
static ColumnIndex index_columns(int64_t nbc, const Patterns& pat, const PatternClasses& pc, F&& wants_at, Workers& workers)
{
    ColumnIndex inv;
    const int64_t n = pc.size();
    // counts by part of the classes and column, then the place of every part's first entry in every list
    const int64_t parts = nbc * workers.most() <= (int64_t{1} << 23) && n > 1024 ? workers.most() : 1;
    Buf<int64_t> place(static_cast<size_t>(parts * nbc));
    // (Parts of as many entries: of a graph's patterns, which are in the order of their lengths, the last sixteenth has a third of them.  65536 rows of 16,
    // sixteen threads: 2.5-2.9 ms in parts of as many patterns and with the places that partners_of wants, 0.8 in these and without.)
    int64_t all = 0;
    for (int64_t k = 0; k < n; ++k) all += pc.len[k];
    std::vector<int64_t> first(static_cast<size_t>(parts) + 1, n);
    for (int64_t k = 0, part = 0, before = 0; k < n && part < parts; before += pc.len[k++])
        while (part < parts && before >= all * part / parts) first[part++] = k;
    auto entries = [&](int64_t part, auto&& take) {
        for (int64_t k = first[part]; k < first[part + 1]; ++k)
            for (int64_t q = pat.ptr[pc.first_row[k]]; q < pat.ptr[pc.first_row[k] + 1]; ++q) take(pat.idx[q], k, q);
    };
    workers.ranges(parts, 1, [&](int64_t p0, int64_t p1, int) {
        for (int64_t part = p0; part < p1; ++part) {
            int64_t* count = place.data() + part * nbc;
            std::fill(count, count + nbc, int64_t{0});
            entries(part, [&](int32_t c, int64_t, int64_t) { ++count[c]; });
        }
    });
    inv.ptr.resize(static_cast<size_t>(nbc) + 1);
    inv.len.resize(static_cast<size_t>(nbc));
    int64_t total = 0;
    for (int64_t c = 0; c < nbc; ++c) {
        inv.ptr[c] = total;
        for (int64_t part = 0; part < parts; ++part) {
            const int64_t count = place[part * nbc + c];
            place[part * nbc + c] = total;
            total += count;
        }
        inv.len[c] = total - inv.ptr[c];
    }
    inv.ptr[nbc] = total;
    inv.classes.resize(static_cast<size_t>(total));
    const bool with_at = wants_at(inv);
    if (with_at) inv.at.resize(pat.idx.size());
    workers.ranges(parts, 1, [&](int64_t p0, int64_t p1, int) {
        for (int64_t part = p0; part < p1; ++part)
            entries(part, [&](int32_t c, int64_t k, int64_t q) {
                const int64_t to = place[part * nbc + c]++;
                inv.classes[to] = static_cast<int32_t>(k);
                if (with_at) inv.at[q] = static_cast<int32_t>(to - inv.ptr[c]);
            });
    });
    return inv;
}

// With which other classes could a cluster opened by a row of class k start to grow?  The first row of another class to
// join has to pass the merge test against the seed's own pattern: 1000 |a n b| > keep |a u b|.  All that is asked of a class is whether
// one of these has rows left, so it is given at most kMostPartners of them; a class with more of them ("many") is taken to have one
// left whatever happens, and its search ends.  (All pairs of 100 000 rows of two entries that share one column would be 5 G:
// 30 GB and 346 s, against 25 s now.  A graph of 65536 rows of 16 has a few classes with more than 16 and none with more than 32.)
constexpr size_t kMostPartners = 32;
struct Partners {
    Buf<int64_t> ptr;              // [n+1]
    Buf<int32_t> of;               // the partners of every class that has not many
    std::vector<uint8_t> many;     // [n]
};

// One thread's search for partners.
// Where a class has many increments to make, they are made without looking, and the counters are looked through (and cleared) once, in
// order; and only some of its columns are counted: b has to share `least` of a's columns, so all but least - m of them (the
// longest lists are left out) already hold m shared ones; whoever reaches m, about nobody by chance, is counted exactly.  Where the
// average class has `least` of them, a few classes are gone through first: a class with many partners has enough of them there.
template <typename Count>
class PartnerSearch {
public:
    PartnerSearch(const Patterns& pat, const PatternClasses& pc, int64_t keep)
        : pat_(pat), pc_(pc), keep_(keep), count_(static_cast<size_t>(pc.size() + kStride), 0) {}

    std::vector<int32_t> found;
    std::vector<std::pair<const int32_t*, const int32_t*>> lists;      // what the columns of class k list in [begin, end), set by the caller

    // Puts the partners of class k among the classes [begin, end) into found; false: more than kMostPartners, and not all of them.
    bool run(int64_t k, int64_t begin, int64_t end)
    {
        found.clear();
        if (begin >= end) return true;
        const int64_t len = pc_.len[k];
        const int64_t least = keep_ * (len + pc_.len[begin]) / (1000 + keep_) + 1;
        int64_t ahead = 0;
        for (const auto& list : lists) ahead += list.second - list.first;
        Count* const count = count_.data();
        const auto passes = [&](int64_t shared, int64_t other) { return 1000 * shared > keep_ * (len + pc_.len[other] - shared); };
        if (ahead <= (end - begin) / 16) {
            size_t x = 0;
            const int32_t* p = nullptr;
            for (; x < lists.size() && found.size() <= kMostPartners; ++x) {
                const int32_t* const stop = lists[x].second;
                for (p = lists[x].first; p < stop; ++p) {
                    const int64_t shared = ++count[*p];
                    if (shared < least || !passes(shared, *p) || passes(shared - 1, *p)) continue;
                    found.push_back(*p);
                    if (found.size() > kMostPartners) { ++p; break; }
                }
            }
            for (size_t y = 0; y < x; ++y)
                for (const int32_t *q = lists[y].first, *stop = y + 1 < x ? lists[y].second : p; q < stop; ++q) count[*q] = 0;
            return found.size() <= kMostPartners;
        }
        // m: what chance gives a pattern of the average number of columns, and four deviations more
        const double hit = static_cast<double>(ahead) / static_cast<double>((end - begin) * len);
        int64_t m = 2;
        for (int round = 0; round < 3; ++round) {
            const double mean = hit * static_cast<double>(len - least + m);
            m = std::min(least, static_cast<int64_t>(mean + 4.0 * std::sqrt(mean)) + 3);
        }
        const int64_t counted = std::min(len, len - least + m);
        if (counted < len)
            std::nth_element(lists.begin(), lists.begin() + counted, lists.end(),
                             [](const auto& x, const auto& y) { return x.second - x.first < y.second - y.first; });
        const int32_t* mine = pat_.idx.data() + pat_.ptr[pc_.first_row[k]];
        int64_t to = begin;
        for (int64_t window = ahead >= least * (end - begin) ? 8 * kStride : end - begin; to < end && found.size() <= kMostPartners; window *= 64) {
            const int64_t from = to;
            to = std::min(end, from + window);
            for (int64_t x = 0; x < counted; ++x) {
                // (in locals: a counter of one byte may lie anywhere, for all the compiler knows)
                const int32_t *p = lists[static_cast<size_t>(x)].first, *const stop = lists[static_cast<size_t>(x)].second;
                if (to == end)
                    for (; p < stop; ++p) ++count[*p];
                else
                    for (; p < stop && *p < to; ++p) ++count[*p];
                lists[static_cast<size_t>(x)].first = p;
            }
            for (int64_t x = from; x < to; x += kStride) {
                Count most = 0;
                for (int64_t y = 0; y < kStride; ++y) most = std::max(most, count[x + y]);
                if (most >= m)
                    for (int64_t other = x; other < std::min(to, x + kStride) && found.size() <= kMostPartners; ++other) {
                        if (count[other] < m) continue;
                        const int32_t* theirs = pat_.idx.data() + pat_.ptr[pc_.first_row[other]];
                        int64_t shared = 0;
                        for (int64_t u = 0, v = 0; u < len && v < pc_.len[other];) {
                            shared += mine[u] == theirs[v];
                            const bool up = mine[u] <= theirs[v], vp = theirs[v] <= mine[u];
                            u += up;
                            v += vp;
                        }
                        if (passes(shared, other)) found.push_back(static_cast<int32_t>(other));
                    }
                std::fill(count + x, count + x + kStride, Count{0});
            }
        }
        return found.size() <= kMostPartners;
    }

private:
    static constexpr int64_t kStride = 64;
    const Patterns& pat_;
    const PatternClasses& pc_;
    const int64_t keep_;
    std::vector<Count> count_;
};

// Each pair is looked for from the shorter pattern: |b| < 1000 |a| / keep bounds the longer one.  What a class with many partners
// did not list, the longer pattern looks for among those classes alone.
template <typename Count>
static Partners partners_of(const Patterns& pat, const PatternClasses& pc, const ColumnIndex& inv, const std::vector<int32_t>& alive,
                            int64_t keep, Workers& workers)
{
    // (alive[k] == 0: every row of the class is in a cluster)
    const int64_t n = pc.size(), nbc = static_cast<int64_t>(inv.len.size());
    struct Local {
        std::unique_ptr<PartnerSearch<Count>> search;
        std::vector<std::pair<int32_t, int32_t>> pairs;        // of partners
        std::vector<std::pair<int32_t, int32_t>> longer;       // (a class, a partner of it that has many)
    };
    std::vector<Local> locals(static_cast<size_t>(workers.most()));
    auto local_of = [&](int thread) -> Local& {
        Local& local = locals[static_cast<size_t>(thread)];
        if (!local.search) local.search = std::make_unique<PartnerSearch<Count>>(pat, pc, keep);
        return local;
    };
    Partners partners;
    partners.many.assign(static_cast<size_t>(n), 0);
    workers.ranges(n, 16, [&](int64_t j0, int64_t j1, int thread) {
        Local& local = local_of(thread);
        PartnerSearch<Count>& search = *local.search;
        for (int64_t j = j0; j < j1; ++j) {
            const int64_t k = n - 1 - j, len = pc.len[k];                       // long patterns, which take longest, first
            if (len == 0 || alive[k] == 0) continue;
            // the first class whose pattern is too long
            const int64_t end = keep == 0 ? n
                : std::partition_point(pc.len.begin() + k, pc.len.end(), [&](int32_t x) { return keep * x < 1000 * len; }) - pc.len.begin();
            search.lists.clear();
            for (int64_t q = pat.ptr[pc.first_row[k]]; q < pat.ptr[pc.first_row[k] + 1]; ++q) {
                const int32_t* p = inv.classes.data() + inv.ptr[pat.idx[q]];
                const int32_t* stop = p + inv.len[pat.idx[q]];
                p = inv.dropped ? std::upper_bound(p, stop, static_cast<int32_t>(k)) : p + inv.at[q] + 1;
                if (p < stop && stop[-1] >= end) stop = std::lower_bound(p, stop, static_cast<int32_t>(end));
                search.lists.emplace_back(p, stop);
            }
            if (!search.run(k, k + 1, end)) partners.many[k] = 1;
            else for (int32_t other : search.found) local.pairs.emplace_back(static_cast<int32_t>(k), other);
        }
    });
    std::vector<int32_t> with_many;
    for (int64_t k = 0; k < n; ++k)
        if (partners.many[k]) with_many.push_back(static_cast<int32_t>(k));
    if (!with_many.empty()) {
        // these by column
        std::vector<int64_t> ptr(static_cast<size_t>(nbc) + 1, 0);
        auto entries = [&](auto&& take) {
            for (int32_t k : with_many)
                for (int64_t q = pat.ptr[pc.first_row[k]]; q < pat.ptr[pc.first_row[k] + 1]; ++q) take(pat.idx[q], k);
        };
        entries([&](int32_t c, int32_t) { ++ptr[c + 1]; });
        prefix_sums(ptr);
        Buf<int32_t> classes(static_cast<size_t>(ptr[nbc]));
        std::vector<int64_t> fill(ptr.begin(), ptr.end() - 1);
        entries([&](int32_t c, int32_t k) { classes[fill[c]++] = k; });
        std::vector<uint8_t> many_too(static_cast<size_t>(n), 0);
        workers.ranges(n, 256, [&](int64_t j0, int64_t j1, int thread) {
            Local& local = local_of(thread);
            PartnerSearch<Count>& search = *local.search;
            for (int64_t j = j0; j < j1; ++j) {
                const int64_t k = n - 1 - j, len = pc.len[k];
                if (len == 0 || alive[k] == 0 || partners.many[k]) continue;
                // (a partner has more than keep len / 1000 columns, and this many of the shared ones list it)
                const int64_t least = keep * (len + keep * len / 1000 + 1) / (1000 + keep) + 1;
                int64_t listing = 0;
                for (int64_t q = pat.ptr[pc.first_row[k]]; q < pat.ptr[pc.first_row[k] + 1]; ++q) listing += ptr[pat.idx[q] + 1] > ptr[pat.idx[q]];
                if (listing < least) continue;
                const int64_t begin = std::partition_point(pc.len.begin(), pc.len.begin() + k, [&](int32_t x) { return keep * len >= 1000 * static_cast<int64_t>(x); }) - pc.len.begin();
                search.lists.clear();
                for (int64_t q = pat.ptr[pc.first_row[k]]; q < pat.ptr[pc.first_row[k] + 1]; ++q) {
                    const int32_t* p = classes.data() + ptr[pat.idx[q]];
                    const int32_t* stop = classes.data() + ptr[pat.idx[q] + 1];
                    stop = std::lower_bound(p, stop, static_cast<int32_t>(k));
                    search.lists.emplace_back(std::lower_bound(p, stop, static_cast<int32_t>(begin)), stop);
                }
                if (!search.run(k, begin, k)) many_too[k] = 1;
                else for (int32_t other : search.found) local.longer.emplace_back(static_cast<int32_t>(k), other);
            }
        });
        for (int64_t k = 0; k < n; ++k) partners.many[k] |= many_too[k];
    }
    auto listed = [&](auto&& take) {
        for (const Local& local : locals) {
            for (const auto& p : local.pairs) { take(p.first, p.second); take(p.second, p.first); }
            for (const auto& p : local.longer) take(p.first, p.second);
        }
    };
    partners.ptr.assign(static_cast<size_t>(n) + 1, 0);
    listed([&](int32_t k, int32_t) { partners.ptr[k + 1] += partners.many[k] ? 0 : 1; });
    prefix_sums(partners.ptr);
    partners.of.resize(static_cast<size_t>(partners.ptr[n]));
    std::vector<int64_t> fill(partners.ptr.begin(), partners.ptr.end() - 1);
    listed([&](int32_t k, int32_t other) { if (!partners.many[k]) partners.of[fill[k]++] = other; });
    return partners;
}

// The same from a search elsewhere, which finds all pairs: no class has many.  False: it did not.
static bool partners_elsewhere(const Patterns& pat, const PatternClasses& pc, const ColumnIndex& inv, const std::vector<int64_t>& first_of_len, int64_t keep,
                               PairSearch& elsewhere, Partners& partners, Workers& workers)
{
    const int64_t n = pc.size(), nbc = static_cast<int64_t>(inv.len.size()), longest = n ? pc.len[n - 1] : 0;
    Buf<uint32_t> ptr(static_cast<size_t>(n) + 1), list_ptr(static_cast<size_t>(nbc) + 1);
    ptr[0] = 0;
    for (int64_t k = 0; k < n; ++k) ptr[k + 1] = ptr[k] + static_cast<uint32_t>(pc.len[k]);
    for (int64_t c = 0; c <= nbc; ++c) list_ptr[c] = static_cast<uint32_t>(inv.ptr[c]);
    Buf<uint32_t> columns(ptr[n]);
    workers.ranges(n, row_grain(n, ptr[n], 4096, workers), [&](int64_t k0, int64_t k1, int) {
        for (int64_t k = k0; k < k1; ++k) std::copy_n(pat.idx.begin() + pat.ptr[pc.first_row[k]], pc.len[k], columns.begin() + ptr[k]);
    });
    const std::vector<uint32_t> from(first_of_len.begin(), first_of_len.end());
    Buf<int32_t> found;
    if (!elsewhere.run(PairSearch::Tables{n, nbc, longest, keep, ptr, columns, list_ptr, inv.classes, from}, found)) return false;
    partners.many.assign(static_cast<size_t>(n), 0);
    partners.ptr.assign(static_cast<size_t>(n) + 1, 0);
    for (int32_t k : found) ++partners.ptr[k + 1];
    prefix_sums(partners.ptr);
    partners.of.resize(found.size());
    std::vector<int64_t> fill(partners.ptr.begin(), partners.ptr.end() - 1);
    for (size_t x = 0; x < found.size(); ++x) partners.of[fill[found[x]]++] = found[x ^ 1];
    return true;
}

int64_t jaccard_cluster(int64_t M, int64_t nbc, const Patterns& pat, int tau_permille, Buf<int32_t>& order, Workers& workers,
                        Buf<int32_t>* by_pattern, PairSearch* elsewhere)
{
    order.clear();
    order.reserve(static_cast<size_t>(M));
    const PatternClasses pc = group_equal_patterns(M, pat, workers);
    const int64_t n_classes = pc.size();
    const int64_t keep = 1000 - tau_permille;
    // What partners_of takes, in the counting of a pattern in a list by one thread (at most half the pairs of every list, a sixth of the time each, shared by the
    // threads), and what a search elsewhere does, which takes the lists as they were made.
    struct Prices { double here, there; };
    auto prices = [&](const ColumnIndex& index) {
        double pairs = 0;
        for (int64_t c = 0; c < nbc; ++c) pairs += 0.5 * static_cast<double>(index.len[c]) * static_cast<double>(index.len[c]);
        return Prices{0.25 * pairs / workers.most(), elsewhere && !index.dropped ? elsewhere->price(n_classes, nbc, index.ptr[nbc], pairs, n_classes ? pc.len[n_classes - 1] : 0)
                                                                                 : std::numeric_limits<double>::infinity()};
    };
    auto found_here = [&](const ColumnIndex& index) { const Prices p = prices(index); return !(p.there < p.here); };
    // inverted index: classes of every block column
    ColumnIndex inv = index_columns(nbc, pat, pc, found_here, workers);

    std::vector<uint8_t> clustered(M, 0);
    // What the counting looks at per class, side by side.
    struct ClassState {
        int32_t alive;         // unclustered rows
        int32_t shared;        // 2 * |pattern n union of the open cluster| + (1 if its rows are in the candidate set)
        int32_t len, pad;
    };
    std::vector<ClassState> state(static_cast<size_t>(n_classes));
    for (int64_t k = 0; k < n_classes; ++k)
        state[k] = ClassState{static_cast<int32_t>(pc.member_ptr[k + 1] - pc.member_ptr[k]), 0, pc.len[k], 0};
    std::vector<int32_t> touched;             // classes with shared != 0, cleared when the cluster closes
    std::vector<int64_t> in_union(nbc, -1);   // id of the cluster whose union holds the column
    struct Column { int32_t c; int64_t at; }; // a column of the union: classes of its list counted so far
    std::vector<Column> columns;
    int32_t counted_to = 0;                   // first class that the lists of the union's columns have not been counted up to
    std::vector<int32_t> walked_over(nbc, 0); // by column: classes without rows met in its list since they were last dropped
    int64_t shortest = 0;                     // shortest non-empty pattern
    for (int64_t k = 0; k < n_classes && shortest == 0; ++k) shortest = pc.len[k];
    const int64_t longest = n_classes ? pc.len[n_classes - 1] : 0;
    std::vector<int64_t> first_of_len(static_cast<size_t>(longest) + 2);      // first class with a pattern of that length or more
    for (int64_t k = n_classes - 1, len = longest + 1; len >= 0; --len) {
        while (k >= 0 && pc.len[k] >= len) --k;
        first_of_len[len] = k + 1;
    }
    AscendingSet candidates(M);
    int64_t n_clusters = 0;
    Partners partners;                        // once they have been asked for
    constexpr int64_t kFirstAsk = 20000, kFirstClusters = 8, kFewClusters = 300000;     // (fewer clusters tell enough once so much has been counted)
    int64_t spent = 0, ask_at = kFirstAsk;    // counting done so far; when to look whether it is worth asking
    int64_t spent_alone = 0;                  // of it, for clusters that no other pattern joined

    // Row `v` (a seed, or one that joins) brings its columns into the union, while the scan stands at it: every class that has
    // one of them shares one more column with the union, and so does each of its rows.  Only rows
    // ahead of the scan can still be visited; their count when the scan reaches them is the
    // class's.  A row is only worth a visit once it could pass the merge test at all.  The
    // test at the visit, with the union U' >= U of that later moment and the count n' of then, is
    // 1000 n' > keep (|w| + U' - n'), which implies (1000 + keep) n' > keep (|w| + U); n' is
    // reached at the last increment, where the same inequality with the U of that moment (smaller
    // still) therefore holds.  So the rows of a class enter the candidate set at the first
    // increment that satisfies it, and no row that would be merged is left out; the exact test is
    // still taken at the visit.  The same bound with the shortest pattern of the matrix in place
    // of |w| comes first, so that most increments read nothing but the counter.
    // A row passes only if keep |w| < 1000 U' and keep U' < 1000 |w| (its count is at most the smaller of the two), and the lists are
    // ordered by |w|: a new column's list is counted from the first class that is long enough now, as the union only grows, and every
    // list of the union as far as the union's size allows now -- the rest when it has grown.  (A graph of 65536 rows: 28 -> 7 ms.)
    auto add_row = [&](int64_t v, int64_t cluster, int64_t& union_size) {
        const size_t known = columns.size();
        for (int64_t q = pat.ptr[v]; q < pat.ptr[v + 1]; ++q)
            if (in_union[pat.idx[q]] != cluster) {
                in_union[pat.idx[q]] = cluster;
                columns.push_back(Column{pat.idx[q], 0});
            }
        if (columns.size() == known) return;
        union_size = static_cast<int64_t>(columns.size());
        const int64_t too_long = keep == 0 ? longest + 1 : std::min(longest + 1, (1000 * union_size + keep - 1) / keep);
        const int32_t begin = static_cast<int32_t>(first_of_len[std::min(longest + 1, keep * union_size / 1000 + 1)]);
        const int32_t end = static_cast<int32_t>(first_of_len[too_long]);
        const int64_t least = keep * (shortest + union_size) / (1000 + keep);   // a count must exceed this to matter for any row
        // (where the bound has not moved, the lists of the columns that were there are as far as they go)
        for (size_t u = known > 0 && end == counted_to ? known : 0; u < columns.size(); ++u) {
            Column& column = columns[u];
            int32_t* classes = inv.classes.data() + inv.ptr[column.c];
            const int64_t len = inv.len[column.c];
            if (u >= known) column.at = std::lower_bound(classes, classes + len, begin) - classes;
            const int64_t from = column.at;
            int64_t x = from, gone = 0;
            for (; x < len && classes[x] < end; ++x) {
                const int32_t k = classes[x];
                ClassState& at = state[k];
                if (at.alive == 0) { ++gone; continue; }
                const int32_t word = (at.shared += 2);
                if (word == 2) touched.push_back(k);
                if (word & 1) continue;                      // its rows are candidates already
                const int64_t n = word >> 1;
                if (!(n > least && (1000 + keep) * n > keep * (at.len + union_size))) continue;
                at.shared = word | 1;
                for (int64_t y = pc.member_ptr[k]; y < pc.member_ptr[k + 1]; ++y) {
                    const int32_t r = pc.members[y];
                    if (r > v && !clustered[r]) candidates.insert(r);
                }
            }
            spent += x - from;
            // Drop classes that are gone for good once walking over them has cost as much as dropping them does (but not before
            // it is known whether partners_of wants the lists as they were made).
            walked_over[column.c] += static_cast<int32_t>(gone);
            if (walked_over[column.c] > len && ask_at != kFirstAsk) {
                walked_over[column.c] = 0;
                int64_t kept = 0, before = 0;
                for (int64_t y = 0; y < len; ++y) {
                    if (y == x) before = kept;
                    if (state[classes[y]].alive > 0) classes[kept++] = classes[y];
                }
                inv.len[column.c] = kept;
                inv.dropped = true;
                x = x == len ? kept : before;
            }
            column.at = x;
        }
        counted_to = end;
    };
    // What it would save: the counting still to come for seeds that end up alone, if the rest of the rows goes like the rows so far, against
    // what the search takes.  With the first look after
    // 300 000 counted and weighed dearer, the whole of smat_preprocess took 1.8 ms for 1317 rows of five entries (now 1.4), 3.4 for 6872 of 19 (2.3),
    // 14.9 for a graph of 65536 rows (13.7).
    auto ask_partners = [&]() {
        const double done = static_cast<double>(order.size()) / static_cast<double>(M);
        const double ahead = static_cast<double>(spent_alone) * (1.0 - done) / done;
        const auto [here, there] = prices(inv);
        if (ahead < std::min(here, there) + 5e4) {
            ask_at = 2 * spent;
            return;
        }
        if (there < here) {
            if (partners_elsewhere(pat, pc, inv, first_of_len, keep, *elsewhere, partners, workers)) {
                ask_at = 0;
                return;
            }
            // It did not, and would not later; what is left for the threads has to pay at their price.
            elsewhere = nullptr;
            if (ahead < here + 5e4) {
                ask_at = 2 * spent;
                return;
            }
        }
        if (inv.at.empty() && !inv.dropped) inv = index_columns(nbc, pat, pc, [](const ColumnIndex&) { return true; }, workers);
        std::vector<int32_t> alive(static_cast<size_t>(n_classes));
        for (int64_t k = 0; k < n_classes; ++k) alive[k] = state[k].alive;
        ask_at = 0;
        const bool bytes = n_classes == 0 || pc.len[n_classes - 1] < 256;
        partners = bytes ? partners_of<uint8_t>(pat, pc, inv, alive, keep, workers) : partners_of<int32_t>(pat, pc, inv, alive, keep, workers);
    };
    // Every row before the scan's position is in a cluster, so a class with a row left has it ahead.
    auto has_partner = [&](int32_t k) {
        if (partners.ptr.empty() || partners.many[k]) return true;      // not asked, or too many to list: it may
        for (int64_t x = partners.ptr[k]; x < partners.ptr[k + 1]; ++x)
            if (state[partners.of[x]].alive > 0) return true;
        return false;
    };

    for (int64_t v = 0; v < M; ++v) {
        if (clustered[v]) continue;
        const int64_t cluster = n_clusters++;
        const int32_t seed_class = pc.class_of[v];
        clustered[v] = 1;
        --state[seed_class].alive;
        order.push_back(static_cast<int32_t>(v));
        if (pc.len[seed_class] == 0 || !has_partner(seed_class)) {
            // empty seed: distance 0 to other empty rows, 1 to everything else; no partner: the rows that join are
            // those with the seed's own pattern, which leave the union as it is
            if (tau_permille > 0)
                for (int64_t y = pc.member_ptr[seed_class]; state[seed_class].alive > 0 && y < pc.member_ptr[seed_class + 1]; ++y) {
                    const int32_t w = pc.members[y];
                    if (clustered[w]) continue;
                    clustered[w] = 1;
                    --state[seed_class].alive;
                    order.push_back(w);
                }
            continue;
        }
        int64_t union_size = 0;
        columns.clear();
        const int64_t spent_before = spent;
        bool alone = true;
        add_row(v, cluster, union_size);
        int64_t pos = v;
        for (;;) {
            const int64_t w = candidates.next(pos + 1);
            if (w < 0) break;
            candidates.erase(w);
            pos = w;
            const int32_t k = pc.class_of[w];
            const int64_t inter = state[k].shared >> 1;
            const int64_t uni = pc.len[k] + union_size - inter;
            if (1000 * inter > keep * uni) {             // 1 - inter/uni < tau/1000
                clustered[w] = 1;
                --state[k].alive;
                order.push_back(static_cast<int32_t>(w));
                alone &= k == seed_class;
                if (inter < pc.len[k]) add_row(w, cluster, union_size);      // otherwise every column of the row is in the union already
            }
        }
        for (int32_t k : touched) state[k].shared = 0;
        touched.clear();
        if (alone) spent_alone += spent - spent_before;
        if (partners.ptr.empty() && spent > ask_at && (n_clusters >= kFirstClusters || spent > kFewClusters)) ask_partners();
    }
    if (by_pattern) {
        // (the rows of B that putting a pattern's rows together can save are those of all its rows but one)
        by_pattern->clear();
        int64_t could_save = 0;
        for (int64_t k = 0; k < n_classes; ++k) could_save += (pc.member_ptr[k + 1] - pc.member_ptr[k] - 1) * pc.len[k];
        if (10 * could_save >= pat.ptr[M]) {
            by_pattern->reserve(static_cast<size_t>(M));
            std::vector<uint8_t> taken(static_cast<size_t>(n_classes), 0);
            for (int32_t r : order) {
                const int32_t k = pc.class_of[r];
                if (taken[k]) continue;
                taken[k] = 1;
                by_pattern->insert(by_pattern->end(), pc.members.begin() + pc.member_ptr[k], pc.members.begin() + pc.member_ptr[k + 1]);
            }
            if (*by_pattern == order) by_pattern->clear();
        }
    }
    return n_clusters;
}

// Per thread, for the passes over block rows: an array over the block columns, made by the first piece a thread takes.
template <typename T>
class PerThread {
public:
    PerThread(const Workers& workers, int64_t n, T fill) : all_(static_cast<size_t>(workers.most())), n_(n), fill_(fill) {}
    T* get(int thread)
    {
        std::vector<T>& v = all_[static_cast<size_t>(thread)];
        if (v.empty()) v.assign(static_cast<size_t>(n_) + 1, fill_);
        return v.data();
    }
private:
    std::vector<std::vector<T>> all_;
    int64_t n_;
    T fill_;
};
constexpr int64_t kBlockRowGrain = 32;

int64_t count_blocks(int64_t M, int64_t nbc, const Patterns& pat, const int32_t* perm, Buf<int32_t>& per_row, Workers& workers)
{
    const int64_t nbr = (M + kBlock - 1) / kBlock;
    per_row.resize(static_cast<size_t>(nbr));
    PerThread<int32_t> seen_in(workers, nbc, -1);
    workers.ranges(nbr, kBlockRowGrain, [&](int64_t b0, int64_t b1, int thread) {
        int32_t* seen = seen_in.get(thread);
        for (int64_t br = b0; br < b1; ++br) {
            int32_t n = 0;
            for (int64_t i = br * kBlock; i < std::min<int64_t>(M, (br + 1) * kBlock); ++i)
                for (int64_t q = pat.ptr[perm[i]]; q < pat.ptr[perm[i] + 1]; ++q)
                    if (seen[pat.idx[q]] != br) { seen[pat.idx[q]] = static_cast<int32_t>(br); ++n; }
            per_row[br] = n;
        }
    });
    return std::accumulate(per_row.begin(), per_row.end(), int64_t{0});
}

static void build_structure(const Csr& a, const Patterns& pat, const Buf<int32_t>& per_row, Bcsr& out, Workers& workers);

// Occupied columns over every `stride`-th block row when rows are read in the order perm: the rows of B that a product asks for.
static int64_t occupied_columns(const Csr& a, const int32_t* perm, int64_t stride, Workers& workers)
{
    const int64_t nbr = (a.M + kBlock - 1) / kBlock, n_counted = (nbr + stride - 1) / stride;
    Buf<int64_t> per_row(static_cast<size_t>(n_counted));
    PerThread<int32_t> seen_in(workers, a.K, -1);
    workers.ranges(n_counted, kBlockRowGrain, [&](int64_t b0, int64_t b1, int thread) {
        int32_t* seen = seen_in.get(thread);
        for (int64_t x = b0; x < b1; ++x) {
            const int64_t br = x * stride;
            int64_t n = 0;
            for (int64_t i = br * kBlock; i < std::min<int64_t>(a.M, (br + 1) * kBlock); ++i)
                for (int64_t p = a.row_ptr[perm[i]]; p < a.row_ptr[perm[i] + 1]; ++p)
                    if (seen[a.col_idx[p]] != br) { seen[a.col_idx[p]] = static_cast<int32_t>(br); ++n; }
            per_row[x] = n;
        }
    });
    return std::accumulate(per_row.begin(), per_row.end(), int64_t{0});
}

// The clustering merges a row into a cluster where it comes upon it, so the rows of several patterns lie mixed in one cluster, some of a
// pattern's perhaps in another, and the sixteen rows of a block row then occupy the columns of most of these patterns: 2 % of
// 627 x 627 hidden blocks 762 000 columns, where by pattern it is 124 000.  What the caller sees (permutation, blocks) is the clustering's; the
// device's block rows, whose products cost a row of B per occupied column, take the rows by pattern where that saves a tenth.  us in
// fp16, before and now: that matrix at N = 160 29.4 and 8.6, N = 1000 185 and 33.
static void grouped_layout(const Csr& a, const Patterns& pat, Buf<int32_t>& by_pattern, Bcsr& out, Workers& workers)
{
    if (by_pattern.empty()) return;
    const int64_t stride = out.nbr >= 256 ? 8 : 1;      // (a sample tells: counting all of a band of 7339 rows takes a tenth of its set-up)
    const int64_t by = occupied_columns(a, by_pattern.data(), stride, workers), now = occupied_columns(a, out.perm.data(), stride, workers);
    if (10 * by > 9 * now) return;
    out.grouped_share = static_cast<double>(by) / static_cast<double>(now);
    out.grouped = std::make_unique<Bcsr>();
    Bcsr& g = *out.grouped;
    g.nbr = out.nbr;
    g.nbc = out.nbc;
    g.used_identity = false;
    g.perm.swap(by_pattern);
    Buf<int32_t> per_row;
    g.n_blocks = count_blocks(a.M, g.nbc, pat, g.perm.data(), per_row, workers);
    build_structure(a, pat, per_row, g, workers);
}

void build_bcsr(const Csr& a, bool reorder, int tau_permille, Bcsr& out, Workers& workers, PairSearch* elsewhere)
{
    const int64_t M = a.M;
    out.nbr = (M + kBlock - 1) / kBlock;
    out.nbc = (a.K + kBlock - 1) / kBlock;
    Patterns pat;
    block_patterns(a, pat, workers);

    out.perm.resize(static_cast<size_t>(M));
    std::iota(out.perm.begin(), out.perm.end(), 0);
    Buf<int32_t> per_row, per_row_cand, by_pattern;
    out.n_blocks_identity = count_blocks(M, out.nbc, pat, out.perm.data(), per_row, workers);
    out.n_blocks = out.n_blocks_identity;
    out.used_identity = true;
    out.n_clusters = 0;
    if (reorder) {
        Buf<int32_t> cand;
        out.n_clusters = jaccard_cluster(M, out.nbc, pat, tau_permille, cand, workers, &by_pattern, elsewhere);
        const int64_t n_cand = count_blocks(M, out.nbc, pat, cand.data(), per_row_cand, workers);
        if (n_cand < out.n_blocks_identity) {            // strictly fewer, else keep P = I
            out.perm.swap(cand);
            per_row.swap(per_row_cand);
            out.n_blocks = n_cand;
            out.used_identity = false;
        }
    }

    build_structure(a, pat, per_row, out, workers);
    grouped_layout(a, pat, by_pattern, out, workers);
}

// Row pointer, block columns and column masks of the BCSR of A' = P A for the permutation
// already in out.perm; per_row holds the number of blocks of every block row.
static void build_structure(const Csr& a, const Patterns& pat, const Buf<int32_t>& per_row, Bcsr& out, Workers& workers)
{
    const int64_t M = a.M;
    out.row_ptr.resize(static_cast<size_t>(out.nbr) + 1);
    out.row_ptr[0] = 0;
    std::copy(per_row.begin(), per_row.end(), out.row_ptr.begin() + 1);
    prefix_sums(out.row_ptr);
    out.col_idx.resize(static_cast<size_t>(out.n_blocks));
    out.col_mask.resize(static_cast<size_t>(out.n_blocks));
    PerThread<uint64_t> bits_of(workers, (out.nbc + 63) / 64, 0);      // block columns of the block row at hand
    PerThread<int32_t> slot_of(workers, out.nbc, -1);                  // their places in col_idx
    workers.ranges(out.nbr, kBlockRowGrain, [&](int64_t b0, int64_t b1, int thread) {
        uint64_t* bits = bits_of.get(thread);
        int32_t* slot = slot_of.get(thread);
        for (int64_t br = b0; br < b1; ++br) {
            const int64_t i_end = std::min<int64_t>(M, (br + 1) * kBlock);
            int32_t* cols = out.col_idx.data() + out.row_ptr[br];
            const int32_t n = out.row_ptr[br + 1] - out.row_ptr[br];
            int32_t at = 0;
            // ascending union of the rows' patterns: collected through the bit set, which then either is read off in
            // order or, where the row has few blocks for its length, only keeps the list free of repetitions
            for (int64_t i = br * kBlock; i < i_end; ++i)
                for (int64_t q = pat.ptr[out.perm[i]]; q < pat.ptr[out.perm[i] + 1]; ++q) {
                    const int32_t c = pat.idx[q];
                    if (bits[c >> 6] >> (c & 63) & 1u) continue;
                    bits[c >> 6] |= uint64_t{1} << (c & 63);
                    cols[at++] = c;
                }
            if (out.nbc / 64 <= 4 * static_cast<int64_t>(n)) {
                at = 0;
                for (int64_t w = 0; w < (out.nbc + 63) / 64; ++w)
                    for (uint64_t x = bits[w]; x; x &= x - 1) cols[at++] = static_cast<int32_t>(64 * w) + __builtin_ctzll(x);
            } else {
                std::sort(cols, cols + n);
            }
            for (int32_t s = 0; s < n; ++s) {
                bits[cols[s] >> 6] = 0;
                slot[cols[s]] = out.row_ptr[br] + s;
                out.col_mask[out.row_ptr[br] + s] = 0;
            }
            // per block: which of its 16 columns hold a stored entry
            for (int64_t i = br * kBlock; i < i_end; ++i) {
                const int64_t r = out.perm[i];
                for (int64_t p = a.row_ptr[r]; p < a.row_ptr[r + 1]; ++p) {
                    const int32_t c = a.col_idx[p];
                    out.col_mask[slot[c / kBlock]] |= static_cast<uint16_t>(1u << (c % kBlock));
                }
            }
        }
    });
}

bool reorder_columns(Csr& a, int tau_permille, Bcsr& b, Workers& workers)
{
    const int64_t M = a.M, K = a.K;
    b.col_perm.resize(static_cast<size_t>(K));
    std::iota(b.col_perm.begin(), b.col_perm.end(), 0);
    b.n_blocks_rows_only = b.n_blocks;
    if (K == 0 || M == 0) return false;
    // column patterns: ascending block rows of A' = P A per column (rows are walked in their new order)
    Patterns cpat;
    cpat.ptr.assign(static_cast<size_t>(K) + 1, 0);
    std::vector<int32_t> last(K, -1);
    for (int64_t i = 0; i < M; ++i) {
        const int64_t r = b.perm[i];
        const int32_t br = static_cast<int32_t>(i / kBlock);
        for (int64_t p = a.row_ptr[r]; p < a.row_ptr[r + 1]; ++p)
            if (last[a.col_idx[p]] != br) { last[a.col_idx[p]] = br; ++cpat.ptr[a.col_idx[p] + 1]; }
    }
    prefix_sums(cpat.ptr);
    cpat.idx.resize(static_cast<size_t>(cpat.ptr[K]));
    {
        std::vector<int64_t> fill(cpat.ptr.begin(), cpat.ptr.end() - 1);
        std::fill(last.begin(), last.end(), -1);
        for (int64_t i = 0; i < M; ++i) {
            const int64_t r = b.perm[i];
            const int32_t br = static_cast<int32_t>(i / kBlock);
            for (int64_t p = a.row_ptr[r]; p < a.row_ptr[r + 1]; ++p)
                if (last[a.col_idx[p]] != br) { last[a.col_idx[p]] = br; cpat.idx[fill[a.col_idx[p]]++] = br; }
        }
    }
    Buf<int32_t> cand, per_row;
    jaccard_cluster(K, b.nbr, cpat, tau_permille, cand, workers);
    const int64_t n_cand = count_blocks(K, b.nbr, cpat, cand.data(), per_row, workers);     // blocks of the transpose = blocks of P A Q
    if (n_cand >= b.n_blocks) return false;              // strictly fewer, else keep Q = I
    b.col_perm.swap(cand);
    b.grouped.reset();                                   // (of A with its columns in the old order)
    // A <- A Q: entry (r, c) moves to the new index of column c; columns ascend again inside every row
    std::vector<int32_t> new_of_old(static_cast<size_t>(K));
    for (int64_t c = 0; c < K; ++c) new_of_old[b.col_perm[c]] = static_cast<int32_t>(c);
    workers.ranges(M, 2048, [&](int64_t r0, int64_t r1, int) {
        std::vector<std::pair<int32_t, uint16_t>> row;
        for (int64_t r = r0; r < r1; ++r) {
            row.clear();
            for (int64_t p = a.row_ptr[r]; p < a.row_ptr[r + 1]; ++p) row.emplace_back(new_of_old[a.col_idx[p]], a.vals[p]);
            std::sort(row.begin(), row.end());
            for (size_t x = 0; x < row.size(); ++x) {
                a.col_idx[a.row_ptr[r] + static_cast<int64_t>(x)] = row[x].first;
                a.vals[a.row_ptr[r] + static_cast<int64_t>(x)] = row[x].second;
            }
        }
    });
    Patterns pat;
    block_patterns(a, pat, workers);
    b.n_blocks = count_blocks(M, b.nbc, pat, b.perm.data(), per_row, workers);      // = n_cand, now by block row
    build_structure(a, pat, per_row, b, workers);
    return true;
}

void work_order(const std::vector<int32_t>& cost_ptr, std::vector<int32_t>& order)
{
    // Workgroups are handed to the eight XCDs of the chip round-robin (workgroup w runs on XCD
    // w mod 8), and every XCD has its own L2.
    //  * Block rows of similar cost (longest <= 1.25 x mean): position w gets a row from the
    //    (w mod 8)-th of eight contiguous ranges of block rows, so that each XCD walks a contiguous
    //    part of the matrix and neighbouring block rows, which tend to touch the same rows of B
    //    (band and mesh matrices), share that XCD's L2.
    //  * Otherwise: longest block rows first, so that the tail of a launch is made of short
    //    ones; the round-robin then gives every XCD the same mix of lengths.
    const int64_t nbr = static_cast<int64_t>(cost_ptr.size()) - 1;
    order.resize(static_cast<size_t>(nbr > 0 ? nbr : 0));
    if (nbr <= 0) return;
    int64_t longest = 0;
    for (int64_t br = 0; br < nbr; ++br)
        longest = std::max<int64_t>(longest, cost_ptr[br + 1] - cost_ptr[br]);
    const bool even_rows = 4 * longest * nbr <= 5 * static_cast<int64_t>(cost_ptr[nbr]);
    if (even_rows) {
        constexpr int kXcds = 8;
        int64_t begin[kXcds + 1];
        for (int x = 0; x <= kXcds; ++x) begin[x] = nbr * x / kXcds;
        int64_t next[kXcds];
        for (int x = 0; x < kXcds; ++x) next[x] = begin[x];
        for (int64_t w = 0; w < nbr; ++w) {
            int x = static_cast<int>(w % kXcds);
            while (next[x] >= begin[x + 1]) x = (x + 1) % kXcds;     // that range is used up: take the next one
            order[w] = static_cast<int32_t>(next[x]++);
        }
    } else {
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
            return (cost_ptr[x + 1] - cost_ptr[x]) > (cost_ptr[y + 1] - cost_ptr[y]);
        });
    }
}

void fill_canonical_vals(const Csr& a, const Bcsr& b, uint16_t* vals)
{
    std::fill(vals, vals + static_cast<size_t>(b.n_blocks) * kBlock * kBlock, uint16_t{0});
    std::vector<int32_t> slot_of(b.nbc, -1);
    for (int64_t br = 0; br < b.nbr; ++br) {
        for (int32_t s = b.row_ptr[br]; s < b.row_ptr[br + 1]; ++s) slot_of[b.col_idx[s]] = s;
        const int64_t i_end = std::min<int64_t>(a.M, (br + 1) * kBlock);
        for (int64_t i = br * kBlock; i < i_end; ++i) {
            const int64_t r = b.perm[i];
            for (int64_t p = a.row_ptr[r]; p < a.row_ptr[r + 1]; ++p) {
                const int32_t c = a.col_idx[p];
                const size_t blk = static_cast<size_t>(slot_of[c / kBlock]);
                vals[blk * 256 + static_cast<size_t>(i % kBlock) * 16 + static_cast<size_t>(c % kBlock)] = a.vals[p];
            }
        }
    }
}

}  // namespace smat
