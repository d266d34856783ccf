// Host-side preprocessing: CSR validation, block-column patterns, Jaccard row
// clustering, identity guard and the BCSR structure (paper sections "Blocked
// format", "Data Structures" and "Preprocessing").  Integer work only; no HIP.
#pragma once

#include <cstdint>
#include <memory>
#include <string>
#include <vector>

#include "workers.h"

namespace smat {

constexpr int kBlock = 16;   // h = w = 16

struct Csr {
    int64_t M = 0, K = 0;
    Buf<int64_t> row_ptr;           // [M+1]
    Buf<int32_t> col_idx;           // [nnz]
    Buf<uint16_t> vals;             // [nnz] bit patterns (an 8-bit type sits in the low byte)
};

struct Bcsr {
    int64_t nbr = 0, nbc = 0;
    Buf<int32_t> perm;               // [M] new -> old
    Buf<int32_t> row_ptr;            // [nbr+1]
    Buf<int32_t> col_idx;            // [n_e]
    Buf<uint16_t> col_mask;          // [n_e] bit c set iff column c of the block holds a stored entry
    int64_t n_blocks = 0, n_blocks_identity = 0;
    bool used_identity = true;
    // row + column reordering only (reorder_columns): new column -> old column, identity if unused
    Buf<int32_t> col_perm;
    int64_t n_blocks_rows_only = 0;
    int64_t n_clusters = 0;
    // The block structure that the block rows on the device are made from, where it is another one (grouped_layout): perm, row_ptr, col_idx, col_mask, n_blocks.
    std::unique_ptr<Bcsr> grouped;
    double grouped_share = 1.0;          // columns that its block rows occupy, of this one's
};

// Returns an empty string when the columns are well formed, else what is wrong with the first row that is not.
// row_ptr has been found to start at 0 and not to decrease.
std::string validate_csr(int64_t M, int64_t K, const int64_t* row_ptr, const int32_t* col_idx, Workers& workers);

// Row patterns: ascending block columns floor(c/16) per row, as a CSR-like pair.
struct Patterns {
    Buf<int64_t> ptr;       // [M+1]
    Buf<int32_t> idx;
};
void block_patterns(const Csr& a, Patterns& pat, Workers& workers);

// A search for the pairs of patterns that pass the merge test against each other, somewhere else than on the host's threads.
class PairSearch {
public:
    virtual ~PairSearch() = default;
    // What run() takes for n patterns with `entries` block columns (of nbc) and `pairs` pairs of entries in a column, in the counting of a pattern in a list
    // that one thread does meanwhile; infinity where it does not take them.
    virtual double price(int64_t n, int64_t nbc, int64_t entries, double pairs, int64_t longest) const = 0;
    // Pattern k (numbered by length, then as they come) has columns[ptr[k]] ..., column c the patterns lists[list_ptr[c]] ... in ascending order;
    // first_of_len[x] is the first pattern of x columns or more, x = 0 ... longest + 1.
    // Puts every pair into `found` once, as two numbers, the shorter pattern's first; false where it could not.
    struct Tables {
        int64_t n, nbc, longest, keep;
        const Buf<uint32_t>&ptr, &columns, &list_ptr;
        const Buf<int32_t>& lists;
        const std::vector<uint32_t>& first_of_len;
    };
    virtual bool run(const Tables& tables, Buf<int32_t>& found) = 0;
};

// Greedy Jaccard clustering; returns the cluster order (new -> old) and the number of clusters.  by_pattern: the rows of each
// pattern together, in the place of the first of them; empty where that is the same order.
int64_t jaccard_cluster(int64_t M, int64_t nbc, const Patterns& pat, int tau_permille, Buf<int32_t>& order, Workers& workers,
                        Buf<int32_t>* by_pattern = nullptr, PairSearch* elsewhere = nullptr);

// Number of nonzero blocks when rows are read in the order perm on the 16-row grid; per_row receives
// the number of every block row.
int64_t count_blocks(int64_t M, int64_t nbc, const Patterns& pat, const int32_t* perm, Buf<int32_t>& per_row, Workers& workers);

// Full pipeline: patterns -> (optional) clustering -> guard -> BCSR structure and column masks.
void build_bcsr(const Csr& a, bool reorder, int tau_permille, Bcsr& out, Workers& workers, PairSearch* elsewhere = nullptr);

// Row + column variant (the one the paper tried next to the row-only reordering, Preprocessing
// section): after build_bcsr, clusters the columns of A' = P A with the same greedy procedure, a
// column's pattern being the block rows it touches, and keeps the column order Q only if P A Q
// has strictly fewer blocks.  If it does, `a` becomes A Q (columns renumbered, ascending inside
// every row), b.col_perm holds Q (new -> old) and the structure of b is rebuilt; returns whether
// it did.
bool reorder_columns(Csr& a, int tau_permille, Bcsr& b, Workers& workers);

// Launch order of the block rows, given their cost as a row_ptr-like prefix array
// (cost of row br = cost_ptr[br+1] - cost_ptr[br]).
void work_order(const std::vector<int32_t>& cost_ptr, std::vector<int32_t>& order);

// Canonical block values (row-major 16x16 per block, zero filled) for export.
void fill_canonical_vals(const Csr& a, const Bcsr& b, uint16_t* vals);

}  // namespace smat
