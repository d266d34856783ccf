// Set-up with the device's help: the search of preprocess.cpp for patterns that could start a cluster, on the kernels of kernels_setup.hip, and the entry points
// for it (include/smat.h).
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <limits>
#include <new>
#include <vector>

#include "api.h"
#include "../../include/smat_bench.h"
#include "kernels.h"

namespace smat {

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

constexpr size_t kMostScratch = size_t{64} << 20;       // a graph of 300 000 rows of 16

// The search for partners of preprocess.cpp on the device, in memory of the caller's, which is asked for once it pays: 13-60 MB that a program does not hold
// yet are up to a millisecond, and bands, blocks and pruned matrices have no use for them.
class DevicePairSearch : public PairSearch {
public:
    // get: asked for `most` bytes at most; `all`: for so many.
    DevicePairSearch(smat_scratch_fn get, void* user, size_t most, bool all = false) : get_(get), user_(user), most_(most), all_(all) {}

    // 0.4 ms for the tables' way up (8.6 MB of a graph of 65536 rows of 16), the launches and the pairs' way down, and 134 million pairs of entries in
    // 0.4 ms; a unit, one pattern counted, is 2.4 ns of a thread.  (That graph, smat_preprocess: 14.7 ms, with sixteen threads looking for partners, 11.2 with the
    // device; 28740 rows 6.8 and 5.5.)  The counters have two bytes at most, entries and pairs numbers of 32 bits.
    double price(int64_t n, int64_t nbc, int64_t entries, double pairs, int64_t longest) const override
    {
        constexpr double kNever = std::numeric_limits<double>::infinity();
        if (n >= (int64_t{1} << 22) || longest >= 65536 || entries >= (int64_t{1} << 31) || pairs >= 4e9 || needed(n, nbc, entries, longest) > most_) return kNever;
        return 1.7e5 + 0.0014 * pairs;
    }

    bool run(const Tables& t, Buf<int32_t>& found) override
    {
        // (room for sixteen pairs per pattern, or what there is)
        const size_t wanted = needed(t.n, t.nbc, static_cast<int64_t>(t.columns.size()), t.longest) + 96 * static_cast<size_t>(t.n);
        const size_t bytes = all_ ? most_ : std::min(most_, wanted);
        void* on = nullptr;
        char* const scratch = static_cast<char*>(get_(bytes, user_, &on));
        const hipStream_t stream = static_cast<hipStream_t>(on);
        if (!scratch || reinterpret_cast<uintptr_t>(scratch) % kAlign != 0) return false;
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &status) != hipSuccess || status != hipStreamCaptureStatusNone) {
            (void)hipGetLastError();
            return false;
        }
        const size_t entries = t.columns.size(), n = static_cast<size_t>(t.n);
        size_t off = 0;
        auto take = [&](size_t count) { char* at = scratch + off; off = align_up(off + count * 4); return reinterpret_cast<uint32_t*>(at); };
        uint32_t* d_found = take(4);
        uint32_t* d_ptr = take(n + 1);
        uint32_t* d_columns = take(entries);
        uint32_t* d_list_ptr = take(static_cast<size_t>(t.nbc) + 1);
        uint32_t* d_lists = take(entries);
        uint32_t* d_first = take(t.first_of_len.size());
        const size_t most = std::min((bytes - off) / 8, size_t{1} << 24);
        auto up = [&](uint32_t* dst, const void* src, size_t count) {
            return count == 0 || hipMemcpyAsync(dst, src, count * 4, hipMemcpyHostToDevice, stream) == hipSuccess;
        };
        bool ok = launch_fill_zero(d_found, 1, stream) == 0 && up(d_ptr, t.ptr.data(), n + 1) && up(d_columns, t.columns.data(), entries) &&
                  up(d_list_ptr, t.list_ptr.data(), t.list_ptr.size()) && up(d_lists, t.lists.data(), entries) &&
                  up(d_first, t.first_of_len.data(), t.first_of_len.size());
        PartnerTables d;
        d.n = t.n;
        d.keep = static_cast<uint32_t>(t.keep);
        d.longest = static_cast<uint32_t>(t.longest);
        d.ptr = d_ptr;
        d.columns = d_columns;
        d.list_ptr = d_list_ptr;
        d.lists = d_lists;
        d.first_of_len = d_first;
        d.pairs = reinterpret_cast<uint32_t*>(scratch + off);
        d.most_pairs = static_cast<uint32_t>(most);
        d.found = d_found;
        const uint32_t first_long = t.first_of_len[static_cast<size_t>(std::min<int64_t>(short_pattern(), t.longest)) + 1];
        double pairs = 0;
        for (int64_t c = 0; c < t.nbc; ++c) pairs += std::pow(static_cast<double>(t.list_ptr[c + 1] - t.list_ptr[c]), 2.0);
        ok = ok && launch_partners(d, first_long, entries > 0 ? pairs / static_cast<double>(entries) : 0.0, stream) == 0;
        uint32_t got[2] = {0, 0};
        ok = ok && hipMemcpyAsync(got, d_found, 8, hipMemcpyDeviceToHost, stream) == hipSuccess;
        ok = hipStreamSynchronize(stream) == hipSuccess && ok;       // also where something failed: the copies read the caller's tables
        const uint32_t count = got[0];
        if (!ok || got[1] != 0 || count > most) {
            (void)hipGetLastError();
            return false;
        }
        found.resize(2 * static_cast<size_t>(count));
        if (count > 0 && (hipMemcpyAsync(found.data(), d.pairs, size_t{8} * count, hipMemcpyDeviceToHost, stream) != hipSuccess ||
                          hipStreamSynchronize(stream) != hipSuccess)) {
            (void)hipGetLastError();
            return false;
        }
        return true;
    }

private:
    // Bytes for n patterns with `entries` block columns in all, and for four pairs per pattern.
    static size_t needed(int64_t n, int64_t nbc, int64_t entries, int64_t longest)
    {
        size_t bytes = 32 * static_cast<size_t>(n);
        for (int64_t words : {int64_t{4}, n + 1, entries, nbc + 1, entries, longest + 2}) bytes += align_up(static_cast<size_t>(words) * 4);
        return bytes;
    }

    smat_scratch_fn get_;
    void* user_;
    size_t most_;
    bool all_;
};

}  // namespace

}  // namespace smat

using smat::DevicePairSearch;
using smat::fail;
using smat::kAlign;
using smat::kMostScratch;

extern "C" {

smat_status_t smat_preprocess_on_device(int64_t M, int64_t K, const int64_t* row_ptr, const int32_t* col_idx, const void* vals, smat_dtype_t dtype,
                                        const smat_options_t* opt, smat_scratch_fn scratch, void* user, smat_handle_t** out)
{
    // (below some hundred thousand entries the host's threads are done before the tables are up)
    // (row_ptr[M] is only read of an M that smat_preprocess does not refuse before it looks at row_ptr)
    const int64_t nnz = row_ptr && M >= 0 && M < (int64_t{1} << 22) ? row_ptr[M] : 0;
    const bool worth = scratch && nnz >= 200000 && nnz < (int64_t{1} << 24);
    DevicePairSearch search(scratch, user, kMostScratch);
    return smat::preprocess(M, K, row_ptr, col_idx, vals, dtype, opt, worth ? &search : nullptr, out);
}

smat_status_t smat_pattern_partners(int64_t n, int64_t nbc, const uint32_t* ptr, const uint32_t* columns, int keep, void* dev_scratch, size_t bytes, void* stream,
                                  int32_t* pairs, int64_t room, int64_t* count)
{
    if (n < 1 || nbc < 1 || !ptr || !columns || !pairs || !count || keep < 0 || keep > 1000) return fail(SMAT_ERR_INVALID_ARG, "invalid argument");
    if (!dev_scratch || reinterpret_cast<uintptr_t>(dev_scratch) % kAlign != 0) return fail(SMAT_ERR_INVALID_ARG, "dev_scratch must be 256-byte aligned");
    try {
        // (the kernels' counters and the searches by length rest on all of this: a column named twice would carry from one pattern's counter into the next one's)
        if (ptr[0] != 0) return fail(SMAT_ERR_INVALID_ARG, "ptr[0] must be 0");
        for (int64_t k = 0; k < n; ++k) {
            if (ptr[k + 1] < ptr[k]) return fail(SMAT_ERR_INVALID_ARG, "ptr decreases");
            for (uint32_t x = ptr[k]; x < ptr[k + 1]; ++x)
                if (columns[x] >= nbc || (x > ptr[k] && columns[x] <= columns[x - 1]))
                    return fail(SMAT_ERR_INVALID_ARG, "columns of a pattern must ascend and lie below n_columns");
        }
        const smat::Buf<uint32_t> p(ptr, ptr + n + 1), cols(columns, columns + ptr[n]);
        smat::Buf<uint32_t> list_ptr(static_cast<size_t>(nbc) + 1, 0u);
        smat::Buf<int32_t> lists(cols.size());
        int64_t longest = 0;
        for (int64_t k = 0; k < n; ++k) {
            const int64_t len = p[k + 1] - p[k];
            if (len < longest) return fail(SMAT_ERR_INVALID_ARG, "patterns are not in the order of their lengths");
            longest = len;
        }
        for (uint32_t c : cols) ++list_ptr[c + 1];
        double of_lists = 0;
        for (int64_t c = 0; c < nbc; ++c) {
            of_lists += 0.5 * list_ptr[c + 1] * list_ptr[c + 1];
            list_ptr[c + 1] += list_ptr[c];
        }
        std::vector<uint32_t> fill(list_ptr.begin(), list_ptr.end() - 1), first_of_len(static_cast<size_t>(longest) + 2, static_cast<uint32_t>(n));
        for (int64_t k = n - 1; k >= 0; --k)
            for (int64_t len = static_cast<int64_t>(p[k + 1]) - p[k]; len >= 0 && first_of_len[len] > k; --len) first_of_len[len] = static_cast<uint32_t>(k);
        for (int64_t k = 0; k < n; ++k)
            for (uint32_t x = p[k]; x < p[k + 1]; ++x) lists[fill[cols[x]]++] = static_cast<int32_t>(k);
        struct Given { void *at, *stream; } given{dev_scratch, stream};
        DevicePairSearch search([](size_t, void* user, void** on) { *on = static_cast<Given*>(user)->stream; return static_cast<Given*>(user)->at; }, &given, bytes,
                                true);
        smat::Buf<int32_t> found;
        if (!std::isfinite(search.price(n, nbc, p[n], of_lists, longest)) ||
            !search.run(smat::PairSearch::Tables{n, nbc, longest, keep, p, cols, list_ptr, lists, first_of_len}, found))
            return fail(SMAT_ERR_UNSUPPORTED, "the search does not take these patterns, or they have too many partners");
        *count = static_cast<int64_t>(found.size() / 2);
        if (*count > room) return fail(SMAT_ERR_INVALID_ARG, "more pairs than there is room for");
        std::copy(found.begin(), found.end(), pairs);
        return SMAT_OK;
    } catch (const std::bad_alloc&) {
        return fail(SMAT_ERR_ALLOC, "out of host memory in smat_pattern_partners");
    }
}

}  // extern "C"
