// jaccard_cluster with a search elsewhere that takes no patterns when it comes to it: what the threads look for by themselves then is what they
// would have looked for without one.  The loops run on one thread here, and the one over all patterns in sixteens, which only partners_of makes, is counted.
#include <algorithm>
#include <cstdio>
#include <random>

#include "../../paper_2408_11551_amd/csrc/preprocess.h"
#include "../../paper_2408_11551_amd/csrc/workers.h"

namespace {
int searches_here = 0;
}

namespace smat {

Workers::Workers(int64_t) { most_ = 8; }
Workers::~Workers() = default;
void Workers::ranges(int64_t n, int64_t grain, const std::function<void(int64_t, int64_t, int)>& body)
{
    searches_here += grain == 16;
    for (int64_t x = 0; x < n; x += grain) body(x, std::min(n, x + grain), 0);
}

}  // namespace smat

struct Declines : smat::PairSearch {
    int asked = 0;
    double price(int64_t, int64_t, int64_t, double, int64_t) const override { return 0; }
    bool run(const Tables&, smat::Buf<int32_t>&) override { ++asked; return false; }
};

// M rows of twelve of nbc block columns.  Of those behind the first hundred one in `alone` is by chance, the others are one of rows 2 ... 99, half of them with
// a column more: rows 0 and 1 are clusters of their own, which is why a search pays at the first look if it costs nothing.
static smat::Patterns patterns(int64_t M, int64_t nbc, int alone)
{
    std::mt19937 rng(7);
    std::vector<std::vector<int32_t>> rows;
    smat::Patterns pat;
    pat.ptr.assign(1, 0);
    auto any = [&](int64_t n) { return static_cast<int32_t>(rng() % static_cast<uint32_t>(n)); };
    for (int64_t r = 0; r < M; ++r) {
        std::vector<int32_t> columns;
        if (r >= 100 && any(alone) != 0) columns = rows[static_cast<size_t>(2 + any(98))];
        while (columns.size() < 12 || (r >= 100 && columns.size() == 12 && any(2))) columns.push_back(any(nbc));
        std::sort(columns.begin(), columns.end());
        columns.erase(std::unique(columns.begin(), columns.end()), columns.end());
        pat.idx.insert(pat.idx.end(), columns.begin(), columns.end());
        pat.ptr.push_back(static_cast<int64_t>(pat.idx.size()));
        rows.push_back(columns);
    }
    return pat;
}

int main()
{
    int never = 0, later = 0;
    for (int64_t M : {int64_t{3000}, int64_t{20000}})
        for (int alone : {1, 8, 64, 200}) {
            const int64_t nbc = 500;
            const smat::Patterns pat = patterns(M, nbc, alone);
            smat::Workers workers(pat.ptr[M]);
            smat::Buf<int32_t> by_itself, declined;
            searches_here = 0;
            const int64_t n_by_itself = smat::jaccard_cluster(M, nbc, pat, 700, by_itself, workers);
            const int wanted = searches_here;
            Declines search;
            searches_here = 0;
            const int64_t n_declined = smat::jaccard_cluster(M, nbc, pat, 700, declined, workers, nullptr, &search);
            std::printf("%d rows, one in %d by chance: asked elsewhere %d times, here %d, without that search %d\n", static_cast<int>(M), alone, search.asked, searches_here, wanted);
            if (n_by_itself != n_declined || by_itself != declined) return std::puts("another order"), 1;
            if (search.asked > 1) return std::puts("asked again"), 1;
            if (searches_here != wanted) return std::puts("not what the threads alone look for"), 1;
            never += search.asked == 1 && wanted == 0;
            later += search.asked == 1 && wanted == 1;
        }
    if (!never || !later) return std::puts("none of a kind"), 1;
    std::puts("OK");
    return 0;
}
