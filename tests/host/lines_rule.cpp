// Goes over measured products with the rule that chooses between the per-row kernels (lines_rule.h).  In: one product a line, eleven numbers.
// Out: their number, the mean of log(time of the kernel chosen / of the faster one), and how many are over 5 % and 10 % slower than on registers.
#include <algorithm>
#include <cmath>
#include <cstdio>

#include "../../paper_2408_11551_amd/csrc/lines_rule.h"

int main()
{
    smat::DeviceBcsr d;
    int es, spread, n = 0, five = 0, ten = 0;
    long long n_order, n_packs, b_rows, K, N, ldb;
    double registers, lds, behind = 0;
    while (std::scanf("%d %lld %lld %d %d %lld %lld %lld %lld %lf %lf", &es, &n_order, &n_packs, &d.max_class, &spread, &b_rows, &K, &N, &ldb, &registers, &lds) == 11) {
        d.n_order = n_order;
        d.n_packs = n_packs;
        d.mean_row_packs = static_cast<double>(n_packs) / static_cast<double>(n_order);
        d.spread = spread != 0;
        d.b_rows = b_rows;
        d.K = K;
        const double us = smat::takes_lines(d, es, reinterpret_cast<const void*>(0x10000000), ldb, N) ? lds : registers;
        ++n;
        behind += std::log(us / std::min(registers, lds));
        five += us > 1.05 * registers;
        ten += us > 1.1 * registers;
    }
    std::printf("%d %.4f %d %d\n", n, behind / n, five, ten);
}
