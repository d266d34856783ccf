// Which products the per-row kernel that gathers B through LDS takes (kernels_lines.hip).  Host only.
#pragma once

#include <cstdint>

#include "kernels.h"
#include "pack_layout.h"

namespace smat {

// es: bytes of an element of B
//
// The lines below were drawn on 1381 products of random, graph, band, hidden-block and pruned matrices (1000 ... 262144 rows, 33 ... 2200 bytes of a row of
// B, all types) and looked at on 1387 others, 652 of mostly wider B (to 8192 bytes) and 477 of the largest: profiles/lines_rule.csv, which
// tests/test_lines_rule.py goes over.  Of all of them, the geometric mean of the times over the faster kernel's is 1.020, over the registers' 0.886
// (everything here: 0.901); 78 products are more than 5 % slower than on registers, 29 of them more than 10 %, at most 1.34.  (The rule before, whose lines
// were drawn between single products: 1.050, 0.912; 165, 85, 1.39.)
inline bool takes_lines(const DeviceBcsr& d, int es, const void* B, int64_t ldb, int64_t N)
{
    const int64_t bytes = N * es, starts = (ldb * es) | static_cast<int64_t>(reinterpret_cast<uintptr_t>(B));
    // block rows with packs of 32 slots, and not a few of them (which are a launch and little else); 32 bytes of a row of B and less are for narrower loads
    if (d.n_order < 64 || d.K == 0 || d.max_class < 2 || bytes <= 32 || bytes > 128 * 65535) return false;
    // rows that are not there are named by the offset 2^31, which has to lie past the end of B (from the dword on in which it begins)
    const int64_t ends = static_cast<int64_t>(reinterpret_cast<uintptr_t>(B) & 3u) + ((d.K - 1) * ldb + N) * es;
    if ((ends + 3) / 4 * 4 > (int64_t{1} << 31)) return false;

    const bool on_dwords = starts % 4 == 0;
    const int64_t slabs = (bytes + (on_dwords ? 0 : 4 - es) + 127) / 128, units = d.n_order * slabs;
    const double rows = static_cast<double>(d.b_rows), uses = rows / static_cast<double>(d.K);              // uses: of a row of B
    const double mb = 1.0e-6 * static_cast<double>(bytes), slab_mb = 128.0e-6 * static_cast<double>(d.K);    // of a row; of one slab of all rows
    // A single slab on dwords is faster here nearly throughout: 0.87 of the time in the mean of 701 products, three more than 1.1 and at most 1.22.
    if (slabs == 1 && on_dwords) return true;
    // Off them what a row is shifted by is moved, which a launch of few packs does not hide, and in the 8-bit types neither do short rows (us on registers, here: 283
    // block rows of 3 packs, N = 55 in fp16 4.6, 5.7; 273 of 4, N = 103 in int8 4.2, 5.8; 1179 of 2, N = 71 in e4m3 4.8, 5.7; but 395 of 9, N = 30 4.1, 3.4).
    // Nor is it worth a whole line for columns that just miss half of one (N = 62 ... 64 in bytes: 0.88 ... 1.34 of the time).  Fewer than 128 block rows go either way
    // (65 ... 101 of 2 ... 38 packs, N = 17 ... 125: 0.73 ... 1.28).
    const bool few = !on_dwords && d.n_order < 128;
    if (slabs == 1) return !(es == 1 && bytes > 61 && bytes <= 64) && (few || (d.n_packs > 2300 && (es == 2 || d.mean_row_packs > 4.0 || d.n_order > 1900)));
    if (starts % 128 == 0) {
        // Several slabs on whole lines.  8-bit types, whose operands cost the other kernel more: throughout, 0.81 of the time, but where many units gather little each (bands of
        // 1087 block rows of 4 packs, N = 743 18.4, 24.1) unless C is large, which is stored past the caches here (3042 of 3, N = 640 45.2, 31.5), and
        // not for a slab that no L2 holds any of (239562 rows of a graph, N = 193 154, 179).
        if (es == 1) return slab_mb <= 16.0 && (uses > 6.0 || units <= 2800 || mb * static_cast<double>(d.K) > 16.0);
        // 16-bit types read A twice as often here as the other kernel does: where rows of B come from all over, of rows kept by column only as long as a slab leaves an L2
        // room (2048 x 2048 hidden blocks, N = 256 47, 63, but 956 x 956, N = 960 59, 47) and there are more than a few long ones (256 of 25 packs, N = 512 16.4, 22.3),
        // and not for rows as long as those of pruned weights (114 block rows of 230 packs, N = 232 25.3, 30.9); or few packs in all.
        const bool by_column = d.max_class != kEntryClass, room = slab_mb <= 3.0 && (d.mean_row_packs < 14.0 || d.n_order > 400);
        return (d.spread && uses <= 60.0 && (by_column ? room : slab_mb <= 16.0)) || d.n_packs * slabs <= 4000;
    }
    // Several slabs off the lines are two lines of most rows each: where a slab of all rows, or what is gathered, is well inside an L2 (24000 rows of 16, N = 332 in int8
    // 25.6, 24.2, but 40000 42.9, 50.8; 30000 of 16, N = 134 in fp16 21.3, 29.4; 400 x 400 hidden blocks, N = 160 in fp16 7.0, 6.1, but 1000 x 1000, N = 134
    // 16.3, 18.3; a graph of 21397 rows, N = 131 in e4m3 off the dwords 18.7, 23.2).
    if (on_dwords) return uses <= 60.0 && (es == 1 ? slab_mb <= 3.0 && (d.spread || uses > 6.0) : d.spread && rows * mb <= 36.0);
    if (es == 1) return slab_mb <= 0.43 || (slab_mb <= 2.0 && uses > 6.0 && bytes > 142 && rows * mb <= 170.0);
    return (d.spread && slabs > 4 && slab_mb <= 1.3) || (slab_mb <= 0.6 && (few || rows * mb > 4.0));
}

}  // namespace smat
