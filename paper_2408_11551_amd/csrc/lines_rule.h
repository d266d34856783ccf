// Which products the per-row kernel that gathers B through LDS takes (kernels_lines.hip).  Host only.
#pragma once

#include <cstdint>

#include "kernels.h"
#include "pack_layout.h"

namespace smat {

// es: bytes of an element of B
inline bool takes_lines(const DeviceBcsr& d, int es, const void* B, int64_t ldb, int64_t N)
{
    const int64_t bytes = N * es, starts = (ldb * es) | static_cast<int64_t>(reinterpret_cast<uintptr_t>(B));
    // block rows with packs of 32 slots, and not a few of them (which are a launch and little else); 32 bytes of a row of B and less are for narrower loads
    if (d.n_order < 64 || d.K == 0 || d.max_class < 2 || bytes <= 32 || bytes > 128 * 65535) return false;
    // rows that are not there are named by the offset 2^31, which has to lie past the end of B (from the dword on in which it begins)
    const int64_t ends = static_cast<int64_t>(reinterpret_cast<uintptr_t>(B) & 3u) + ((d.K - 1) * ldb + N) * es;
    if ((ends + 3) / 4 * 4 > (int64_t{1} << 31)) return false;
    const bool entries = d.max_class == kEntryClass, on_lines = starts % 128 == 0;
    const int64_t span = bytes + (starts % 4 == 0 ? 0 : 4 - es);
    // A single slab is faster there nearly throughout.  (us here and there.  On lines: 2048 block rows of 21 packs, N = 64 in fp16 19.1, 17.4, N = 128 in e4m3 20.5,
    // 15.9; a graph of 65536 rows, N = 64 15.9, 14.2, N = 32 11.5, 8.5.  On dwords: 50021 rows of a band, N = 34 in bf16 7.4, 5.8; the graph, N = 24 11.4, 8.9;
    // 1117 block rows of 38, N = 100 in e4m3 26.9, 24.2.  Off them: the band, N = 17 6.4, 4.7, N = 33 8.6, 6.7, N = 63 9.2, 7.2, N = 91 in int8 8.0, 8.0; the graph, N = 33 17.4,
    // 14.0; 1117 of 38, N = 33 in fp16 31.9, 24.8, N = 65 in e4m3 34.8, 25.9.)  Not for short rows kept by entry across a whole line of
    // bytes, with a slab of more than an L2 holds: 60000 rows of 10 entries, N = 128 in e5m2 13.3, 14.4.
    // Nor off the dwords, where moving what a row is shifted by takes its time: for a few long rows (69 block rows of 51 packs, N = 33 in fp16 6.1, 6.9, N = 90 in
    // e4m3 6.0, 8.0), for columns that just miss half a line (2048 block rows of 8, N = 63 in e4m3 7.0, 8.1), and for such short rows on pairs of bytes (60000 of
    // 10, N = 110 in int8 18.1, 20.1).
    if (span <= 128) {
        const bool short_rows = es == 1 && entries && d.mean_row_packs < 6.0 && static_cast<double>(d.K) * 128.0 >= 6.0e6;
        if (starts % 4 == 0) return !(short_rows && on_lines && bytes > 112);
        return !(d.n_order < 100 && d.mean_row_packs >= 32.0) && !(es == 1 && span > 64 && bytes <= 64) && !(short_rows && starts % 2 == 0 && bytes > 96);
    }
    // Several slabs off the lines are two lines of most rows each: only where one slab of all rows is well inside an L2 (us here and there, inputs not in the caches: 14000 rows of 20 entries, N = 160 in fp16 14.9, 11.7, N = 559 44.9, 38.1, in e4m3
    // 29.5, 27.2, N = 144 15.2, 10.9; 24000 of 16, N = 332 in int8 25.6, 24.2, but 40000 42.9, 50.8, and in fp16 30000 of 16, N = 134 21.3, 29.4; 400 x 400 hidden blocks,
    // N = 160 in fp16 7.0, 6.1, but 1000 x 1000, N = 134 16.3, 18.3).
    const int64_t slabs = (bytes + 127) / 128;
    const double packs = d.mean_row_packs;
    if (!on_lines) {
        const double narrow_slab = static_cast<double>(d.K) * 128.0;
        // (how far the other kernel's wider slabs, of loads as wide as it can, are behind: 9029 rows of 20, N = 332 in e4m3 17.3, 11.7, N = 668 16.4, 19.3)
        const int64_t most = es == 1 ? (starts % 16 == 0 ? 4 : starts % 4 == 0 ? 3 : 5) : (starts % 16 == 0 ? 4 : starts % 4 == 0 ? 5 : 10);
        if (slabs > most || packs >= (entries ? (es == 1 ? 16.0 : 12.0) : 14.0)) return false;
        return es == 1 ? narrow_slab <= 3.1e6 : d.spread && narrow_slab <= (entries ? 1.9e6 : 1.0e6);
    }
    // They read A once for each, where the other kernel's are twice as wide, and rows kept by entry are expanded once for each; what they save is what
    // one slab less would have found in the L2s, and half-empty slabs.  (us here and there, inputs not in the caches:)
    // 8-bit types, whose operands cost the other kernel more: faster throughout.  14000 rows of 16 entries, N = 256 15.3, 9.0, N = 1024 27.7, 22.2; 7000 of 30
    // 16.8, 11.7 at N = 512; a band of 201, N = 256 7.3, 5.4; 2048 x 2048 hidden blocks, N = 256 30.6, 26.7.
    // 16-bit types, rows by column: where rows of B come from all over.  627 block rows of 7 packs, N = 1024 33.3, 26.0; 1117 of 12, N = 512 39.5, 38.0; but
    // 1700 of 17, N = 256 39.1, 43.2, and bands of 81 and 257 columns 24.1, 26.4 and 15.7, 17.3.
    // By entry: short rows throughout (18000 of 12, N = 256 13.7, 11.8; 7000 of 6, N = 1024 13.7, 11.4; 2000 of 6 5.1, 5.5), longer ones in few slabs or where a
    // wide slab does not fit an L2 (16384 of 16, N = 128 10.2, 8.9, N = 384 17.0, 15.7, N = 512 23.1, 23.3; 30000 of 16 49.7, 39.8), the longest
    // also in three, of which the other kernel's last is half empty (12000 of 50, N = 192 24.5, 19.4, N = 512 41.1, 43.7; 40000 of 30, N = 256 53.5, 44.3; 24000
    // of 30 25.3, 28.3).
    const double wide_slab = static_cast<double>(d.K) * 256.0;
    if (es == 1) return packs < (entries ? 16.0 : 14.0) && (slabs <= 8 || !entries || wide_slab >= 5.0e6);
    if (!d.spread) return false;
    if (!entries) return packs < 14.0;
    if (packs < 12.0) return slabs <= (packs < 7.0 ? 16 : 6) || wide_slab >= 5.0e6;
    return slabs == 3 ? packs < 30.0 : packs < 16.0 && wide_slab >= (slabs == 2 ? 5.0e6 : 8.0e6);
}

}  // namespace smat
