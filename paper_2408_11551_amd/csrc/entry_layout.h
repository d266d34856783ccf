// Layout of the entry list (kernels_entries.hip), shared by the host code that plans it and the kernels.
//
// The stored entries of the matrix row by row, in the caller's order of rows, four to a record: four column numbers of 16 bits and four
// values, 16 bytes for the 16-bit types and 12 for the 8-bit ones.  A row begins with a record of its own; what the last one has too many names column K, a row
// of zeros in LDS.
#pragma once

#include <cstddef>
#include <cstdint>

namespace smat {

constexpr int kEntriesPerRecord = 4;
constexpr int entry_record_bytes(int es) { return es == 2 ? 16 : 12; }

// All of B is in LDS, as many columns of it at a time as there are or as LDS holds: columns per pass (a power of two; 0: not even one), and passes.
constexpr size_t kEntryLds = 144 * 1024;
constexpr int64_t kEntryMostColumns = 16;      // of B per pass
inline size_t entry_lds(int64_t K, int es, int64_t columns) { return (static_cast<size_t>(K + 1) * static_cast<size_t>(columns * es) + 15) / 16 * 16; }
inline int64_t entry_columns(int64_t K, int es, int64_t N)
{
    int64_t columns = 1;
    while (columns < N && columns < kEntryMostColumns) columns *= 2;
    while (columns > 0 && entry_lds(K, es, columns) > kEntryLds) columns /= 2;
    return columns;
}

// A launch of one or more passes: sixteen waves to a workgroup, `lanes` lanes to a row, as many as still give every compute unit what it holds at a time in one
// round.  (Two workgroups to a unit need 64 registers, which more than eight bytes of a row of B do not fit, and half of its LDS each.)
constexpr int kEntryThreads = 1024;
constexpr int entry_resident(int64_t row_bytes) { return row_bytes <= 8 ? 2 : 1; }
struct EntryLaunch { int lanes; int64_t workgroups; };         // of a pass
inline EntryLaunch entry_launch(int64_t M, int64_t K, int es, int64_t columns, int64_t passes)
{
    const int64_t resident = 256 * (entry_lds(K, es, columns) > 80 * 1024 ? 1 : entry_resident(columns * es));
    const int64_t most = resident > passes ? resident / passes : 1;
    auto workgroups = [&](int lanes) { return (M * lanes + kEntryThreads - 1) / kEntryThreads; };
    const int lanes = workgroups(64) <= most ? 64 : workgroups(32) <= most ? 32 : 16;
    return EntryLaunch{lanes, workgroups(lanes) < most ? workgroups(lanes) : most};
}

}  // namespace smat
