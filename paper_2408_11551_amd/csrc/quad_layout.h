// Layout of one step of the two-of-four tile kernel (kernels_quads.hip), shared by the host code that plans it and the
// kernels.
//
// A step has quad_columns(es) k slots: as many rows of B in an LDS panel.  Panel rows 4 m .. 4 m + 3 are a quad: of their four
// columns of A a row stores at most two entries.
//
// Which value multiplies which panel row: the kernel reads panel rows 32 r + 8 g .. 32 r + 8 g + 7 as the r-th eight k of lane group g of the
// right operand (16-bit types r = 0, 1; 8-bit types r = 0 .. 3).  The instruction takes the k of its left operand in order, lane
// group G the G-th quarter of them, and its right operand in halves, of which every lane group has a quarter.  (Checked on the
// device, value by value and position by position, for the 16-bit types, e4m3 and int8.)  `halves`: an 8-bit type whose 128 k slots go to
// two instructions of a 16-bit type, 64 each; the first has a lane's first eight bytes of values and lower half of positions.
//
// Values: per step and block row 1 KiB, lane l = 16 G + i the 16 bytes at 16 l: row i, the pairs of values of its quads, in order.
// Positions: two bits per value, ascending inside a pair; per step and wave (four block rows) and lane the block rows' words one after the
// other, 16 bits each for the 16-bit types and 32 for the 8-bit types.
// Rows: per step the rows of B of the panel, K for none, in the order the lanes fetch them: four consecutive words are one lane's four loads.
#pragma once

#include <cstddef>
#include <cstdint>

#if defined(__HIPCC__)
#define SMAT_QUAD_HD __host__ __device__
#else
#define SMAT_QUAD_HD
#endif

namespace smat {

SMAT_QUAD_HD constexpr int quad_columns(int es) { return es == 2 ? 64 : 128; }

// panel row of word x of a step's table: load x % 4 of the lanes that carry unit x / 4
SMAT_QUAD_HD inline int quad_panel_row(int es, int x)
{
    const int unit = x >> 2, load = x & 3;
    return es == 2 ? 16 * load + unit : 32 * (unit >> 3) + 8 * load + (unit & 7);
}
// and the other way round
SMAT_QUAD_HD inline int quad_table_word(int es, int row)
{
    return es == 2 ? 4 * (row & 15) + (row >> 4) : 4 * (8 * (row >> 5) + (row & 7)) + ((row >> 3) & 3);
}

struct QuadSlot { int lane_group, pair; };
// lane group of the left operand and pair of values (inside the lane's 16 bytes) of a panel row
SMAT_QUAD_HD inline QuadSlot quad_slot(int es, bool halves, int row)
{
    const int r = row >> 5, g = (row & 31) >> 3, h = (row >> 2) & 1;
    if (halves) return QuadSlot{2 * (r & 1) + (g >> 1), 4 * (r >> 1) + 2 * (g & 1) + h};
    return es == 2 ? QuadSlot{2 * r + (g >> 1), 2 * (g & 1) + h}
                   : QuadSlot{2 * (r >> 1) + (g >> 1), 4 * (g & 1) + 2 * (r & 1) + h};
}
// first panel row of the quad of a pair
SMAT_QUAD_HD inline int quad_first_row(int es, bool halves, int lane_group, int pair)
{
    if (halves) return 64 * (pair >> 2) + 32 * (lane_group >> 1) + 8 * (2 * (lane_group & 1) + ((pair >> 1) & 1)) + 4 * (pair & 1);
    return es == 2 ? 32 * (lane_group >> 1) + 8 * (2 * (lane_group & 1) + (pair >> 1)) + 4 * (pair & 1)
                   : 32 * (2 * (lane_group >> 1) + ((pair >> 1) & 1)) + 8 * (2 * (lane_group & 1) + (pair >> 2)) + 4 * (pair & 1);
}

// shared memory of the bind-time scatter: a place per column, a bit per row of a block row and place
inline size_t quad_place_bytes(int64_t K) { return (static_cast<size_t>(K) * 2 + 15) / 16 * 16; }
inline size_t quad_fill_lds(int64_t K, int64_t max_steps, int es)
{
    return quad_place_bytes(K) + 16 * static_cast<size_t>(max_steps) * static_cast<size_t>(quad_columns(es)) / 8;
}
constexpr size_t kQuadFillLds = 64 * 1024;

// The kernel for few columns keeps all rows of B in LDS, as many bytes of each as there are columns or as LDS holds: the whole
// (the sum of the waves' partial tiles takes 32 KiB), bytes of a row -- 0 if not even eight fit -- and passes over the columns.
inline size_t quad_rows_lds(int64_t max_steps, int es, int row_bytes)
{
    const size_t panel = static_cast<size_t>(max_steps) * static_cast<size_t>(quad_columns(es)) * static_cast<size_t>(row_bytes);
    return panel < 32768 ? 32768 : panel;
}
constexpr size_t kQuadRowsLds = 144 * 1024;
inline int quad_row_bytes(int es, int64_t N, int64_t max_steps)
{
    int bytes = N * es <= 8 ? 8 : N * es <= 16 || es == 1 ? 16 : 32;
    while (bytes >= 8 && quad_rows_lds(max_steps, es, bytes) > kQuadRowsLds) bytes /= 2;
    return bytes >= 8 ? bytes : 0;
}
inline int64_t quad_row_passes(int es, int64_t N, int row_bytes)
{
    const int64_t columns = row_bytes / es < 16 ? row_bytes / es : 16;
    return (N + columns - 1) / columns;
}

}  // namespace smat
