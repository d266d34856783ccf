// HIP kernel for gfx950: the per-row kernel (spmm_rows.h) with the rows of B gathered through LDS, a line or half a line of each.
//
// Work split: a workgroup of KW waves takes one block row and one slab of 128 bytes of every row of B (64 columns, or 128 of the
// 8-bit types), or of 64 where N has no more; wave ks walks packs ks, ks + KW, ... of the block row, the partial tiles are summed
// through LDS in a fixed order.
//
// What bounds products of sparse matrices is the gather of B, and what bounds that is how many cache lines a compute unit may wait for at a
// time, so it goes the faster the more of them are in the L2: 16-byte loads of rows of 128 bytes from a table of 2 / 4 / 8 / 16 MB come in
// at 24.4 / 22.8 / 13.6 / 9.7 TB/s, and just so in rows of 256 (8-byte loads: 13.0 / 13.0 / 12.2 / 9.2).  Slabs of one line make that
// table as small as it can be, but sixteen lanes that fetch eight bytes each, as the matrix instruction would have it, do not: here eight
// lanes fetch a row's line with sixteen bytes each, straight into LDS, and the transposing reads make the operand from there, without the
// permutes that the other kernel spends on it.
// Rows of B that begin off 16-byte pieces, where that kernel has to make do with loads of a few columns, are gathered just the same:
// these loads ask for dwords, and what is off by less is moved after the transposition (50021 rows of a band, N = 33 in bf16 8.85 -> 7.35 us).
#include <type_traits>
#include <utility>

#include <hip/hip_runtime.h>

#include "kernels.h"
#include "mfma_types.h"
#include "pack_layout.h"
#include "tile_common.h"

// compiled once per type of operand: SMAT_LINES_DT, its number in smat.h
#if SMAT_LINES_DT == 0
#define SMAT_LINES_TYPE "f16"
#elif SMAT_LINES_DT == 1
#define SMAT_LINES_TYPE "bf16"
#elif SMAT_LINES_DT == 2
#define SMAT_LINES_TYPE "e4m3"
#elif SMAT_LINES_DT == 3
#define SMAT_LINES_TYPE "e5m2"
#else
#define SMAT_LINES_TYPE "i8"
#endif
#if SMAT_LINES_DT < 2
#define SMAT_LINES_N64 "2"
#define SMAT_LINES_N128 "4"
#else
#define SMAT_LINES_N64 "4"
#define SMAT_LINES_N128 "8"
#endif

namespace smat {

namespace {

// Packs whose loads are under way while one is multiplied, and packs in LDS, 4 KiB each.  (What LDS holds are waves, and more of them count
// for more than a deeper ring: 16384 rows of 16 entries, N = 256, 11.8 us, with two packs ahead 14.9, with three 15.6.)
constexpr int kAhead = 1;
constexpr int kRing = kAhead + 1;

// the reads into v have returned, and all other LDS operations of the wave
template <int N>
__device__ __forceinline__ void lds_reads_done(u32x2_t (&v)[N])
{
    static_assert(N == 8 || N == 6 || N == 4 || N == 3, "");
    if constexpr (N == 8)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]));
    else if constexpr (N == 6)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]));
    else if constexpr (N == 4)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
    else
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]));
}

struct LineWalk {
    const uint32_t* slots;
    const uint8_t* vals;
    int npacks, ks, lane;
    uint32_t first_byte, bytes;        // of the slab in a row of B: where it begins, and how many there are of the row from there on
    uint32_t ldb_bytes, K, lds;
    uint32_t off_dword;                // bytes by which B begins past a dword
};

// bits 0 .. 3 of x as bytes of ones
__device__ __forceinline__ uint32_t bytes_of_bits(uint32_t x)
{
    const uint32_t ones = __umul24(x & 15u, 0x204081u) & 0x01010101u;
    return (ones << 8) - ones;
}

// v of this lane, or, where the mask has ones, of the lane BY further on among sixteen; those after the sixteenth are the first of next's
template <int BY>
__device__ __forceinline__ uint32_t from_further(uint32_t v, uint32_t next, uint32_t mask)
{
    const int wrapped = __builtin_amdgcn_mov_dpp(static_cast<int>(next), 0x120 + 16 - BY, 0xF, 0xF, true);                    // row_ror
    const int moved = __builtin_amdgcn_update_dpp(wrapped, static_cast<int>(v), 0x100 + BY, 0xF, 0xF, false);                 // row_shl
    return (v & ~mask) | (static_cast<uint32_t>(moved) & mask);
}

// The packs of a row of class L (pack_layout.h) or of an entry row.  A pack's rows of B lie in LDS in the order of its slot table, SLAB
// bytes each; 16-byte piece p of row (g, kk) -- lane group and position -- at p ^ swizzle, so that the 32 lanes that LDS serves at a time
// meet every bank once.
// SHIFTED: rows of B begin anywhere.  A row is fetched from the dword on that it begins in, so that its columns lie up to 4 / ES - 1 places
// further on in LDS.  What a transposing read brings a lane of a shifted row belongs to a lane before it, and is moved there: by DPP, for all rows of
// the pack, and then taken for those that are shifted.
template <int DT, int KW, int SLAB, int NX, bool SHIFTED, int L, bool ENTRY, bool IN_PARTS = false>
__device__ __forceinline__ void walk_lines(const LineWalk& w, __amdgpu_buffer_rsrc_t b_rsrc, typename Elem<DT>::Acc (&acc)[NX])
{
    constexpr int ES = Elem<DT>::ES;
    constexpr int PIECES = SLAB / 16, ROWS = 64 / PIECES;  // pieces of a row, rows of a load
    constexpr int NL = 4 * L > ROWS ? 4 * L / ROWS : 1;    // loads per pack
    constexpr uint32_t kPack = 32u * SLAB;                 // bytes of a pack's rows
    constexpr int AB = (ENTRY ? 8 : L) * ES;               // bytes of values per lane
    constexpr uint32_t kPackValues = ENTRY ? 64u : 64u * L * ES, kPackSlots = 16u * L;
    const int lane = w.lane, i = lane & 15, g = lane >> 4;
    const int count = w.ks < w.npacks ? (w.npacks - w.ks + KW - 1) / KW : 0;
    if (count == 0) return;
    const __amdgpu_buffer_rsrc_t slots_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w.slots), 0, w.npacks * static_cast<int>(kPackSlots), kRsrcFlags);
    const __amdgpu_buffer_rsrc_t vals_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(w.vals), 0, w.npacks * static_cast<int>(kPackValues), kRsrcFlags);
    auto swizzle = [](int g_, int kk) {
        if constexpr (SLAB == 128) return ES == 2 ? 2 * (((kk & 3) >> 1) + 2 * (g_ & 1)) : (kk >> 1) + 4 * (g_ & 1);
        else return ES == 2 ? 2 * (g_ & 1) : (kk >> 2) + 2 * (g_ & 1);
    };
    // Load e: rows ROWS e ... of the table, lane l the piece l % PIECES of row ROWS e + l / PIECES.
    uint32_t src_off[NL], from_lane[NL];
#pragma unroll
    for (int e = 0; e < NL; ++e) {
        const int at = ROWS * e + lane / PIECES;
        const uint32_t byte = 16u * static_cast<uint32_t>((lane & (PIECES - 1)) ^ swizzle(at / L, at % L));
        src_off[e] = byte < w.bytes && at < 4 * L ? w.first_byte + byte : kOutOfRange;
        from_lane[e] = 4u * static_cast<uint32_t>(at);
    }
    // Reads of group of columns x: 16-bit types kk = 0 .. 3 and, four rows on, 4 .. 7; 8-bit types all eight
    uint32_t tr_addr[NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) {
        const int kk = (ES == 2 ? i >> 2 : i >> 1) & (L - 1);
        const int piece = ES == 2 ? (2 * x) ^ swizzle(g, kk) : x ^ swizzle(g, kk);
        tr_addr[x] = w.lds + static_cast<uint32_t>(L * g + kk) * SLAB + 16u * static_cast<uint32_t>(piece) + 8u * (ES == 2 ? i & 3 : i & 1);
    }
    const uint32_t slot_voff = static_cast<uint32_t>(lane & (4 * L - 1)) * 4u;
    const uint32_t val_voff = static_cast<uint32_t>(ENTRY ? g : lane) * AB;
    const uint32_t row_match = static_cast<uint32_t>(i) * 0x11111111u;

    // Loads of pack h of this wave.  Past the last one the table is the last pack's, the rows are K (no access) and the values out of range (zeros).
    auto pack_of = [&](int h) { return static_cast<uint32_t>(w.ks + KW * (h < count ? h : count - 1)); };
    auto load_slots = [&](int h) { return static_cast<uint32_t>(__builtin_amdgcn_raw_buffer_load_b32(slots_rsrc, slot_voff, pack_of(h) * kPackSlots, 0)); };
    auto load_values = [&](int h) {
        const uint32_t voff = val_voff | (h < count ? 0u : kOutOfRange), soff = pack_of(h) * kPackValues;
        u32x4 a = u32x4{0u, 0u, 0u, 0u};
        if constexpr (AB == 16) {
            a = buf_load16(vals_rsrc, voff, soff);
        } else if constexpr (AB == 8) {
            const i32x2 v = __builtin_amdgcn_raw_buffer_load_b64(vals_rsrc, voff, soff, 0);
            a[0] = static_cast<uint32_t>(v[0]);
            a[1] = static_cast<uint32_t>(v[1]);
        } else if constexpr (AB == 4) {
            a[0] = static_cast<uint32_t>(__builtin_amdgcn_raw_buffer_load_b32(vals_rsrc, voff, soff, 0));
        } else {
            a[0] = static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(vals_rsrc, voff, soff, 0));
        }
        return a;
    };
    // returns, for an entry pack, the row numbers of the lane group's entries (four bits each)
    auto load_rows = [&](int h, uint32_t raw, int buf) -> uint32_t {
        const bool live = h < count;
#pragma unroll
        for (int e = 0; e < NL; ++e) {
            const uint32_t m = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(static_cast<int>(from_lane[e]), static_cast<int>(raw)));
            uint32_t off = __umul24(live ? m : w.K, w.ldb_bytes);
            // (the dword in which row K would begin may be the one in which the last row ends)
            if constexpr (SHIFTED) off = live && (m & 0xFFFFFFu) < w.K ? (off + w.off_dword) & ~3u : kOutOfRange;
            load_to_lds16((lds_void*)(uintptr_t)(w.lds + kPack * static_cast<uint32_t>(buf) + 1024u * e), b_rsrc, SHIFTED ? (off + (src_off[e] & ~kOutOfRange)) | (src_off[e] & kOutOfRange) : off + src_off[e], 0u);
        }
        if constexpr (ENTRY) {
            uint32_t m[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) m[k] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(4 * (8 * g + k), static_cast<int>(raw)));
            const uint32_t lo = __builtin_amdgcn_perm(m[1], m[0], 0x0C0C0703u), hi = __builtin_amdgcn_perm(m[3], m[2], 0x0C0C0703u);
            return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
        } else {
            return 0u;
        }
    };

    // by how many places the rows of a pack are shifted: bits 0 and 1, a word each, one bit per entry of the table
    struct Shifts { uint32_t low, high; };
    auto shifts_of = [&](uint32_t raw) {
        const uint32_t place = ((__umul24(raw, w.ldb_bytes) + w.off_dword) & 3u) / ES;
        return Shifts{static_cast<uint32_t>(__ballot(place & 1u)), ES == 1 ? static_cast<uint32_t>(__ballot(place & 2u)) : 0u};
    };

    uint32_t raw[kRing], row_numbers[kRing];
    Shifts shifts[kRing] = {};
    u32x4 a[kRing];
#pragma unroll
    for (int h = 0; h < kAhead; ++h) raw[h] = load_slots(h);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < kAhead; ++h) {
        a[h] = load_values(h);
        raw[(h + kAhead) % kRing] = load_slots(h + kAhead);       // (in the place of pack h - 1's)
        __builtin_amdgcn_sched_barrier(0);
        row_numbers[h] = load_rows(h, raw[h], h);
        if constexpr (SHIFTED) shifts[h] = shifts_of(raw[h]);
        __builtin_amdgcn_sched_barrier(0);
    }
    auto step = [&](auto u_, int s) __attribute__((always_inline)) {
        constexpr int u = decltype(u_)::value, next = (u + kAhead) % kRing;
        a[next] = load_values(s + kAhead);
        const uint32_t rows = raw[next];
        raw[(u + 2 * kAhead) % kRing] = load_slots(s + 2 * kAhead);
        __builtin_amdgcn_sched_barrier(0);
        row_numbers[next] = load_rows(s + kAhead, rows, next);
        if constexpr (SHIFTED) shifts[next] = shifts_of(rows);
        __builtin_amdgcn_sched_barrier(0);
        // What was asked for before the loads of the packs ahead is there.  Counted are those into LDS alone: of the others the compiler takes out
        // what nothing reads any more at the end of a walk.
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"(kAhead * NL));
        __builtin_amdgcn_sched_barrier(0);
        u32x2_t v[ES * NX];
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            if constexpr (ES == 2) {
                v[2 * x] = lds_read_tr<kPack * u>(tr_addr[x]);
                if constexpr (L == 8) v[2 * x + 1] = lds_read_tr<kPack * u + 4 * SLAB>(tr_addr[x]);
                else v[2 * x + 1] = u32x2_t{0u, 0u};
            } else {
                v[x] = lds_read_tr8<kPack * u>(tr_addr[x]);
            }
        }
        lds_reads_done(v);
        u32x4 av = a[u];
        if constexpr (ENTRY) {
            // left operand of lane (g, i): the value of entry (g, kk) where that entry's row is i, else zero; `miss` has a zero nibble there
            const uint32_t miss = row_numbers[u] ^ row_match;
            constexpr int PER = 4 / ES;
#pragma unroll
            for (int q = 0; q < 8 / PER; ++q) {
                uint32_t keep = 0u;
#pragma unroll
                for (int e = 0; e < PER; ++e)
                    if (((miss >> (4 * (PER * q + e))) & 15u) == 0u) keep |= (ES == 2 ? 0xFFFFu : 0xFFu) << (8 * ES * e);
                av[q] &= keep;
            }
        }
        if constexpr (SHIFTED) {
            const uint32_t low = shifts[u].low >> (L * g), high = shifts[u].high >> (L * g);
            constexpr int D = (L * ES + 3) / 4;            // dwords with rows of the lane's group, of each group of columns
            if constexpr (ES == 1) {
                uint32_t by_2[D];
#pragma unroll
                for (int q = 0; q < D; ++q) by_2[q] = bytes_of_bits(high >> (4 * q));
#pragma unroll
                for (int x = 0; x < NX; ++x)
#pragma unroll
                    for (int q = 0; q < D; ++q) v[x][q] = from_further<2>(v[x][q], x + 1 < NX ? v[(x + 1) % NX][q] : 0u, by_2[q]);
            }
            uint32_t by_1[D];
#pragma unroll
            for (int q = 0; q < D; ++q)
                by_1[q] = ES == 1 ? bytes_of_bits(low >> (4 * q)) : ((0u - ((low >> (2 * q)) & 1u)) & 0xFFFFu) | ((0u - ((low >> (2 * q + 1)) & 1u)) & 0xFFFF0000u);
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int q = 0; q < D; ++q) {
                    constexpr int V = ES == 2 ? 2 : 1;     // reads of a group of columns
                    v[V * x + q / 2][q % 2] = from_further<1>(v[V * x + q / 2][q % 2], x + 1 < NX ? v[V * ((x + 1) % NX) + q / 2][q % 2] : 0u, by_1[q]);
                }
        }
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            u32x4 b = ES == 2 ? u32x4{v[2 * x][0], v[2 * x][1], v[2 * x + 1][0], v[2 * x + 1][1]} : u32x4{v[x][0], v[x][1], 0u, 0u};
            // (positions past L hold another row's elements)
            if constexpr (L == 2) b = u32x4{ES == 2 ? b[0] : b[0] & 0xFFFFu, 0u, 0u, 0u};
            if constexpr (L == 4 && ES == 1) b[1] = 0u;
            if constexpr (IN_PARTS) acc[x] = mfma_pack_in_parts<DT, L>(av, b, acc[x]);
            else acc[x] = mfma_pack<DT>(av, b, acc[x]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto several = [&](int s, int n, auto... u) __attribute__((always_inline)) { (void)((decltype(u)::value < n && (step(u, s + decltype(u)::value), true)) && ...); };
    const int iters = count / kRing, rem = count % kRing;
    for (int it = 0; it < iters; ++it) with_constants(std::make_integer_sequence<int, kRing>{}, [&](auto... u) __attribute__((always_inline)) { several(kRing * it, kRing, u...); });
    with_constants(std::make_integer_sequence<int, kRing - 1>{}, [&](auto... u) __attribute__((always_inline)) { several(kRing * iters, rem, u...); });
}

}  // namespace

// Columns of a slab, a multiple of four: with what a row is shifted by they have to be in it.
template <int ES, int SLAB, bool SHIFTED>
__host__ __device__ constexpr int columns_of_slab(int N) { return SHIFTED && N > (SLAB - 4) / ES + 1 ? (SLAB - 4) / ES / 4 * 4 : SLAB / ES; }

// NX: groups of sixteen columns that there are in a slab, or three quarters of them where N has no more
template <int DT, int KW, int SLAB, int NX, bool SHIFTED>
__global__ __launch_bounds__(64 * KW)
void spmm_lines_kernel(const int32_t* __restrict__ work, const uint32_t* __restrict__ slots, const void* __restrict__ vals,
                       const int32_t* __restrict__ perm, const void* __restrict__ B, uint32_t b_bytes, uint32_t ldb_bytes,
                       uint32_t K, typename Elem<DT>::Out* __restrict__ C, int64_t ldc, int N, int n_order, uint32_t off_dword, int in_parts)
{
    using Acc = typename Elem<DT>::Acc;
    using Out = typename Elem<DT>::Out;
    constexpr int ES = Elem<DT>::ES, COLS = 16 * NX;
    constexpr int kArea = kRing * 32 * SLAB;               // LDS of a wave
    constexpr int LD = COLS + (ES == 2 ? 4 : 0);           // row of a tile on its way out, words (padded where there is room)
    static_assert(16 * LD * 4 <= kArea, "a tile takes the place of the rows of B");
    extern __shared__ u32x4 lds_dyn[];
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int ks = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    // The (slab, block row) pairs, slab by slab, dealt to the eight XCDs in contiguous shares, as kSlabsByXcd does in spmm_rows.h: an XCD's L2 has to
    // hold few slabs, each of them 128 K bytes (27350 rows of 12 entries, N = 960: 71 us with the slabs in turn, 49 like this).
    const uint32_t share = (blockIdx.x & 7u) * gridDim.y + blockIdx.y, record = (blockIdx.x & ~7u) | (share & 7u), slab = share >> 3;
    if (record >= static_cast<uint32_t>(n_order)) return;
    const i32x4 rec = reinterpret_cast<const i32x4*>(work)[record];
    const int br = rec[0] & 0x0FFFFFFF, cls = rec[0] >> 28;
    const int step = columns_of_slab<ES, SLAB, SHIFTED>(N), n0 = static_cast<int>(slab) * step;
    LineWalk w;
    w.slots = slots + static_cast<size_t>(static_cast<uint32_t>(rec[2])) * 8;
    w.vals = static_cast<const uint8_t*>(vals) + static_cast<size_t>(static_cast<uint32_t>(rec[3])) * 64;
    w.npacks = rec[1];
    w.ks = ks;
    w.lane = lane;
    w.first_byte = static_cast<uint32_t>(n0) * ES;
    w.bytes = static_cast<uint32_t>(N - n0) * ES + (SHIFTED ? 4 - ES : 0);
    w.ldb_bytes = ldb_bytes;
    w.K = K;
    w.lds = lds_offset_of(lds_dyn) + static_cast<uint32_t>(ks) * kArea;
    w.off_dword = off_dword;
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(B), 0, static_cast<int>(b_bytes), kRsrcFlags);
    // where this thread's pieces of four columns go: asked for now
    constexpr int Q = COLS / 4, EP = (16 * Q + 64 * KW - 1) / (64 * KW);
    int out_rows[EP];
#pragma unroll
    for (int k = 0; k < EP; ++k) out_rows[k] = static_cast<int>(threadIdx.x) + 64 * KW * k < 16 * Q ? perm[br * 16 + (static_cast<int>(threadIdx.x) + 64 * KW * k) / Q] : -1;
    Acc acc[NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) acc[x] = Acc{0, 0, 0, 0};
    constexpr bool PARTS = DT == kE4M3 || DT == kE5M2;
    if (PARTS && cls == 2 && in_parts) walk_lines<DT, KW, SLAB, NX, SHIFTED, 8, false, PARTS>(w, b_rsrc, acc);
    else if (PARTS && cls == 1 && in_parts) walk_lines<DT, KW, SLAB, NX, SHIFTED, 4, false, PARTS>(w, b_rsrc, acc);
    else if (cls == 2) walk_lines<DT, KW, SLAB, NX, SHIFTED, 8, false>(w, b_rsrc, acc);
    else if (cls == kEntryClass) walk_lines<DT, KW, SLAB, NX, SHIFTED, 8, true>(w, b_rsrc, acc);
    else if (cls == 1) walk_lines<DT, KW, SLAB, NX, SHIFTED, 4, false>(w, b_rsrc, acc);
    else walk_lines<DT, KW, SLAB, NX, SHIFTED, 2, false>(w, b_rsrc, acc);
    // nothing may still be on its way into LDS
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)");
    __builtin_amdgcn_sched_barrier(0);

    // acc[x][y] = C'[4 g + y][n0 + 16 x + i] of this wave's packs
    Out* const tile = reinterpret_cast<Out*>(reinterpret_cast<uint8_t*>(lds_dyn) + static_cast<size_t>(ks) * kArea);
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) tile[(4 * g + y) * LD + 16 * x + i] = acc[x][y];
    if constexpr (KW == 1) __builtin_amdgcn_wave_barrier();
    else __syncthreads();
#pragma unroll
    for (int k = 0; k < EP; ++k) {
        const int e = static_cast<int>(threadIdx.x) + 64 * KW * k;
        const int row = e / Q, c = 4 * (e % Q);
        const int64_t out_row = out_rows[k];
        if (out_row < 0 || c >= step || n0 + c >= N) continue;
        const Out* src = reinterpret_cast<const Out*>(lds_dyn) + row * LD + c;
        Acc v = *reinterpret_cast<const Acc*>(src);
#pragma unroll
        for (int x = 1; x < KW; ++x) v += *reinterpret_cast<const Acc*>(src + x * (kArea / 4));
        Out* dst = C + out_row * ldc + n0 + c;
        if (n0 + c + 4 <= N) {
            // past the L2s, which hold B (32768 rows, N = 256: 1 us of 65)
            typedef __attribute__((address_space(1))) Acc global_acc __attribute__((aligned(4)));
            __builtin_nontemporal_store(v, (global_acc*)dst);
        } else {
#pragma unroll
            for (int x = 0; x < 3; ++x)
                if (n0 + c + x < N) dst[x] = v[x];
        }
    }
}

template <int DT, int KW, int SLAB, int NX, bool SHIFTED>
static int launch_lines(const DeviceBcsr& d, const void* B, int64_t ldb, void* C, int64_t ldc, int64_t N, hipStream_t s)
{
    constexpr int ES = Elem<DT>::ES;
    const int step = columns_of_slab<ES, SLAB, SHIFTED>(static_cast<int>(N));
    const dim3 grid(static_cast<unsigned>((d.n_order + 7) / 8 * 8), static_cast<unsigned>((N + step - 1) / step));
    // (from the dword in which B begins to that in which it ends)
    const uint32_t off_dword = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(B) & 3u);
    const uint32_t b_bytes = static_cast<uint32_t>((off_dword + ((d.K - 1) * ldb + N) * ES + 3) / 4 * 4);
    hipLaunchKernelGGL((spmm_lines_kernel<DT, KW, SLAB, NX, SHIFTED>), grid, dim3(64 * KW), KW * kRing * 32 * SLAB, s, d.work, d.slots, d.vals, d.perm,
                       static_cast<const uint8_t*>(B) - off_dword, b_bytes, static_cast<uint32_t>(ldb * ES), static_cast<uint32_t>(d.K),
                       static_cast<typename Elem<DT>::Out*>(C), ldc, static_cast<int>(N), static_cast<int>(d.n_order), off_dword, d.full_packs);
    return static_cast<int>(hipGetLastError());
}

template <int DT, int SLAB, int NX, bool SHIFTED>
static int launch_lines_split(const DeviceBcsr& d, int kw, const void* B, int64_t ldb, void* C, int64_t ldc, int64_t N, hipStream_t s)
{
    switch (kw) {
    case 8: return launch_lines<DT, 8, SLAB, NX, SHIFTED>(d, B, ldb, C, ldc, N, s);
    case 4: return launch_lines<DT, 4, SLAB, NX, SHIFTED>(d, B, ldb, C, ldc, N, s);
    case 2: return launch_lines<DT, 2, SLAB, NX, SHIFTED>(d, B, ldb, C, ldc, N, s);
    default: return launch_lines<DT, 1, SLAB, NX, SHIFTED>(d, B, ldb, C, ldc, N, s);
    }
}

// (n: sixteenths of the columns of a slab, as in kernels_8bit.hip and kernels.hip)
#define SMAT_LINES_NAMES(n, how) {"spmm_" SMAT_LINES_TYPE "_n" n "k1" how, "spmm_" SMAT_LINES_TYPE "_n" n "k2" how, "spmm_" SMAT_LINES_TYPE "_n" n "k4" how, "spmm_" SMAT_LINES_TYPE "_n" n "k8" how}
static const char* const kNames[2][2][4] = {
    {SMAT_LINES_NAMES(SMAT_LINES_N64, "s1c1_lds_l8"), SMAT_LINES_NAMES(SMAT_LINES_N64, "s1c1_ldso_l8")},
    {SMAT_LINES_NAMES(SMAT_LINES_N128, "s1c1_lds_l8"), SMAT_LINES_NAMES(SMAT_LINES_N128, "s1c1_ldso_l8")}};

template <int DT>
int launch_lines_type(const DeviceBcsr& d, const void* B, int64_t ldb, void* C, int64_t ldc, int64_t N, void* stream, const char** variant)
{
    constexpr int ES = Elem<DT>::ES;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool on_dwords = ((ldb * ES) | static_cast<int64_t>(reinterpret_cast<uintptr_t>(B))) % 4 == 0;
    const int64_t span = N * ES + (on_dwords ? 0 : 4 - ES);
    const int slab = span <= 64 ? 64 : 128;
    // a quarter less to read, to move and to multiply where the columns are in three quarters of the slab (50021 rows of a band, 33 columns in bf16
    // off the dwords 7.10 -> 6.68 us, 65 columns in int8 9.25 -> 7.70)
    const bool less = 4 * span <= 3 * slab;
    // Waves per block row: until there are two for every SIMD, as long as a wave has four packs to walk; five where some rows are much longer
    // than the average; and a little later for four waves that move what they read.  (us with 1 / 2 / 4 waves: 1117 block rows of 12 packs, N = 64 10.3 / 7.4
    // / 8.1; 2048 of 21 18.6 / 17.4 / 18.8; 4096 of a graph, 8 on average, 19.9 / 16.5 / 19.2; 166 of 22 9.4 / 6.1 / 4.8.  Moved: 1117 of 38, N = 65 in e4m3
    // 44.4 / 28.0 / 26.1; 2500 of 6, N = 125 in e5m2 12.6 / 13.2 / 14.3; of a graph, N = 33 in fp16 15.6 / 14.0 / 17.0, but N = 125 in int8, which moves
    // four times as much, 20.7 / 22.5 / 25.0; the graph's half, 1875, 15.9 / 11.8 / 12.3.)
    const int64_t units = d.n_order * ((span + slab - 1) / slab);
    const bool skewed = static_cast<double>(d.max_row_packs) > 2.0 * d.mean_row_packs, full = ES == 1 && !on_dwords && span > 96;
    int kw = 1;
    while (kw < 8 && d.mean_row_packs >= 4.0 * kw && units * kw < (skewed ? (full ? 3000 : 5000) : !on_dwords && kw > 1 ? 3000 : 2200)) kw *= 2;
    *variant = kNames[slab == 128][!on_dwords][kw == 8 ? 3 : kw >> 1];
    if (slab == 128) {
        constexpr int NX = 8 / ES;
        if (on_dwords) return less ? launch_lines_split<DT, 128, NX * 3 / 4, false>(d, kw, B, ldb, C, ldc, N, s) : launch_lines_split<DT, 128, NX, false>(d, kw, B, ldb, C, ldc, N, s);
        return less ? launch_lines_split<DT, 128, NX * 3 / 4, true>(d, kw, B, ldb, C, ldc, N, s) : launch_lines_split<DT, 128, NX, true>(d, kw, B, ldb, C, ldc, N, s);
    }
    constexpr int NX = 4 / ES;
    if constexpr (NX == 4) {
        if (less) return on_dwords ? launch_lines_split<DT, 64, 3, false>(d, kw, B, ldb, C, ldc, N, s) : launch_lines_split<DT, 64, 3, true>(d, kw, B, ldb, C, ldc, N, s);
    }
    return on_dwords ? launch_lines_split<DT, 64, NX, false>(d, kw, B, ldb, C, ldc, N, s) : launch_lines_split<DT, 64, NX, true>(d, kw, B, ldb, C, ldc, N, s);
}
template int launch_lines_type<SMAT_LINES_DT>(const DeviceBcsr&, const void*, int64_t, void*, int64_t, int64_t, void*, const char**);

}  // namespace smat
