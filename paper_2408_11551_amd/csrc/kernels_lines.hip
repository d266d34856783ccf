// HIP kernel for gfx950: the per-row kernel (spmm_rows.h) for rows of B on whole cache lines, gathered through LDS.
//
// Work split: a workgroup of KW waves takes one block row and one slab of 128 bytes of every row of B (64 columns, or 128 of the
// 8-bit types); wave ks walks packs ks, ks + KW, ... of the block row, the partial tiles are summed through LDS in a fixed order.
//
// What bounds products of sparse matrices is the gather of B, and what bounds that is how many cache lines a compute unit may wait for at a
// time, so it goes the faster the more of them are in the L2: 16-byte loads of rows of 128 bytes from a table of 2 / 4 / 8 / 16 MB come in
// at 24.4 / 22.8 / 13.6 / 9.7 TB/s, and just so in rows of 256 (8-byte loads: 13.0 / 13.0 / 12.2 / 9.2).  Slabs of one line make that
// table as small as it can be, but sixteen lanes that fetch eight bytes each, as the matrix instruction would have it, do not: here eight
// lanes fetch a row's line with sixteen bytes each, straight into LDS, and the transposing reads make the operand from there, without the
// permutes that the other kernel spends on it.
#include <algorithm>
#include <cstdio>
#include <type_traits>
#include <utility>

#include <hip/hip_runtime.h>

#include "kernels.h"
#include "mfma_types.h"
#include "pack_layout.h"
#include "tile_common.h"

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
    static_assert(N == 8 || N == 4, "");
    if constexpr (N == 8)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]));
    else
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
}

struct LineWalk {
    const uint32_t* slots;
    const uint8_t* vals;
    int npacks, ks, lane;
    uint32_t first_byte, bytes;        // of the slab in a row of B: where it begins, and how many there are of the row from there on
    uint32_t ldb_bytes, K, lds;
};

// The packs of a row of class L (pack_layout.h) or of an entry row.  A pack's rows of B lie in LDS in the order of its slot table, 128
// bytes each; 16-byte piece p of row (g, kk) -- lane group and position -- at p ^ swizzle, so that the 32 lanes that LDS serves at a time
// meet every bank once.
template <int DT, int KW, int L, bool ENTRY>
__device__ __forceinline__ void walk_lines(const LineWalk& w, __amdgpu_buffer_rsrc_t b_rsrc, typename Elem<DT>::Acc (&acc)[8 / Elem<DT>::ES])
{
    constexpr int ES = Elem<DT>::ES, NX = 8 / ES;          // NX groups of sixteen columns
    constexpr int NL = L / 2;                              // loads of eight rows per pack
    constexpr int AB = (ENTRY ? 8 : L) * ES;               // bytes of values per lane
    constexpr uint32_t kPackValues = ENTRY ? 64u : 64u * L * ES, kPackSlots = 16u * L;
    const int lane = w.lane, i = lane & 15, g = lane >> 4;
    const int count = w.ks < w.npacks ? (w.npacks - w.ks + KW - 1) / KW : 0;
    if (count == 0) return;
    const __amdgpu_buffer_rsrc_t slots_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w.slots), 0, w.npacks * static_cast<int>(kPackSlots), kRsrcFlags);
    const __amdgpu_buffer_rsrc_t vals_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(w.vals), 0, w.npacks * static_cast<int>(kPackValues), kRsrcFlags);
    auto swizzle = [](int g_, int kk) { return ES == 2 ? 2 * (((kk & 3) >> 1) + 2 * (g_ & 1)) : (kk >> 1) + 4 * (g_ & 1); };
    // Load e: rows 8 e ... 8 e + 7 of the table, lane l the piece l % 8 of row 8 e + l / 8.
    uint32_t src_off[NL], from_lane[NL];
#pragma unroll
    for (int e = 0; e < NL; ++e) {
        const int at = 8 * e + (lane >> 3);
        const uint32_t byte = 16u * static_cast<uint32_t>((lane & 7) ^ swizzle(at / L, at % L));
        src_off[e] = byte < w.bytes ? w.first_byte + byte : kOutOfRange;
        from_lane[e] = 4u * static_cast<uint32_t>(at);
    }
    // Reads of group of columns x: 16-bit types kk = 0 .. 3 and, 512 bytes on, 4 .. 7; 8-bit types all eight
    uint32_t tr_addr[NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) {
        const int kk = (ES == 2 ? i >> 2 : i >> 1) & (L - 1);
        const int piece = ES == 2 ? (2 * x) ^ swizzle(g, kk) : x ^ swizzle(g, kk);
        tr_addr[x] = w.lds + static_cast<uint32_t>(L * g + kk) * 128u + 16u * static_cast<uint32_t>(piece) + 8u * (ES == 2 ? i & 3 : i & 1);
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
            load_to_lds16((lds_void*)(uintptr_t)(w.lds + 4096u * static_cast<uint32_t>(buf) + 1024u * e), b_rsrc, __umul24(live ? m : w.K, w.ldb_bytes) + src_off[e], 0u);
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

    uint32_t raw[kRing], row_numbers[kRing];
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
        __builtin_amdgcn_sched_barrier(0);
    }
    auto step = [&](auto u_, int s) __attribute__((always_inline)) {
        constexpr int u = decltype(u_)::value, next = (u + kAhead) % kRing;
        a[next] = load_values(s + kAhead);
        const uint32_t rows = raw[next];
        raw[(u + 2 * kAhead) % kRing] = load_slots(s + 2 * kAhead);
        __builtin_amdgcn_sched_barrier(0);
        row_numbers[next] = load_rows(s + kAhead, rows, next);
        __builtin_amdgcn_sched_barrier(0);
        // What was asked for before the loads of the packs ahead is there.  Counted are those into LDS alone: of the others the compiler takes out
        // what nothing reads any more at the end of a walk.
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"(kAhead * NL));
        __builtin_amdgcn_sched_barrier(0);
        u32x2_t v[8];
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            if constexpr (ES == 2) {
                v[2 * x] = lds_read_tr<4096 * u>(tr_addr[x]);
                if constexpr (L == 8) v[2 * x + 1] = lds_read_tr<4096 * u + 512>(tr_addr[x]);
                else v[2 * x + 1] = u32x2_t{0u, 0u};
            } else {
                v[x] = lds_read_tr8<4096 * u>(tr_addr[x]);
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
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            u32x4 b = ES == 2 ? u32x4{v[2 * x][0], v[2 * x][1], v[2 * x + 1][0], v[2 * x + 1][1]} : u32x4{v[x][0], v[x][1], 0u, 0u};
            // (positions past L hold another row's elements)
            if constexpr (L == 2) b = u32x4{ES == 2 ? b[0] : b[0] & 0xFFFFu, 0u, 0u, 0u};
            if constexpr (L == 4 && ES == 1) b[1] = 0u;
            acc[x] = mfma_pack<DT>(av, b, acc[x]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto several = [&](int s, int n, auto... u) __attribute__((always_inline)) { (void)((decltype(u)::value < n && (step(u, s + decltype(u)::value), true)) && ...); };
    const int iters = count / kRing, rem = count % kRing;
    for (int it = 0; it < iters; ++it) with_constants(std::make_integer_sequence<int, kRing>{}, [&](auto... u) __attribute__((always_inline)) { several(kRing * it, kRing, u...); });
    with_constants(std::make_integer_sequence<int, kRing - 1>{}, [&](auto... u) __attribute__((always_inline)) { several(kRing * iters, rem, u...); });
}

}  // namespace

template <int DT, int KW>
__global__ __launch_bounds__(64 * KW)
void spmm_lines_kernel(const int32_t* __restrict__ work, const uint32_t* __restrict__ slots, const void* __restrict__ vals,
                       const int32_t* __restrict__ perm, const void* __restrict__ B, uint32_t b_bytes, uint32_t ldb_bytes,
                       uint32_t K, typename Elem<DT>::Out* __restrict__ C, int64_t ldc, int N, int n_order)
{
    using Acc = typename Elem<DT>::Acc;
    using Out = typename Elem<DT>::Out;
    constexpr int ES = Elem<DT>::ES, COLS = 128 / ES, NX = 8 / ES;
    constexpr int LD = COLS + (ES == 2 ? 4 : 0);           // row of a tile on its way out, words (padded where there is room)
    static_assert(16 * LD * 4 <= kRing * 4096, "a tile takes the place of the rows of B");
    extern __shared__ u32x4 lds_dyn[];
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int ks = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    // The (slab, block row) pairs, slab by slab, dealt to the eight XCDs in contiguous shares, as kSlabsByXcd does in spmm_rows.h: an XCD's L2 has to
    // hold few slabs, each of them 128 K bytes (27350 rows of 12 entries, N = 960: 71 us with the slabs in turn, 49 like this).
    const uint32_t share = (blockIdx.x & 7u) * gridDim.y + blockIdx.y, record = (blockIdx.x & ~7u) | (share & 7u), slab = share >> 3;
    if (record >= static_cast<uint32_t>(n_order)) return;
    const i32x4 rec = reinterpret_cast<const i32x4*>(work)[record];
    const int br = rec[0] & 0x0FFFFFFF, cls = rec[0] >> 28;
    const int n0 = static_cast<int>(slab) * COLS;
    LineWalk w;
    w.slots = slots + static_cast<size_t>(static_cast<uint32_t>(rec[2])) * 8;
    w.vals = static_cast<const uint8_t*>(vals) + static_cast<size_t>(static_cast<uint32_t>(rec[3])) * 64;
    w.npacks = rec[1];
    w.ks = ks;
    w.lane = lane;
    w.first_byte = slab * 128u;
    w.bytes = static_cast<uint32_t>(N - n0) * ES;
    w.ldb_bytes = ldb_bytes;
    w.K = K;
    w.lds = lds_offset_of(lds_dyn) + static_cast<uint32_t>(ks) * (kRing * 4096u);
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(B), 0, static_cast<int>(b_bytes), kRsrcFlags);
    // where this thread's pieces of four columns go: asked for now
    constexpr int Q = COLS / 4, EP = (16 * Q + 64 * KW - 1) / (64 * KW);
    int out_rows[EP];
#pragma unroll
    for (int k = 0; k < EP; ++k) out_rows[k] = static_cast<int>(threadIdx.x) + 64 * KW * k < 16 * Q ? perm[br * 16 + (static_cast<int>(threadIdx.x) + 64 * KW * k) / Q] : -1;
    Acc acc[NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) acc[x] = Acc{0, 0, 0, 0};
    if (cls == 2) walk_lines<DT, KW, 8, false>(w, b_rsrc, acc);
    else if (cls == kEntryClass) walk_lines<DT, KW, 8, true>(w, b_rsrc, acc);
    else if (cls == 1) walk_lines<DT, KW, 4, false>(w, b_rsrc, acc);
    else walk_lines<DT, KW, 2, false>(w, b_rsrc, acc);
    // nothing may still be on its way into LDS
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)");
    __builtin_amdgcn_sched_barrier(0);

    // acc[x][y] = C'[4 g + y][n0 + 16 x + i] of this wave's packs
    Out* const tile = reinterpret_cast<Out*>(reinterpret_cast<uint8_t*>(lds_dyn) + static_cast<size_t>(ks) * (kRing * 4096));
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) tile[(4 * g + y) * LD + 16 * x + i] = acc[x][y];
    if constexpr (KW == 1) __builtin_amdgcn_wave_barrier();
    else __syncthreads();
#pragma unroll
    for (int k = 0; k < EP; ++k) {
        const int e = static_cast<int>(threadIdx.x) + 64 * KW * k, row = e / Q, c = 4 * (e % Q);
        if (e >= 16 * Q) break;
        const Out* src = reinterpret_cast<const Out*>(lds_dyn) + row * LD + c;
        Acc v = *reinterpret_cast<const Acc*>(src);
#pragma unroll
        for (int x = 1; x < KW; ++x) v += *reinterpret_cast<const Acc*>(src + x * (kRing * 1024));
        const int64_t out_row = out_rows[k];
        if (out_row < 0 || n0 + c >= N) continue;
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

template <int DT, int KW>
static int launch_lines(const DeviceBcsr& d, const void* B, int64_t ldb, void* C, int64_t ldc, int64_t N, hipStream_t s)
{
    constexpr int ES = Elem<DT>::ES;
    const dim3 grid(static_cast<unsigned>((d.n_order + 7) / 8 * 8), static_cast<unsigned>((N * ES + 127) / 128));
    // (the end of B rounded up to a dword, which rows on whole lines have)
    const uint32_t b_bytes = static_cast<uint32_t>((((d.K - 1) * ldb + N) * ES + 3) / 4 * 4);
    hipLaunchKernelGGL((spmm_lines_kernel<DT, KW>), grid, dim3(64 * KW), KW * kRing * 4096, s, d.work, d.slots, d.vals, d.perm, B, b_bytes,
                       static_cast<uint32_t>(ldb * ES), static_cast<uint32_t>(d.K), static_cast<typename Elem<DT>::Out*>(C), ldc,
                       static_cast<int>(N), static_cast<int>(d.n_order));
    return static_cast<int>(hipGetLastError());
}

template <int DT>
static int launch_lines_dtype(const DeviceBcsr& d, const void* B, int64_t ldb, void* C, int64_t ldc, int64_t N, hipStream_t s, const char** variant)
{
    constexpr int ES = Elem<DT>::ES;
    // Waves per block row: until there are two for every SIMD, as long as a wave has four packs to walk; five where some rows are much longer
    // than the average.  (us with 1 / 2 / 4 waves: 1117 block rows of 12 packs, N = 64 10.3 / 7.4 / 8.1; 2048 of 21 18.6 / 17.4 / 18.8; 4096 of
    // a graph, 8 on average, 19.9 / 16.5 / 19.2; 166 of 22 9.4 / 6.1 / 4.8.)
    const int64_t units = d.n_order * ((N * ES + 127) / 128);
    const double enough = static_cast<double>(d.max_row_packs) > 2.0 * d.mean_row_packs ? 5000.0 : 2200.0;
    int kw = 1;
    while (kw < 8 && d.mean_row_packs >= 4.0 * kw && static_cast<double>(units * kw) < enough) kw *= 2;
    // (n: sixteenths of the columns of a slab, as there)
    static thread_local char name[40];
    snprintf(name, sizeof(name), "spmm_%s_n%dk%ds1c1_lds_l8", DT == kF16 ? "f16" : DT == kBF16 ? "bf16" : DT == kE4M3 ? "e4m3" : DT == kE5M2 ? "e5m2" : "i8", 8 / ES, kw);
    *variant = name;
    switch (kw) {
    case 8: return launch_lines<DT, 8>(d, B, ldb, C, ldc, N, s);
    case 4: return launch_lines<DT, 4>(d, B, ldb, C, ldc, N, s);
    case 2: return launch_lines<DT, 2>(d, B, ldb, C, ldc, N, s);
    default: return launch_lines<DT, 1>(d, B, ldb, C, ldc, N, s);
    }
}

int launch_spmm_lines(const DeviceBcsr& d, int dtype, const void* B, int64_t ldb, void* C, int64_t ldc, int64_t N, void* stream, const char** variant)
{
    const int es = dtype == kF16 || dtype == kBF16 ? 2 : 1;
    const int64_t bytes = N * es;
    // rows of B on whole lines, and more than half of one; block rows with packs of 32 slots, and not a few of them (which are a launch and little else)
    if (d.n_order < 64 || d.K == 0 || d.max_class < 2 || bytes <= 64 || bytes > 128 * 65535) return kNotLines;
    if ((ldb * es) % 128 != 0 || reinterpret_cast<uintptr_t>(B) % 128 != 0) return kNotLines;
    // A single slab is faster here throughout (2048 block rows of 21 packs, K = 32768, N = 64 in fp16 19.1 -> 17.4 us, N = 128 in e4m3 20.5 -> 15.9; a
    // graph of 65536 rows, N = 64 19.1 -> 16.5).  Several slabs read A once for each, where the other kernel's are twice as wide.  It has no
    // use for narrow ones where it keeps long rows in step (2048 block rows of 21 packs, N = 256 47 against 62 us), and rows kept by entry,
    // which are expanded once per slab, are for narrow ones only where wide ones do not fit the L2s (us there and here: 40000 rows of 25
    // entries, N = 256 48.8, 39.3; 27350 of 12, N = 960 70.3, 49.1; 16384 of 16, N = 512 22.7, 23.9; 12000 of 30, N = 512 24.1, 28.4; 4000 of 20, N = 4032 37.8,
    // 46.1).  Rows kept by column: 627 block rows of 7 packs, N = 1024 33.3, 26.0; 1117 of 12, N = 512 39.5, 38.0; 1700 of 17, N = 256 39.1, 43.2.
    const bool entries = d.max_class == kEntryClass;
    if (bytes > 128 && (d.mean_row_packs >= (entries ? 16.0 : 14.0) || (entries && static_cast<double>(d.K) * 256.0 < 5.0e6))) return kNotLines;
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (dtype) {
    case kF16: return launch_lines_dtype<kF16>(d, B, ldb, C, ldc, N, s, variant);
    case kBF16: return launch_lines_dtype<kBF16>(d, B, ldb, C, ldc, N, s, variant);
    case kE4M3: return launch_lines_dtype<kE4M3>(d, B, ldb, C, ldc, N, s, variant);
    case kE5M2: return launch_lines_dtype<kE5M2>(d, B, ldb, C, ldc, N, s, variant);
    default: return launch_lines_dtype<kI8>(d, B, ldb, C, ldc, N, s, variant);
    }
}

}  // namespace smat
