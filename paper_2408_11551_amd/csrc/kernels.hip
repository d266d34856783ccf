// HIP kernels for gfx950 (CDNA4, wave64): device-side BCSR value fill and the 16-bit
// instantiations (fp16, bf16) of the per-row SpMM kernel (spmm_rows.h); the 8-bit ones are
// in kernels_8bit.hip.
#include "lines_rule.h"
#include "spmm_rows.h"

namespace smat {

// ---------------------------------------------------------------------------
// bind-time kernels
// ---------------------------------------------------------------------------
__global__ void fill_zero_kernel(u32x4* dst, size_t n16)
{
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n16; i += stride)
        dst[i] = u32x4{0u, 0u, 0u, 0u};
}

int launch_fill_zero(void* dst, size_t n16, void* stream)
{
    if (n16 == 0) return 0;
    const int threads = 256;
    const size_t want = (n16 + threads - 1) / threads;
    const int blocks = static_cast<int>(want < 8192 ? want : 8192);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(threads), 0, static_cast<hipStream_t>(stream),
                       static_cast<u32x4*>(dst), n16);
    return static_cast<int>(hipGetLastError());
}

// Bind-time: the values of a block row and, with it, its slot table (pack_layout.h), one workgroup per block row, sixteen threads per
// row.  What bounds a bind is the host and the copies to the device, so the tables are made here from what is copied anyway
// (65536 rows, 1.05 M entries: 21 ms when the host made and sent them).
// Block rows kept by column: each entry's block is found by binary search over the block row's ascending block columns, its
// place is the entry's slot in the block's pack; the slot table is written block by block.  Block rows kept by entry: the entries of the
// block row are numbered by column, then by row; an entry's number is the count of those before it, row by row of the
// block row.  The slot table was filled with K; an entry turns the K of its word into its column and adds its row number to the top byte
// of a word of its lane group, both by exclusive-or, so the order does not matter.
// The CSR values arrive as 16-bit words; T is the stored element (the 8-bit types keep the low byte).
constexpr int kEntryColumns = 4096;          // entries of a block row whose columns are kept in shared memory

template <typename T>
__global__ __launch_bounds__(256)
void bcsr_fill_kernel(DeviceBcsr d, const int64_t* __restrict__ csr_row_ptr, const int32_t* __restrict__ csr_col_idx,
                      const uint16_t* __restrict__ csr_vals, const int32_t* __restrict__ col_perm, T* __restrict__ vals_out,
                      uint32_t* __restrict__ slots_out)
{
    __shared__ int32_t columns[kEntryColumns];
    __shared__ int64_t first[16];            // the rows' entries in the CSR arrays
    __shared__ int count_to[17];             // entries of the rows before
    const int64_t br = blockIdx.x;
    const int npacks = d.pack_ptr[br + 1] - d.pack_ptr[br];
    if (npacks == 0) return;
    const int cls = d.row_class[br];
    T* row_vals = vals_out + static_cast<size_t>(d.vals_off[br]) * (64 / sizeof(T));
    uint32_t* table = slots_out + static_cast<size_t>(d.slots_off[br]) * 8;
    auto b_row = [&](int c) { return static_cast<uint32_t>(col_perm ? col_perm[c] : c); };
    if (cls != kEntryClass) {
        const int lo0 = d.blk_ptr[br], hi0 = d.blk_ptr[br + 1];
        const int L = 2 << cls;
        for (int s = lo0 + static_cast<int>(threadIdx.x); s < hi0; s += 256) {
            const uint32_t meta = d.blk_meta[s];
            int rank = static_cast<int>(meta >> 16);
            for (uint32_t mask = meta & 0xFFFFu; mask; mask &= mask - 1u, ++rank)
                table[static_cast<size_t>(d.blk_pack[s]) * (4 * L) + slot_group(rank) * L + slot_pos(rank)] =
                    b_row(d.blk_col[s] * 16 + __ffs(mask) - 1);
        }
        const int rr = static_cast<int>(threadIdx.x >> 4);
        const int64_t i = br * 16 + rr;
        if (i >= d.M) return;
        const int64_t r = d.perm[i], p1 = csr_row_ptr[r + 1];
        int hint = lo0;
        for (int64_t p = csr_row_ptr[r] + (threadIdx.x & 15); p < p1; p += 16) {
            const int c = csr_col_idx[p];
            const int bc = c >> 4;
            int lo = hint, hi = hi0;                 // columns ascend, so the block never moves back
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (d.blk_col[mid] < bc) lo = mid + 1; else hi = mid;
            }
            hint = lo;
            const uint32_t meta = d.blk_meta[lo];
            const int rank = static_cast<int>(meta >> 16) + __popc(meta & 0xFFFFu & ((1u << (c & 15)) - 1u));
            row_vals[static_cast<size_t>(d.blk_pack[lo]) * pack_elems(L) + pack_elem_index(L, rr, slot_group(rank), slot_pos(rank))] =
                static_cast<T>(csr_vals[p]);
        }
        return;
    }
    if (threadIdx.x < 16) {
        const int64_t i = br * 16 + threadIdx.x;
        const int64_t r = i < d.M ? d.perm[i] : -1;
        first[threadIdx.x] = r >= 0 ? csr_row_ptr[r] : 0;
        count_to[threadIdx.x + 1] = r >= 0 ? static_cast<int>(csr_row_ptr[r + 1] - csr_row_ptr[r]) : 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        count_to[0] = 0;
        for (int j = 1; j <= 16; ++j) count_to[j] += count_to[j - 1];
    }
    __syncthreads();
    const int n = count_to[16];
    const bool local = n <= kEntryColumns;
    auto row_of = [&](int x) {
        int j = 0;
        for (int step = 8; step; step >>= 1)
            if (count_to[j + step] <= x) j += step;
        return j;
    };
    if (local) {
        for (int x = threadIdx.x; x < n; x += 256) {
            const int j = row_of(x);
            columns[x] = csr_col_idx[first[j] + (x - count_to[j])];
        }
        __syncthreads();
    }
    for (int x = threadIdx.x; x < n; x += 256) {
        const int rr = row_of(x);
        const int64_t p = first[rr] + (x - count_to[rr]);
        const int c = csr_col_idx[p];
        int e = 0;
        for (int j = 0; j < 16; ++j) {
            const int below = j < rr ? c + 1 : c;      // columns that come before (c, this row) in row j
            int lo = 0, hi = count_to[j + 1] - count_to[j];
            const int32_t* row = csr_col_idx + first[j];
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if ((local ? columns[count_to[j] + mid] : row[mid]) < below) lo = mid + 1; else hi = mid;
            }
            e += lo;
        }
        const int rank = e & 31, g = slot_group(rank), kk = slot_pos(rank);
        row_vals[static_cast<size_t>(e >> 5) * (64 / sizeof(T)) + entry_elem_index(g, kk)] = static_cast<T>(csr_vals[p]);
        uint32_t* group = table + static_cast<size_t>(e >> 5) * 32 + g * 8;
        atomicXor(&group[kk], static_cast<uint32_t>(d.K) ^ b_row(c));
        atomicXor(&group[kk >> 1], static_cast<uint32_t>(rr) << (24 + 4 * (kk & 1)));
    }
}

__global__ void fill_word_kernel(uint32_t* dst, uint32_t word, size_t n)
{
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = word;
}

int launch_bcsr_fill(const DeviceBcsr& d, const int64_t* csr_row_ptr, const int32_t* csr_col_idx, const uint16_t* csr_vals,
                     const int32_t* col_perm, void* vals_out, uint32_t* slots_out, size_t slot_words, int elem_bytes, void* stream)
{
    if (d.M == 0) return 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (slot_words > 0)
        hipLaunchKernelGGL(fill_word_kernel, dim3(static_cast<unsigned>(std::min<size_t>((slot_words + 255) / 256, 8192))), dim3(256), 0, s,
                           slots_out, static_cast<uint32_t>(d.K), slot_words);
    const dim3 grid(static_cast<unsigned>(d.nbr));
    if (elem_bytes == 1)
        hipLaunchKernelGGL(bcsr_fill_kernel<uint8_t>, grid, dim3(256), 0, s, d, csr_row_ptr, csr_col_idx, csr_vals, col_perm,
                           static_cast<uint8_t*>(vals_out), slots_out);
    else
        hipLaunchKernelGGL(bcsr_fill_kernel<uint16_t>, grid, dim3(256), 0, s, d, csr_row_ptr, csr_col_idx, csr_vals, col_perm,
                           static_cast<uint16_t*>(vals_out), slots_out);
    return static_cast<int>(hipGetLastError());
}

int launch_spmm(const DeviceBcsr& d, int dtype, const void* B, int64_t ldb, void* C, int64_t ldc,
                int64_t N, void* stream, const char** variant)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int narrow = launch_spmm_narrow(d, dtype, B, ldb, C, ldc, N, stream, variant);
    if (narrow != kNotNarrow) return narrow;
    if (takes_lines(d, dtype == kF16 || dtype == kBF16 ? 2 : 1, B, ldb, N)) {
        switch (dtype) {
        case kF16: return launch_lines_type<kF16>(d, B, ldb, C, ldc, N, stream, variant);
        case kBF16: return launch_lines_type<kBF16>(d, B, ldb, C, ldc, N, stream, variant);
        case kE4M3: return launch_lines_type<kE4M3>(d, B, ldb, C, ldc, N, stream, variant);
        case kE5M2: return launch_lines_type<kE5M2>(d, B, ldb, C, ldc, N, stream, variant);
        default: return launch_lines_type<kI8>(d, B, ldb, C, ldc, N, stream, variant);
        }
    }
    switch (dtype) {
    case kF16: return launch_dtype<kF16>(d, B, ldb, C, ldc, N, s, variant);
    case kBF16: return launch_dtype<kBF16>(d, B, ldb, C, ldc, N, s, variant);
    case kE4M3: return launch_spmm_e4m3(d, B, ldb, C, ldc, N, stream, variant);
    case kE5M2: return launch_spmm_e5m2(d, B, ldb, C, ldc, N, stream, variant);
    case kI8: return launch_spmm_i8(d, B, ldb, C, ldc, N, stream, variant);
    default: return static_cast<int>(hipErrorInvalidValue);
    }
}

}  // namespace smat
