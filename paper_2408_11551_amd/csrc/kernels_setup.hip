// HIP kernels for gfx950: which row patterns could start a cluster together (preprocess.cpp, Partners).
//
// The pairs of patterns that share block columns are gone through by the lists of the shorter pattern's columns: every longer pattern that a
// list names gets a counter up by one, and the lists are gone through a second time for the counters that reached what the merge test
// asks for at least.  So the work is that of the lists, however many patterns there are.
//
//   * Patterns of more than kShortPattern columns: a workgroup each, exact counters of one or two bytes for a window of the patterns at a
//     time (64 KiB of LDS).  Who comes to a counter first in the second pass takes it, and leaves zero behind.
//   * Shorter ones, which are most of them: a wave each, without a barrier, and 2048 or 8192 counters for all patterns, several to a counter.
//     The few pairs that reach `least` by accident are told by comparing their columns, as are those that do.  (Few as long as the lists are
//     short: launch_partners.)
//
// What bounds it: the lists, read twice each from the L2s, and for a workgroup's pattern two barriers and the trip to its lists between them.  A graph
// of 65536 rows of 16 (52 000 patterns, 134 million pairs of entries): 223 us for the long ones and 216 for the short, 740 with a workgroup for every
// pattern and a global counter of pairs; sixteen host threads 4700-5000.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace smat {

namespace {

constexpr uint32_t kShortPattern = 32;         // (at most 64: a lane per column)
constexpr int kLongThreads = 512, kLongWaves = kLongThreads / 64;
constexpr uint32_t kLongLds = 64 * 1024;
constexpr int kShortThreads = 256, kShortWaves = kShortThreads / 64;
constexpr uint32_t kSketch = 2048, kWideSketch = 8192;      // counters of two bytes per wave
// Partners that a pattern may have as the shorter one; pairs held from which they are put down.
constexpr uint32_t kMostOfLong = 512, kHeldOfLong = 256, kMostOfShort = 128, kHeldOfShort = 64;

struct Pattern { uint32_t first, len, end, least; };

// Pattern k, the first pattern that is too long to be a partner, and the columns that a partner shares at least.
__device__ __forceinline__ Pattern pattern_of(const PartnerTables& t, uint32_t k)
{
    Pattern p;
    p.first = t.ptr[k];
    p.len = t.ptr[k + 1] - p.first;
    const uint64_t too_long = t.keep == 0 ? ~uint64_t{0} : (uint64_t{1000} * p.len + t.keep - 1) / t.keep;
    p.end = too_long > t.longest ? static_cast<uint32_t>(t.n) : t.first_of_len[too_long];
    p.least = static_cast<uint32_t>(uint64_t{2} * t.keep * p.len / (1000 + t.keep)) + 1;       // (all others are as long at least)
    return p;
}

__device__ __forceinline__ bool passes(const PartnerTables& t, uint32_t shared, uint32_t mine, uint32_t theirs)
{
    return uint64_t{1000} * shared > static_cast<uint64_t>(t.keep) * (mine + theirs - shared);
}

// Pairs found by a workgroup or a wave, put down some tens at a time between two patterns.  (One counter for all, in memory, is good for 40 pairs per
// us: 740 us for the graph above, whatever else was done.)  There is room for the most that a pattern may have beside those that are held when it begins.  One with
// more gives the search up: the host's lists no more than a few of each, and all of 20 000 rows that share a column would be 200 million.  A workgroup looks for
// that once per pattern, a wave after 64 comparisons (once per pattern, 50 000 loads of one word took as long as the rest), and ends.  50 000 rows of
// 16 and a column in all of them: 18.0 -> 0.21 ms, most of it as the long ones no longer come first; 20 000 of 40 1.49 -> 0.46; 20 000 of three 1.55 -> 0.14.
template <uint32_t ROOM> struct HeldPairs { uint32_t n, to, pairs[2 * ROOM]; };

template <uint32_t ROOM>
__device__ __forceinline__ void put_pair(HeldPairs<ROOM>& held, uint32_t k, uint32_t other)
{
    const uint32_t at = atomicAdd(&held.n, 1u);
    if (at >= ROOM) return;
    held.pairs[2 * at] = k;
    held.pairs[2 * at + 1] = other;
}

// The two halves of putting them down, which a barrier (a fence, for a wave's) parts; x of `threads` threads.
template <uint32_t ROOM>
__device__ __forceinline__ void make_room(const PartnerTables& t, HeldPairs<ROOM>& held, uint32_t x)
{
    if (x == 0 && held.n > 0) held.to = atomicAdd(t.found, held.n);
}

template <uint32_t ROOM>
__device__ __forceinline__ void put_down(const PartnerTables& t, const HeldPairs<ROOM>& held, uint32_t x, uint32_t threads)
{
    for (; x < held.n; x += threads) {
        const size_t to = static_cast<size_t>(held.to) + x;
        if (to >= t.most_pairs) return;
        t.pairs[2 * to] = held.pairs[2 * x];
        t.pairs[2 * to + 1] = held.pairs[2 * x + 1];
    }
}

__device__ __forceinline__ uint32_t given_up(const PartnerTables& t) { return __hip_atomic_load(t.found + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void give_up(const PartnerTables& t) { atomicOr(t.found + 1, 1u); }

__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane)
{
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), static_cast<int>(lane)));
}

// f(pattern) for the patterns of lists[begin .. stop) in [from, to); from > 0.
template <typename F>
__device__ __forceinline__ void listed(const PartnerTables& t, uint32_t begin, uint32_t stop, uint32_t from, uint32_t to, int lane, F&& f)
{
    for (uint32_t x = begin + static_cast<uint32_t>(lane); x < stop; x += 256) {
        uint32_t other[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) other[u] = x + 64u * u < stop ? t.lists[x + 64u * u] : 0u;
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
            if (other[u] >= from && other[u] < to) f(other[u]);
    }
}

}  // namespace

// Patterns number `first` and above.  BITS: of a counter; no pattern has more than 2^BITS - 1 columns.
template <int BITS>
__global__ __launch_bounds__(kLongThreads)
void long_partners_kernel(PartnerTables t, uint32_t first, uint32_t window)
{
    extern __shared__ uint32_t counts[];
    __shared__ HeldPairs<kMostOfLong + kHeldOfLong> held;
    __shared__ uint32_t enough;
    constexpr uint32_t PER = 32 / BITS, MASK = (1u << BITS) - 1u;
    const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(tid >> 6));
    if (tid == 0) {
        held.n = 0;
        enough = given_up(t);
    }
    for (uint32_t x = static_cast<uint32_t>(tid); x < (window + PER - 1) / PER; x += kLongThreads) counts[x] = 0;
    __syncthreads();
    if (enough) return;
    for (int64_t y = blockIdx.x; y < t.n - first; y += gridDim.x) {
        // a short one to begin with, of which those have too many partners that share a column with thousands; then the long ones, which take longest
        const uint32_t k = y < gridDim.x ? first + static_cast<uint32_t>(y) : static_cast<uint32_t>(t.n - 1 - (y - gridDim.x));
        const Pattern p = pattern_of(t, k);
        const uint32_t held_before = held.n;                         // (pairs are put there behind the first barrier below)
        for (uint32_t w0 = k + 1; w0 < p.end; w0 += window) {
            const uint32_t w1 = min(p.end, w0 + window);
            auto each = [&](auto&& f) __attribute__((always_inline)) {
                for (uint32_t q0 = 0; q0 < p.len; q0 += 64 * kLongWaves) {
                    // a lane asks for the place of a list
                    const uint32_t q = q0 + wave + kLongWaves * static_cast<uint32_t>(lane);
                    uint32_t begin = 0, stop = 0;
                    if (q < p.len) {
                        const uint32_t c = t.columns[p.first + q];
                        begin = t.list_ptr[c];
                        stop = t.list_ptr[c + 1];
                    }
                    for (uint32_t i = 0; i < 64 && q0 + wave + kLongWaves * i < p.len; ++i)
                        listed(t, lane_value(begin, i), lane_value(stop, i), w0, w1, lane, f);
                }
            };
            each([&](uint32_t other) { atomicAdd(&counts[(other - w0) / PER], 1u << (BITS * ((other - w0) % PER))); });
            __syncthreads();
            if (tid == 0) enough = given_up(t);
            each([&](uint32_t other) {
                const uint32_t place = BITS * ((other - w0) % PER);
                const uint32_t shared = atomicAnd(&counts[(other - w0) / PER], ~(MASK << place)) >> place & MASK;
                if (shared >= p.least && passes(t, shared, p.len, t.ptr[other + 1] - t.ptr[other])) put_pair(held, k, other);
            });
            __syncthreads();
            // (uniform: both are written between the barriers only)
            if (enough || held.n - held_before > kMostOfLong) {
                if (tid == 0) give_up(t);
                return;
            }
        }
        // (the last pattern's, or enough of them: uniform, as nobody counts here)
        if (held.n >= kHeldOfLong || y + gridDim.x >= t.n - first) {
            make_room(t, held, static_cast<uint32_t>(tid));
            __syncthreads();
            put_down(t, held, static_cast<uint32_t>(tid), kLongThreads);
            __syncthreads();
            if (tid == 0) held.n = 0;
            __syncthreads();
        }
    }
}

// Patterns below number `last`, of kShortPattern columns at most.  (A counter reaches at most 32 n / 2048: n is below 2^22.)
template <uint32_t SKETCH>
__global__ __launch_bounds__(kShortThreads)
void short_partners_kernel(PartnerTables t, uint32_t last)
{
    __shared__ uint32_t sketches[kShortWaves][SKETCH / 2];
    __shared__ HeldPairs<kMostOfShort + kHeldOfShort> helds[kShortWaves];
    const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(tid >> 6));
    uint32_t* const counts = sketches[wave];
    auto& held = helds[wave];
    if (lane == 0) held.n = 0;
    wave_fence();
    auto empty_hands = [&]() {
        make_room(t, held, static_cast<uint32_t>(lane));
        wave_fence();
        put_down(t, held, static_cast<uint32_t>(lane), 64);
        wave_fence();
        if (lane == 0) held.n = 0;
        wave_fence();
    };
    for (int64_t y = static_cast<int64_t>(blockIdx.x) * kShortWaves + wave; y < last; y += static_cast<int64_t>(gridDim.x) * kShortWaves) {
        const uint32_t k = last - 1 - static_cast<uint32_t>(y);
        const Pattern p = pattern_of(t, k);
        if (p.len == 0) break;                         // the empty pattern is number 0
        const uint32_t held_before = held.n;
        for (uint32_t x = static_cast<uint32_t>(lane); x < SKETCH / 2; x += 64) counts[x] = 0;
        uint32_t column = 0, begin = 0, stop = 0;
        if (static_cast<uint32_t>(lane) < p.len) {
            column = t.columns[p.first + static_cast<uint32_t>(lane)];
            begin = t.list_ptr[column];
            stop = t.list_ptr[column + 1];
        }
        wave_fence();
        for (uint32_t q = 0; q < p.len; ++q)
            listed(t, lane_value(begin, q), lane_value(stop, q), k + 1, p.end, lane,
                   [&](uint32_t other) { atomicAdd(&counts[other % SKETCH / 2], 1u << (16 * (other % 2))); });
        wave_fence();
        uint32_t compared = 0;
        auto too_many = [&]() {
            wave_fence();
            const bool more = held.n - held_before > kMostOfShort;
            if (more && lane == 0) give_up(t);
            return more;
        };
        for (uint32_t q = 0; q < p.len; ++q) {
            const uint32_t from = lane_value(begin, q), to = lane_value(stop, q);
            for (uint32_t x0 = from; x0 < to; x0 += 256) {
                const uint32_t x = x0 + static_cast<uint32_t>(lane);
                uint32_t named[4];
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) named[u] = x + 64u * u < to ? t.lists[x + 64u * u] : 0u;
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    const uint32_t other = named[u];
                    // columns shared, or more
                    const uint32_t most = other > k && other < p.end ? min(counts[other % SKETCH / 2] >> (16 * (other % 2)) & 0xFFFFu, p.len) : 0u;
                    const bool may = most >= p.least && passes(t, most, p.len, t.ptr[other + 1] - t.ptr[other]);
                    for (uint64_t left = __ballot(may); left; left &= left - 1, ++compared) {
                        const uint32_t who = lane_value(other, static_cast<uint32_t>(__builtin_ctzll(left)));
                        const uint32_t at = t.ptr[who], their = t.ptr[who + 1] - at;
                        // the columns that both have, and the first of them: the pair is found once
                        uint64_t both = 0;
                        for (uint32_t z = 0; z < their; z += 64) {
                            const uint32_t c = z + static_cast<uint32_t>(lane) < their ? t.columns[at + z + static_cast<uint32_t>(lane)] : ~0u;
                            for (uint32_t m = 0; m < p.len; ++m)
                                if (__ballot(c == lane_value(column, m))) both |= uint64_t{1} << m;
                        }
                        if (static_cast<uint32_t>(__builtin_ctzll(both)) == q && lane == 0 &&
                            passes(t, static_cast<uint32_t>(__builtin_popcountll(both)), p.len, their))
                            put_pair(held, k, who);
                    }
                }
                // (here too: a pattern that shares a column with thousands is compared with them one by one)
                if (compared >= 64) {
                    compared = 0;
                    if (too_many() || __builtin_amdgcn_readfirstlane(static_cast<int>(given_up(t)))) return;
                }
            }
        }
        if (too_many()) return;
        if (held.n >= kHeldOfShort) empty_hands();
    }
    empty_hands();
}

int launch_partners(const PartnerTables& t, uint32_t first_long, double mean_list, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    // A counter holds mean_list / counters per column of a pattern by accident and a partner at least 2 keep / (1000 + keep), whatever the pattern's length.  Above
    // a third of that ever more pairs have to be told by their columns: 4200 rows of 50 (lists of 700) 1930 us with 2048 counters, 104 with 8192, which hold
    // four times the lists; a graph of rows of 16 (lists of 256) 197 with 2048.
    const double most_list = 0.35 * 2.0 * t.keep / (1000.0 + t.keep);
    const uint32_t sketch = mean_list <= most_list * kSketch ? kSketch : kWideSketch;
    if (mean_list > most_list * kWideSketch && t.n > kWideSketch) first_long = 0;
    // (short patterns first: where a search is given up it is mostly theirs, and the other kernel ends at once)
    if (first_long > 0) {
        const uint32_t groups = (first_long + kShortWaves - 1) / kShortWaves;
        const dim3 grid(groups < 2048 ? groups : 2048);
        if (sketch == kSketch) hipLaunchKernelGGL(short_partners_kernel<kSketch>, grid, dim3(kShortThreads), 0, s, t, first_long);
        else hipLaunchKernelGGL(short_partners_kernel<kWideSketch>, grid, dim3(kShortThreads), 0, s, t, first_long);
    }
    if (t.n > first_long) {
        const bool bytes = t.longest < 256;
        const uint32_t counter = bytes ? 1 : 2, most = kLongLds / counter, left = static_cast<uint32_t>(t.n) - first_long;
        const uint32_t window = left < most ? (left + 3) / 4 * 4 : most;
        const dim3 grid(left < 768 ? left : 768);
        if (bytes) hipLaunchKernelGGL(long_partners_kernel<8>, grid, dim3(kLongThreads), window * counter, s, t, first_long, window);
        else hipLaunchKernelGGL(long_partners_kernel<16>, grid, dim3(kLongThreads), window * counter, s, t, first_long, window);
    }
    return static_cast<int>(hipGetLastError());
}

uint32_t short_pattern() { return kShortPattern; }

}  // namespace smat
