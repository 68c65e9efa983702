// Stable LSD radix sort of (key, value) pairs, up to 8 bits per pass.
//
// Used where particles arrive in arbitrary order: encoding float input into
// the cell-ordered state (Sec. III-A, stable with respect to the input order)
// and the fallback compaction when a particle moves more than one coarse cell
// in a step.  Each pass: per-tile digit histograms, one exclusive scan over
// the digit-major histogram, then a stable scatter.
//
// A pass is bound by memory (a key read for the histogram, a pair read and
// written by the scatter), so the number of passes decides: 8 bits a pass
// instead of 4, the key bits shared evenly by the passes (21 bits: 7, 7, 7).
// A tile's pairs are put in digit order in LDS before they are stored, so the
// stores of one digit are consecutive.  11.2 million pairs of 21 bits: six
// 4-bit passes 0.69 ms, three of these 0.25.
#include <utility>

#include "common.h"

namespace cube {

namespace {

constexpr int kSortThreads = 512;
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kMaxBits = 8;
constexpr int kMaxDigits = 1 << kMaxBits;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kWaveTile = kSortTile / kSortWaves;     // consecutive pairs of one wave

__global__ __launch_bounds__(kSortThreads) void k_digit_hist(const uint32_t* __restrict__ key, int64_t n,
                                                              int shift, int digits, int64_t nb,
                                                              int32_t* __restrict__ hist) {
    __shared__ int cnt[kMaxDigits];
    if (threadIdx.x < kMaxDigits) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    uint32_t k[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const int64_t e = base + it * kSortThreads + threadIdx.x;
        k[it] = e < n ? key[e] : 0u;
    }
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const int64_t e = base + it * kSortThreads + threadIdx.x;
        if (e < n) atomicAdd(&cnt[(k[it] >> shift) & (digits - 1)], 1);
    }
    __syncthreads();
    if ((int)threadIdx.x < digits) hist[(int64_t)threadIdx.x * nb + blockIdx.x] = cnt[threadIdx.x];
}

// IOTA: the values are the indices (the first pass of an index sort)
template <bool IOTA>
__global__ __launch_bounds__(kSortThreads) void k_digit_scatter(
    const uint32_t* __restrict__ key, const uint32_t* __restrict__ val, int64_t n, int shift, int bits, int64_t nb,
    const int32_t* __restrict__ base_of, uint32_t* __restrict__ key_out, uint32_t* __restrict__ val_out) {
    __shared__ uint32_t buf[kSortTile];
    __shared__ int wc[kSortWaves][kMaxDigits];     // pairs of a wave's part, then its first slot, per digit
    __shared__ int to_global[kMaxDigits];          // a digit's output position minus its position in the tile
    __shared__ int s_scan[kSortThreads / kWave + 1];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    const uint64_t lt = (1ull << lane) - 1ull;
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    const int64_t wbase = base + (int64_t)wid * kWaveTile;
    const int digits = 1 << bits;
    for (int i = threadIdx.x; i < kSortWaves * kMaxDigits; i += kSortThreads) (&wc[0][0])[i] = 0;
    uint32_t k[kSortItems], v[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const int64_t e = wbase + it * kWave + lane;
        k[it] = e < n ? key[e] : 0u;
        v[it] = IOTA ? (uint32_t)e : e < n ? val[e] : 0u;
    }
    __syncthreads();
    // rank among the wave's pairs of the same digit, in input order: the
    // lanes with this digit are found bit by bit, their count so far is in LDS
    int rank[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const bool ok = wbase + it * kWave + lane < n;
        const int d = (int)(k[it] >> shift) & (digits - 1);
        uint64_t same = __ballot(ok);
#pragma unroll
        for (int b = 0; b < kMaxBits; ++b) {
            const uint64_t m = __ballot((d >> b) & 1);
            same &= (d >> b) & 1 ? m : ~m;
        }
        const int before = __popcll(same & lt);
        // every lane reads the count so far before the first of its digit raises it
        const int so_far = wc[wid][d];
        rank[it] = so_far + before;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (ok && before == 0) wc[wid][d] = so_far + __popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // first slot of every (digit, wave) in the tile's digit order
    int mine = 0;
    if ((int)threadIdx.x < digits)
        for (int w = 0; w < kSortWaves; ++w) mine += wc[w][threadIdx.x];
    int total;
    int first = block_exclusive_scan(mine, s_scan, &total);
    if ((int)threadIdx.x < digits) {
        to_global[threadIdx.x] = base_of[(int64_t)threadIdx.x * nb + blockIdx.x] - first;
        for (int w = 0; w < kSortWaves; ++w) {
            const int c = wc[w][threadIdx.x];
            wc[w][threadIdx.x] = first;
            first += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        rank[it] += wc[wid][(k[it] >> shift) & (digits - 1)];
        if (wbase + it * kWave + lane < n) buf[rank[it]] = k[it];
    }
    __syncthreads();
    int out[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const int i = it * kSortThreads + threadIdx.x;
        if (i < total) {
            const uint32_t x = buf[i];
            out[it] = i + to_global[(x >> shift) & (digits - 1)];
            key_out[out[it]] = x;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSortItems; ++it)
        if (wbase + it * kWave + lane < n) buf[rank[it]] = v[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const int i = it * kSortThreads + threadIdx.x;
        if (i < total) val_out[out[it]] = buf[i];
    }
}

}  // namespace

size_t sort_workspace_bytes(int64_t n) {
    int64_t nb = (n + kSortTile - 1) / kSortTile;
    int64_t h = (int64_t)kMaxDigits * nb;
    return (size_t)(2 * ((h + 1 + 15) / 16 * 16)) * sizeof(int32_t) + scan_workspace_bytes(h) + 256;
}

void stable_sort_pairs(uint32_t*& key, uint32_t*& val, uint32_t*& key_tmp, uint32_t*& val_tmp, int64_t n, int bits,
                       bool index_values, void* ws, hipStream_t s) {
    const int64_t nb = (n + kSortTile - 1) / kSortTile;
    int32_t* hist = static_cast<int32_t*>(ws);
    const int64_t room = ((int64_t)kMaxDigits * nb + 1 + 15) / 16 * 16;
    int32_t* hscan = hist + room;
    void* scan_ws = hscan + room;
    if (bits < 1) bits = 1;
    const int passes = (bits + kMaxBits - 1) / kMaxBits;
    for (int p = 0, shift = 0; p < passes; ++p) {
        const int b = (bits - shift + passes - p - 1) / (passes - p);
        const int digits = 1 << b;
        hipLaunchKernelGGL(k_digit_hist, dim3((unsigned)nb), dim3(kSortThreads), 0, s, key, n, shift, digits, nb, hist);
        exclusive_scan_i32(hist, hscan, (int64_t)digits * nb, scan_ws, s);
        if (p == 0 && index_values)
            hipLaunchKernelGGL(k_digit_scatter<true>, dim3((unsigned)nb), dim3(kSortThreads), 0, s, key, val, n,
                               shift, b, nb, hscan, key_tmp, val_tmp);
        else
            hipLaunchKernelGGL(k_digit_scatter<false>, dim3((unsigned)nb), dim3(kSortThreads), 0, s, key, val, n,
                               shift, b, nb, hscan, key_tmp, val_tmp);
        std::swap(key, key_tmp);
        std::swap(val, val_tmp);
        shift += b;
    }
}

}  // namespace cube
