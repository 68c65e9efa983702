// Exclusive prefix sum of int32 cell counts -> cell offsets (Sec. III-A: a
// per-cell count locates each cell's particles in the cell-ordered arrays).
//
// Passes over tiles of 4096 values: per-tile totals, then a tile-local scan
// plus the tile's base.  Up to kDirectTiles tiles every workgroup adds up the
// totals before its own, above that the totals are scanned first (recursively).
// Each thread owns 16 consecutive values so the loads are 64-byte vectors.
// The scan of a step's new counts also takes their maxima and decides how the
// step goes on, which were launches of their own (4 to 5 us each on a small box).
#include <algorithm>

#include "common.h"

namespace cube {

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int64_t kDirectTiles = 4096;      // 16 KB of totals read per workgroup at most
// workgroups up to which the last of them to finish does a step's scalar work;
// above, a launch costs less than the workgroups' atomics on one address (12 ns each)
constexpr int64_t kTicketBlocks = 256;

__device__ __forceinline__ bool gated(const int32_t* gate) { return gate && *(volatile const int32_t*)gate; }

__global__ __launch_bounds__(kScanThreads) void k_tile_sums(const int32_t* __restrict__ in,
                                                             int64_t n, int32_t* __restrict__ sums,
                                                             const int32_t* gate) {
    if (gated(gate)) return;
    __shared__ int lds[kScanThreads / kWave + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int acc = 0;
    if (base + kScanItems <= n) {
        const int4* p = reinterpret_cast<const int4*>(in + base);
#pragma unroll
        for (int i = 0; i < kScanItems / 4; ++i) {
            int4 q = p[i];
            acc += q.x + q.y + q.z + q.w;
        }
    } else {
        for (int i = 0; i < kScanItems; ++i)
            if (base + i < n) acc += in[base + i];
    }
    int total;
    block_exclusive_scan(acc, lds, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Totals, largest count and largest 2 x 2 x 2 block count (periodic) of tiles of
// kScanTile cells in storage order, where the +x, +y, +z neighbours are 1, Tc
// and Tc^2 entries ahead but at a tile's faces.  Memory-bound (the neighbours
// of a workgroup's cells are in its cache); the cell's coordinates advance by
// carries, since dividing for each cell made the pass 0.9 ms at 512^3 cells
// against 0.3.  1024 threads per tile: a small box has few tiles, each a chain
// of loads.
constexpr int kStatThreads = 1024;

__global__ __launch_bounds__(kStatThreads) void k_cell_stats(Geom g, const int32_t* __restrict__ counts,
                                                              int32_t* __restrict__ sums, int32_t* __restrict__ max_out,
                                                              int32_t* __restrict__ block8_out, const int32_t* gate) {
    if (gated(gate)) return;
    __shared__ int red[3][kStatThreads / kWave];
    const int Tc = g.Tc, nt = g.nt, tc2 = Tc * Tc, tc3 = tc2 * Tc;
    const int n = (int)g.ncells;
    int i = (int)blockIdx.x * kScanTile + (int)threadIdx.x;
    int sum = 0, mx = 0, mb = 0;
    if (i < n) {
        int t = i / tc3;
        const int local = i - t * tc3;
        int lz = local / tc2, ly = local / Tc - lz * Tc, lx = local % Tc;
        int tz = t / (nt * nt), ty = t / nt - tz * nt, tx = t % nt;
        const int sx = kStatThreads % Tc, sy = kStatThreads / Tc % Tc, sz = kStatThreads / tc2;
#pragma unroll
        for (int it = 0; it < kScanTile / kStatThreads && i < n; ++it, i += kStatThreads) {
            const int dx = lx + 1 < Tc ? 1 : (tx + 1 < nt ? tc3 : (1 - nt) * tc3) - (Tc - 1);
            const int dy = ly + 1 < Tc ? Tc : (ty + 1 < nt ? nt * tc3 : (1 - nt) * nt * tc3) - (tc2 - Tc);
            const int dz = lz + 1 < Tc ? tc2 : (tz + 1 < nt ? nt * nt * tc3 : (1 - nt) * nt * nt * tc3) - (tc3 - tc2);
            const int c = counts[i];
            const int block = c + counts[i + dx] + counts[i + dy] + counts[i + dx + dy] + counts[i + dz] +
                              counts[i + dx + dz] + counts[i + dy + dz] + counts[i + dx + dy + dz];
            sum += c;
            mx = max(mx, c);
            mb = max(mb, block);
            lx += sx;
            ly += sy;
            lz += sz;
            if (lx >= Tc) {
                lx -= Tc;
                ++ly;
            }
            if (ly >= Tc) {
                ly -= Tc;
                ++lz;
            }
            while (lz >= Tc) {
                lz -= Tc;
                if (++tx == nt) {
                    tx = 0;
                    if (++ty == nt) {
                        ty = 0;
                        ++tz;
                    }
                }
            }
        }
    }
    sum = wave_sum(sum);
    mx = wave_max(mx);
    mb = wave_max(mb);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[0][threadIdx.x / kWave] = sum;
        red[1][threadIdx.x / kWave] = mx;
        red[2][threadIdx.x / kWave] = mb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kStatThreads / kWave; ++w) {
            sum += red[0][w];
            mx = max(mx, red[1][w]);
            mb = max(mb, red[2][w]);
        }
        if (sums) sums[blockIdx.x] = sum;
        // one address for the whole grid: skip atomics the maximum already covers
        if (max_out && mx > *(volatile int32_t*)max_out) atomicMax(max_out, mx);
        if (mb > *(volatile int32_t*)block8_out) atomicMax(block8_out, mb);
    }
}

// How the step goes on, from its own data (see StepScalars::halt).
__device__ __forceinline__ void decide(StepScalars* sc) {
    if (sc->overflow) sc->halt = 2;
    else if (sc->far_count > 0) sc->halt = 1;
}

__global__ void k_decide(StepScalars* sc) {
    if (threadIdx.x == 0 && !gated(&sc->halt)) decide(sc);
}

// DIRECT: `base` holds the tiles' totals, else their scan.  sc (optional): the
// last workgroup to finish decides the step; every workgroup has then read
// the gate that the decision closes.
template <bool DIRECT>
__global__ __launch_bounds__(kScanThreads) void k_tile_scan(const int32_t* __restrict__ in, int64_t n,
                                                             const int32_t* __restrict__ base,
                                                             int32_t* __restrict__ out, const int32_t* gate,
                                                             StepScalars* sc) {
    if (gated(gate)) return;
    __shared__ int lds[kScanThreads / kWave + 1];
    const int64_t first = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int v[kScanItems];
    const bool full = first + kScanItems <= n;
    if (full) {
        const int4* p = reinterpret_cast<const int4*>(in + first);
#pragma unroll
        for (int i = 0; i < kScanItems / 4; ++i) {
            int4 q = p[i];
            v[4 * i] = q.x; v[4 * i + 1] = q.y; v[4 * i + 2] = q.z; v[4 * i + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) v[i] = (first + i < n) ? in[first + i] : 0;
    }
    int before = 0;
    if (DIRECT) {
        int part = 0;
        for (int b = threadIdx.x; b < (int)blockIdx.x; b += kScanThreads) part += base[b];
        block_exclusive_scan(part, lds, &before);
    } else {
        before = base[blockIdx.x];
    }
    int acc = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) acc += v[i];
    int total;
    int run = block_exclusive_scan(acc, lds, &total) + before;
    if (full) {
        int4* o = reinterpret_cast<int4*>(out + first);
#pragma unroll
        for (int i = 0; i < kScanItems / 4; ++i) {
            int4 q;
            q.x = run; run += v[4 * i];
            q.y = run; run += v[4 * i + 1];
            q.z = run; run += v[4 * i + 2];
            q.w = run; run += v[4 * i + 3];
            o[i] = q;
        }
    } else {
        for (int i = 0; i < kScanItems; ++i) {
            if (first + i < n) out[first + i] = run;
            run += v[i];
        }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = before + total;
    if (sc && threadIdx.x == 0 && atomicAdd(&sc->scan_ticket, 1) == (int)gridDim.x - 1) decide(sc);
}

inline int64_t round16(int64_t x) { return (x + 15) / 16 * 16; }

// out[0] += sum of in (64-bit), out[1] = min(out[1], smallest value): two
// atomics per workgroup
__global__ __launch_bounds__(kScanThreads) void k_count_check(const int32_t* __restrict__ in, int64_t n,
                                                               long long* __restrict__ out) {
    __shared__ long long s_sum[kScanThreads / kWave];
    __shared__ int s_min[kScanThreads / kWave];
    long long sum = 0;
    int mn = 0x7fffffff;
    for (int64_t i = (int64_t)blockIdx.x * kScanThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kScanThreads) {
        const int v = in[i];
        sum += v;
        mn = min(mn, v);
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        sum += __shfl_xor(sum, d, kWave);
        mn = min(mn, __shfl_xor(mn, d, kWave));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_sum[threadIdx.x / kWave] = sum;
        s_min[threadIdx.x / kWave] = mn;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kScanThreads / kWave; ++w) {
            sum += s_sum[w];
            mn = min(mn, s_min[w]);
        }
        atomicAdd(reinterpret_cast<unsigned long long*>(&out[0]), (unsigned long long)sum);
        atomicMin(&out[1], (long long)mn);
    }
}

}  // namespace

void launch_count_check(const int32_t* counts, int64_t n, long long* out, hipStream_t s) {
    const unsigned blocks = (unsigned)std::min<int64_t>(1024, std::max<int64_t>(1, (n + kScanTile - 1) / kScanTile));
    hipLaunchKernelGGL(k_count_check, dim3(blocks), dim3(kScanThreads), 0, s, counts, n, out);
}

size_t scan_workspace_bytes(int64_t n) {
    size_t bytes = 0;
    int64_t m = n;
    while (m > kScanTile) {
        const int64_t nb = (m + kScanTile - 1) / kScanTile;
        bytes += (size_t)(round16(nb) + round16(nb + 1)) * sizeof(int32_t);
        m = nb;
    }
    return bytes + 256;
}

namespace {

// out[0..n] from the totals of in's tiles in `sums` (nb of them; the
// workspace follows them)
void scan_tiles(const int32_t* in, int32_t* out, int64_t n, int32_t* sums, int64_t nb, hipStream_t s,
                const int32_t* gate, StepScalars* sc) {
    if (nb <= kDirectTiles) {
        hipLaunchKernelGGL(k_tile_scan<true>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, sums, out, gate, sc);
        return;
    }
    int32_t* sums_scan = sums + round16(nb);
    exclusive_scan_i32(sums, sums_scan, nb, sums_scan + round16(nb + 1), s, gate);
    hipLaunchKernelGGL(k_tile_scan<false>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, sums_scan, out, gate,
                       sc);
}

}  // namespace

// keep every array 64-byte aligned: the tile kernels use 16-byte vectors
void exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, void* ws, hipStream_t s, const int32_t* gate) {
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    int32_t* sums = static_cast<int32_t*>(ws);
    if (nb > 1)
        hipLaunchKernelGGL(k_tile_sums, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, sums, gate);
    scan_tiles(in, out, n, sums, nb, s, gate, nullptr);
}

void launch_cell_stats(const Geom& g, const int32_t* counts, int32_t* block8, hipStream_t s) {
    hipLaunchKernelGGL(k_cell_stats, dim3(grid1d(g.ncells, kScanTile)), dim3(kStatThreads), 0, s, g, counts, nullptr,
                       nullptr, block8, nullptr);
}

void launch_cell_offsets(const Geom& g, const int32_t* counts, int32_t* offsets, void* ws, int32_t* max_count,
                         int32_t* block8, hipStream_t s) {
    int32_t* sums = static_cast<int32_t*>(ws);
    const int64_t nb = (g.ncells + kScanTile - 1) / kScanTile;
    hipLaunchKernelGGL(k_cell_stats, dim3((unsigned)nb), dim3(kStatThreads), 0, s, g, counts, sums, max_count, block8,
                       nullptr);
    scan_tiles(counts, offsets, g.ncells, sums, nb, s, nullptr, nullptr);
}

void launch_step_scan(const Geom& g, const int32_t* counts_new, int32_t* offsets_new, void* ws, StepScalars* sc,
                      hipStream_t s) {
    int32_t* sums = static_cast<int32_t*>(ws);
    const int64_t nb = (g.ncells + kScanTile - 1) / kScanTile;
    hipLaunchKernelGGL(k_cell_stats, dim3((unsigned)nb), dim3(kStatThreads), 0, s, g, counts_new, sums,
                       &sc->new_max_count, &sc->new_max_block8, &sc->halt);
    const bool fused = nb <= kTicketBlocks;
    scan_tiles(counts_new, offsets_new, g.ncells, sums, nb, s, &sc->halt, fused ? sc : nullptr);
    if (!fused) hipLaunchKernelGGL(k_decide, dim3(1), dim3(64), 0, s, sc);
}

}  // namespace cube
