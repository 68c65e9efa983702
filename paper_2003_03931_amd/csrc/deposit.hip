// Cloud-in-cell mass assignment (Sec. II: density by interpolating particles
// onto a mesh; the tile's fine mesh is the tile plus its buffer) on the
// fixed-point positions of Eq. (2).
//
// Owner-computes: every workgroup owns a cube of target cells, pulls the
// particles of the coarse cells that can reach it (its own plus one coarse
// cell on each face) straight from the cell-ordered arrays, accumulates the
// exact CIC weights in LDS as 64-bit integers and writes each target cell
// once -- no global atomics, bit-reproducible.
//
// Exactness: a coordinate in target-cell units is P / D with P = 2(c 256 + m)+1
// and D = 512 / (target cells per coarse cell), so every CIC weight is an
// integer multiple of 1/D per axis and of 1/D^3 in 3-D.  The FP32 output is
// round(acc / D^3 / cell_volume - 1), the single rounding of the exact value.
// A target cell gathers particles of at most one 2 x 2 x 2 block of coarse
// cells, each weight at most D^3, so 32-bit accumulators are exact whenever
// D^3 times the largest such block count is below 2^32 (the caller checks the
// state's block counts); otherwise 64-bit.
//
// The brick kernel serves the periodic single-tile mesh and the diagnostic
// mesh; tile meshes of a tiled box use the z-marching form further down.
#include <algorithm>

#include "common.h"

namespace cube {

namespace {

constexpr int kDepThreads = 256;

// A periodic mesh of M^3 cells, cpc of them per coarse cell: the fine mesh of a
// single periodic tile (real values) or, DIAG, the diagnostic mesh (complex).
// MAXSRC bounds the source window, (BW / cpc + 2)^3 coarse cells; MAPCAP is
// the number of window particles whose source cell is looked up from a
// per-particle map (larger windows fall back to a binary search).
// full > 0: large bricks (kDiagBrick cells a side) whose window holds more
// than `full` particles only mark the small bricks (kDiagPart) in them, in the
// imaginary part of each one's first cell; small bricks, in a launch that
// follows, return where they find no mark.
constexpr int kDiagBrick = 16, kDiagPart = 8;

template <int BW, bool DIAG, class ACC, int MAXSRC, int MAPCAP>
__global__ __launch_bounds__(kDepThreads) void k_deposit(Geom g, const int32_t* __restrict__ offsets, Planes p,
                                                          float* __restrict__ out, int M, int cpc, int log2D,
                                                          double scale, int full) {
    static_assert(MAXSRC <= 1024, "fixed-step search over the source window");
    __shared__ __align__(16) ACC acc[BW * BW * BW];
    __shared__ int s_start[MAXSRC];
    __shared__ int s_pref[MAXSRC + 1];
    __shared__ int s_rel[MAXSRC];                // window coordinates + 1, 8 bits each
    __shared__ uint16_t s_map[MAPCAP];
    __shared__ int s_scan[kDepThreads / kWave + 1];

    const int nbx = (M + BW - 1) / BW;
    const int b = (int)xcd_logical_block();
    const int T0[3] = {(b % nbx) * BW, ((b / nbx) % nbx) * BW, (b / (nbx * nbx)) * BW};
    const int bw[3] = {min(BW, M - T0[0]), min(BW, M - T0[1]), min(BW, M - T0[2])};
    int nsa[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) nsa[k] = (bw[k] + cpc - 1) / cpc + 2;
    const int nsrc = nsa[0] * nsa[1] * nsa[2];
    // source frame origin (coarse cells): one cell before the block
    const int S0[3] = {T0[0] / cpc - 1, T0[1] / cpc - 1, T0[2] / cpc - 1};

    auto cell_at = [&](int x, int y, int z) { return (int64_t)x + (int64_t)M * (y + (int64_t)M * z); };
    if (DIAG && BW == kDiagPart && full > 0 && out[2 * cell_at(T0[0], T0[1], T0[2]) + 1] == 0.0f) return;

    static_assert(sizeof(acc) % sizeof(uint4) == 0, "accumulators are cleared 16 bytes at a time");
    for (int i = threadIdx.x; i < (int)(sizeof(acc) / sizeof(uint4)); i += kDepThreads)
        reinterpret_cast<uint4*>(acc)[i] = make_uint4(0u, 0u, 0u, 0u);

    // per-thread run of up to kPer source cells: counts, then a block scan
    constexpr int kPer = (MAXSRC + kDepThreads - 1) / kDepThreads;
    int my_cnt[kPer];
    int run = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int s = threadIdx.x * kPer + q;
        int cnt = 0;
        if (s < nsrc) {
            const int rx = s % nsa[0], ry = (s / nsa[0]) % nsa[1], rz = s / (nsa[0] * nsa[1]);
            s_rel[s] = rx | (ry << 8) | (rz << 16);
            const int64_t c = canon(g, wrapi(S0[0] + rx, g.Nc), wrapi(S0[1] + ry, g.Nc), wrapi(S0[2] + rz, g.Nc));
            const int st = offsets[c];
            cnt = offsets[c + 1] - st;
            s_start[s] = st;
        }
        my_cnt[q] = cnt;
        run += cnt;
    }
    int total;
    int base = block_exclusive_scan(run, s_scan, &total);
    if (DIAG && BW == kDiagBrick && full > 0 && total > full) {
        constexpr int K = kDiagBrick / kDiagPart;
        const int t = threadIdx.x;
        const int x = T0[0] + t % K * kDiagPart, y = T0[1] + t / K % K * kDiagPart, z = T0[2] + t / (K * K) * kDiagPart;
        if (t < K * K * K && x < M && y < M && z < M) out[2 * cell_at(x, y, z) + 1] = 1.0f;
        return;
    }
    const bool mapped = total <= MAPCAP;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int s = threadIdx.x * kPer + q;
        if (s < nsrc) {
            s_pref[s] = base;
            if (mapped)
                for (int j = 0; j < my_cnt[q]; ++j) s_map[base + j] = (uint16_t)s;
        }
        base += my_cnt[q];
    }
    if (threadIdx.x == 0) s_pref[nsrc] = total;
    __syncthreads();

    const int D = 1 << log2D;
    const int halfD = D >> 1;
    constexpr int U = 8;                       // particles per thread with loads in flight
    for (int base = 0; base < total; base += kDepThreads * U) {
        int mm[U][3], src_of[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = base + u * kDepThreads + threadIdx.x;
            src_of[u] = -1;
            if (e < total) {
                const int s = mapped ? (int)s_map[e] : find_cell_fixed<(MAXSRC <= 256 ? 8 : 10)>(s_pref, nsrc, e);
                const int pidx = s_start[s] + (e - s_pref[s]);
                src_of[u] = s;
#pragma unroll
                for (int k = 0; k < 3; ++k) mm[u][k] = p.m[k][pidx];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = src_of[u];
            if (s < 0) continue;
            const int rl = s_rel[s];
            const int rel[3] = {(rl & 255) - 1, ((rl >> 8) & 255) - 1, (rl >> 16) - 1};
            int i0[3];
            unsigned w1[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int P = 2 * (rel[k] * 256 + mm[u][k]) + 1;   // units of 1/D target cells
                const int Pm = P - halfD;
                i0[k] = Pm >> log2D;                                // floor division
                w1[k] = (unsigned)(Pm & (D - 1));
            }
#pragma unroll
            for (int oz = 0; oz < 2; ++oz) {
                const int iz = i0[2] + oz;
                if (iz < 0 || iz >= bw[2]) continue;
                const unsigned wz = oz ? w1[2] : (unsigned)D - w1[2];
#pragma unroll
                for (int oy = 0; oy < 2; ++oy) {
                    const int iy = i0[1] + oy;
                    if (iy < 0 || iy >= bw[1]) continue;
                    // weights are at most D <= 512 per axis: 24-bit products
                    const unsigned wyz = (unsigned)__umul24(oy ? w1[1] : (unsigned)D - w1[1], wz);
#pragma unroll
                    for (int ox = 0; ox < 2; ++ox) {
                        const int ix = i0[0] + ox;
                        if (ix < 0 || ix >= bw[0]) continue;
                        const ACC w = (ACC)(unsigned)__umul24(ox ? w1[0] : (unsigned)D - w1[0], wyz);
                        if (w) atomicAdd(&acc[(iz * BW + iy) * BW + ix], w);
                    }
                }
            }
        }
    }
    __syncthreads();

    // exact value * scale - 1, rounded once to FP32
    if (!DIAG) {
        // four x-consecutive cells per float4 store (the block origin and the
        // mesh side are multiples of 4, and so is bw[0])
        constexpr int Q = BW / 4;
        for (int i4 = threadIdx.x; i4 < Q * BW * BW; i4 += kDepThreads) {
            const int ix = 4 * (i4 % Q), iy = (i4 / Q) % BW, iz = i4 / (Q * BW);
            if (ix >= bw[0] || iy >= bw[1] || iz >= bw[2]) continue;
            const ACC* a = &acc[(iz * BW + iy) * BW + ix];
            float4 v;
            v.x = (float)fma((double)a[0], scale, -1.0);
            v.y = (float)fma((double)a[1], scale, -1.0);
            v.z = (float)fma((double)a[2], scale, -1.0);
            v.w = (float)fma((double)a[3], scale, -1.0);
            *reinterpret_cast<float4*>(out + cell_at(T0[0] + ix, T0[1] + iy, T0[2] + iz)) = v;
        }
        return;
    }
    for (int i = threadIdx.x; i < BW * BW * BW; i += kDepThreads) {
        const int ix = i % BW, iy = (i / BW) % BW, iz = i / (BW * BW);
        if (ix >= bw[0] || iy >= bw[1] || iz >= bw[2]) continue;
        const float v = (float)((double)acc[i] * scale - 1.0);
        const int64_t cell = cell_at(T0[0] + ix, T0[1] + iy, T0[2] + iz);
        out[2 * cell] = v;
        out[2 * cell + 1] = 0.0f;
    }
}

// The fine deposit of a batch of tile meshes, marching along z: a workgroup
// owns a BW x BW column of fine cells through the whole tile mesh and walks
// it in chunks of CZ fine planes (CZ / cpc coarse layers).  A chunk pulls the
// particles of its own coarse layers only (with one coarse cell on each side
// in x and y): its particles reach at most one plane below the chunk and one
// past it, so the accumulator is a ring of CZ + 2 planes, of which a chunk
// finishes CZ.  Per owned cell a chunk reads (BW / cpc + 2)^2 / (BW / cpc)^2
// of the particles (1.56x for 32 x 32 columns at cpc = 4) against the brick's
// (BW / cpc + 2)^3 / (BW / cpc)^3 (3.4x for 16^3 bricks).  The weights, the
// exactness and the single FP32 rounding are those of the brick kernel above.
//
// The stores (1.05 GB per 64 tiles of 160^3) take as long as the particles,
// the LDS atomics next to nothing; in two phases, particles then stores, the
// times add up (228 us without any particle, 228 for the particles, 456
// together).  So a chunk is one phase and one barrier, in which a thread
//   loads U consecutive particles, their cells found by a map of every U-th
//   particle and the following cells' bounds;
//   takes its cells of the planes that the previous chunk finished and clears
//   them for the ring's next turn;
//   waits for the loads (they and the stores share one in-order counter), then
//   stores the planes;
//   adds the particles, eight corners each without bounds checks: rows and
//   planes have spare cells between them for the corners that fall off the
//   column (a particle none of whose corners is in it is skipped).
// The ring holds the CZ planes being written and the CZ + 2 being added to.
// With eight planes a layer (cpc = 8) that would leave one workgroup per CU:
// there (TWO) a second phase takes and stores the planes just finished, from a
// ring of CZ + 2, and issues the next chunk's loads before (500 us as one
// phase of 1024 threads, 456 to 463 as two of 512; chunks of two phases in
// whole columns took 464 to 475).
// Source tables are built two chunks ahead: ranges loaded and counts scanned
// within the waves in one phase, ranks finished in the next.
//
// A column may be cut in z: part i of `parts` finishes the planes of its own
// chunks and starts one chunk early, whose particles reach its first planes.
// The launch cuts where workgroups would leave the chip's last round empty
// (column_parts).  64 tiles of a 1024^3 step: 471 us in two phases and whole
// columns, 415 now (1.27 GB moved, 3.1 TB/s); 8 tiles 111 -> 59.
template <int BW, int CZ, int NT, int U, bool TWO, class ACC, int MAXSRC, int MAPCAP>
__global__ __launch_bounds__(NT) void k_deposit_zm(Geom g, const int32_t* __restrict__ offsets, Planes p,
                                                    float* __restrict__ out, int cpc, int log2D, double scale,
                                                    int tile0, int parts) {
    static_assert(MAXSRC <= NT && MAXSRC <= 256, "a source cell per thread, cells in a byte");
    static_assert(BW % 4 == 0 && NT % (BW * BW / 4) == 0, "float4 rows, whole planes per pass");
    // planes z0 - 1 .. z0 + CZ of the chunk at z0, and the CZ before them
    constexpr int NP = (TWO ? 1 : 2) * CZ + 2;
    constexpr int RS = BW + 4, PS = (BW + 1) * RS;   // row and plane strides: spare cells at x = -1, BW and y = -1, BW
    constexpr int OFF = RS + 4;                  // cell (0, 0) of the first plane
    __shared__ __align__(16) ACC acc[OFF + NP * PS];
    // the source cells that hold particles, two chunks' tables
    __shared__ int s_pref[2][MAXSRC + U];        // rank of the cell's first particle
    __shared__ int2 s_cell[2][MAXSRC];           // first particle minus its rank; coordinates: x, y from the column's ring, z in the chunk
    __shared__ uint8_t s_map[2][MAPCAP / U];     // cell of every U-th particle
    constexpr int SWAVES = (MAXSRC + kWave - 1) / kWave;
    __shared__ int2 s_wave[2][SWAVES];           // a wave's particles and filled cells

    const int M = g.F;
    const int nbx = (M + BW - 1) / BW;
    const int64_t lb = xcd_logical_block();
    const int b = (int)(lb % gridDim.x) / parts, part = (int)(lb % gridDim.x) % parts;   // column, its part
    const int ky = (int)(lb / gridDim.x);       // tile within the batch
    const int T0x = (b % nbx) * BW, T0y = (b / nbx) * BW;
    const int bwx = min(BW, M - T0x), bwy = min(BW, M - T0y);
    const int nsx = (bwx + cpc - 1) / cpc + 2, nsy = (bwy + cpc - 1) / cpc + 2;
    const int LC = CZ / cpc;                     // coarse layers per chunk (a whole number of chunks per mesh)
    const int nch = g.Fc / LC, nsrc = nsx * nsy * LC;
    const int j0 = nch * part / parts, j1 = nch * (part + 1) / parts;   // this part's chunks
    const int tile = tile0 + ky;
    const int tx = tile % g.nt, ty = (tile / g.nt) % g.nt, tz = tile / (g.nt * g.nt);
    float* mesh = out + (int64_t)ky * M * M * M;

    static_assert(sizeof(acc) % sizeof(uint4) == 0, "accumulators are cleared 16 bytes at a time");
    for (int i = threadIdx.x; i < (int)(sizeof(acc) / sizeof(uint4)); i += NT)
        reinterpret_cast<uint4*>(acc)[i] = make_uint4(0u, 0u, 0u, 0u);

    // this thread's source cell in every chunk: its column is fixed
    const int t = threadIdx.x, sx = t % nsx, sy = t / nsx % nsy, sz = t / (nsx * nsy);
    const int fx = T0x / cpc - 1 + sx, fy = T0y / cpc - 1 + sy;
    const bool source = t < nsrc && fx >= 0 && fx < g.Fc && fy >= 0 && fy < g.Fc;
    const int gx = wrapi(fx + tx * g.Tc - g.hc, g.Nc), gy = wrapi(fy + ty * g.Tc - g.hc, g.Nc);
    const int gz0 = wrapi(sz + tz * g.Tc - g.hc, g.Nc);
    int my_st = 0, my_cnt = 0;
    auto fetch = [&](int j) {                    // particle range of chunk j's source cell
        my_st = my_cnt = 0;
        if (source && j >= 0 && j < j1) {
            int cz = gz0 + j * LC;               // below 2 Nc: the tile box is no larger than the mesh
            cz = cz >= g.Nc ? cz - g.Nc : cz;
            const int64_t c = canon(g, gx, gy, cz);
            my_st = offsets[c];
            my_cnt = offsets[c + 1] - my_st;
        }
    };
    // the chunk's table: counts scanned within the waves, then (after a
    // barrier) the cells' first ranks; empty cells are left out
    int tab_st = 0, tab_cnt = 0, tab_incl = 0, tab_slot = 0, my_total = 0, my_cells = 0;
    auto table_begin = [&](int buf) {
        tab_st = my_st;
        tab_cnt = my_cnt;
        if (t >= SWAVES * kWave) return;
        tab_incl = wave_inclusive_scan(tab_cnt);
        const uint64_t filled = __ballot(tab_cnt > 0);
        tab_slot = __popcll(filled & ((1ull << (t & (kWave - 1))) - 1ull));
        if ((t & (kWave - 1)) == kWave - 1) s_wave[buf][t / kWave] = make_int2(tab_incl, __popcll(filled));
    };
    auto table_end = [&](int buf) {
        int before = 0, slot = tab_slot, cells = 0;
        my_total = 0;
#pragma unroll
        for (int w = 0; w < SWAVES; ++w) {
            const int2 v = s_wave[buf][w];
            before += w < t / kWave ? v.x : 0;
            slot += w < t / kWave ? v.y : 0;
            my_total += v.x;
            cells += v.y;
        }
        const int first = before + tab_incl - tab_cnt;
        if (tab_cnt > 0) {
            s_pref[buf][slot] = first;
            s_cell[buf][slot] = make_int2(tab_st - first, sx | (sy << 8) | (sz << 16));
            if (my_total <= MAPCAP)
                for (int e = (first + U - 1) / U; U * e < first + tab_cnt; ++e) s_map[buf][e] = (uint8_t)slot;
        }
        if (t < U) s_pref[buf][cells + t] = my_total;
        my_cells = cells;
    };
    static_assert(MAXSRC <= NT, "a thread per source cell");
    // in-cell bytes and cells (-1: none) of particles e0 .. e0 + U - 1 of a chunk;
    // every lane loads, so that the wait counts stay exact
    auto load = [&](int buf, int total, int cells, int e0, uint32_t mm[U][3], int rel[U]) {
        const int* pref = s_pref[buf];
        // past the end: the last particle's cell, read and dropped
        const int end = max(total - 1, 0), es = min(e0, end);
        int c = total <= MAPCAP ? (int)s_map[buf][es / U] : find_cell_fixed<8>(pref, cells, es);
        c = min(c, max(cells - 1, 0));
        int bound[U - 1];                        // no cell is empty: U particles are in U cells at most
#pragma unroll
        for (int a = 0; a < U - 1; ++a) bound[a] = pref[c + 1 + a];
        int2 sc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = min(e0 + u, end);
            int k = c;
#pragma unroll
            for (int a = 0; a < U - 1; ++a) k += bound[a] <= e;
            sc[u] = s_cell[buf][k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = e0 + u < total;
            rel[u] = live ? sc[u].y : -1;
            const uint32_t q = live ? (uint32_t)(sc[u].x + e0 + u) : 0u;
#pragma unroll
            for (int k = 0; k < 3; ++k) mm[u][k] = p.m[k][q];
        }
    };

    const int D = 1 << log2D;
    const int halfD = D >> 1;
    const float scalef = (float)scale;           // a power of two
    int ring = 0;                                // accumulator plane of z0 - 1 of the chunk being added
    auto add = [&](const uint32_t m[U], const int rel[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (rel[u] < 0) continue;
            // coarse cell relative to the column's first cell in x and y and
            // to the chunk's first layer in z
            const int cell[3] = {(rel[u] & 255) - 1, ((rel[u] >> 8) & 255) - 1, rel[u] >> 16};
            int i0[3];
            unsigned w1[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int P = 2 * (cell[k] * 256 + (int)((m[u] >> (8 * k)) & 255u)) + 1;   // units of 1/D target cells
                const int Pm = P - halfD;
                i0[k] = Pm >> log2D;                                // floor division
                w1[k] = (unsigned)(Pm & (D - 1));
            }
            if ((unsigned)(i0[0] + 1) > (unsigned)BW || (unsigned)(i0[1] + 1) > (unsigned)BW) continue;
            // weights are at most D <= 128 per axis: 24-bit products
            const unsigned w0[3] = {(unsigned)D - w1[0], (unsigned)D - w1[1], (unsigned)D - w1[2]};
            // plane i0 of the chunk is ring plane i0 + 1 after its first
            int z = ring + i0[2] + 1;
            z = z >= NP ? z - NP : z;
            const int z1 = z + 1 == NP ? 0 : z + 1;
            ACC* at = acc + OFF + i0[1] * RS + i0[0];
#pragma unroll
            for (int oz = 0; oz < 2; ++oz) {
                ACC* pl = at + (oz ? z1 : z) * PS;
                const unsigned wz = oz ? w1[2] : w0[2];
                const unsigned wy0 = (unsigned)__umul24(w0[1], wz), wy1 = (unsigned)__umul24(w1[1], wz);
                atomicAdd(pl, (ACC)(unsigned)__umul24(w0[0], wy0));
                atomicAdd(pl + 1, (ACC)(unsigned)__umul24(w1[0], wy0));
                atomicAdd(pl + RS, (ACC)(unsigned)__umul24(w0[0], wy1));
                atomicAdd(pl + RS + 1, (ACC)(unsigned)__umul24(w1[0], wy1));
            }
        }
    };
    // waits for a batch's loads here: the bytes of a particle in one word
    auto arrived = [&](const uint32_t mm[U][3], uint32_t m[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            m[u] = mm[u][0] | (mm[u][1] << 8) | (mm[u][2] << 16);
            asm volatile("" : "+v"(m[u]));
        }
    };

    // this thread's four cells of a plane in the write-out
    constexpr int PT = BW * BW / 4, PER = NT / PT;   // threads per plane, planes per pass
    static_assert(CZ % PER == 0, "whole passes");
    const int wx = 4 * (t % (BW / 4)), wy = t / (BW / 4) % BW, wp = t / PT;
    const bool wlive = wx < bwx && wy < bwy;
    float* wdst = mesh + (T0x + wx) + (int64_t)M * (T0y + wy);
    struct alignas(16) Quad {
        ACC v[4];
    };
    // four cells of ring plane q (below 2 NP), cleared for the ring's next turn
    auto take = [&](int q) {
        q = q >= NP ? q - NP : q;
        Quad* a = reinterpret_cast<Quad*>(acc + OFF + q * PS + wy * RS + wx);
        const Quad s4 = *a;
        *a = Quad{{0, 0, 0, 0}};
        const ACC* v = s4.v;
        if (max(max(v[0], v[1]), max(v[2], v[3])) < (ACC)(1u << 24)) {
            // the sums and the power-of-two scale are exact in FP32, and
            // the fused multiply-add rounds once: the FP64 result
            return make_float4(fmaf((float)v[0], scalef, -1.0f), fmaf((float)v[1], scalef, -1.0f),
                               fmaf((float)v[2], scalef, -1.0f), fmaf((float)v[3], scalef, -1.0f));
        }
        return make_float4((float)fma((double)v[0], scale, -1.0), (float)fma((double)v[1], scale, -1.0),
                           (float)fma((double)v[2], scale, -1.0), (float)fma((double)v[3], scale, -1.0));
    };
    auto put = [&](int z, float4 v) {
        if (wlive && z >= 0 && z < M) *reinterpret_cast<float4*>(wdst + (int64_t)z * M * M) = v;
    };

    // planes finished by chunk c, from ring plane q on; `own`: they are this
    // part's (chunk j0 - 1 is another's, or none)
    uint32_t mm[U][3], m[U];
    int rel[U];
    auto flush = [&](int c, int q, bool own) {
        float4 v[CZ / PER];
#pragma unroll
        for (int i = 0; i < CZ / PER; ++i) v[i] = take(q + i * PER + wp);
        arrived(mm, m);
        asm volatile("" : "+v"(my_st), "+v"(my_cnt));
        if (own) {
#pragma unroll
            for (int i = 0; i < CZ / PER; ++i) put(c * CZ - 1 + i * PER + wp, v[i]);
        }
    };
    // phase j: particles of chunk j, table of chunk j + 1, ranges of chunk
    // j + 2, planes of chunk j - 1 (TWO: of chunk j); the first chunk is j0 - 1
    int total = 0, cells = 0;                    // of chunk j
    load(0, 0, 0, 0, mm, rel);
    arrived(mm, m);
    for (int j = j0 - 3; j <= j1; ++j) {
        const int buf = j & 1;
        if (TWO && j == j1) break;
        fetch(j + 2);
        if (!TWO) {
            load(buf, total, cells, U * t, mm, rel);
            if (j >= j0) flush(j - 1, ring + NP - CZ, j > j0);
            else arrived(mm, m);
            if (j == j1) break;
        }
        if (j >= j0 - 2) table_end(buf ^ 1);     // of chunk j + 1
        add(m, rel);
        for (int e0 = U * NT + U * t; e0 < total; e0 += U * NT) {
            load(buf, total, cells, e0, mm, rel);
            arrived(mm, m);
            add(m, rel);
        }
        table_begin(buf);                        // of chunk j + 2
        if (TWO) {
            lds_barrier();
            load(buf ^ 1, my_total, my_cells, U * t, mm, rel);
            if (j >= j0 - 1) flush(j, ring, j >= j0);
            else arrived(mm, m);
        }
        total = my_total;
        cells = my_cells;
        if (j >= j0 - 1) {
            ring += CZ;
            ring = ring >= NP ? ring - NP : ring;
        }
        lds_barrier();
    }
    // past the last chunk its upper plane is complete too (the one above lies
    // outside the mesh)
    if (j1 == nch && wp == 0) put(M - 1, take(ring));
}

// The value of the lane whose index differs in bit X (1 or 2), by DPP.
template <int X>
__device__ __forceinline__ unsigned quad_xor(unsigned v) {
    constexpr int kPerm = X == 1 ? 0xB1 : 0x4E;      // quad_perm [1,0,3,2] or [2,3,0,1]
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, kPerm, 0xf, 0xf, true);
}

// Coarse-mesh deposit (one mesh cell per storage cell): a workgroup owns a
// BW^3 cube of mesh cells and walks the (BW+2)^3 storage cells that can reach
// it, one cell per lane (L = 1) or per quad of lanes (L = 4) at a time.  Along each axis a particle at in-cell
// byte m weighs (in 1/512 of a cell) 255 - 2m and 2m + 257 on the cells at
// offsets -1 and 0 when m < 128, and 767 - 2m and 2m - 255 on offsets 0 and
// +1 otherwise.  The lane sums the 27 products over its cell's particles in
// 32-bit registers, four particles at a time (one 4-byte load per axis, the
// next four in flight meanwhile), and adds the sums to 64-bit LDS
// accumulators that are padded by the slots' reach: no bounds checks,
// constant offsets, one LDS atomic per cell and slot instead of eight per
// particle.  A product is at most 511^3, so 32 of them fit 32 bits; fuller
// cells are added every 32 particles.  A quad exchanges halves twice first,
// so that each lane holds the whole sums of a quarter of the slots.  Integer
// sums: the result does not depend on the order and equals the
// particle-by-particle deposit bit for bit.
//
// Bound by vector instructions: in the 1024^3 step 1.02 per clock and CU with
// 42 of 64 lanes at work (cells of eight particles on average go by fours, and
// a wave is as long as its longest lane), 146 lane slots for each particle and
// cube that reads it (1.42 of them).  Its 7.8 GB would take 1.3 ms.  A cell per
// thread with byte loads, bounds checks per slot and a wave waiting at every
// cell for its fullest one took 9.06 ms there, lanes stepping through their own
// cells take 5.7 to 6.1.
template <int BW, int NT, int L>
__global__ __launch_bounds__(NT) void k_coarse_deposit(Geom g, const int32_t* __restrict__ offsets, Planes p,
                                                        float2* __restrict__ out, double scale) {
    constexpr int SW = BW + 2, PW = BW + 4;
    constexpr int NS = SW * SW * SW;
    constexpr int U = 4, ROUND = 32 / (U * L);    // particles together, and such loads per exact 32-bit sum
    constexpr int CELLS = NT / L;                 // cells in work
    static_assert(L == 1 || L == 4, "one lane or a quad");
    __shared__ __align__(16) unsigned long long acc[PW * PW * PW];
    __shared__ int s_axis[3][SW];                 // canonical index of a cell: one term per axis
    const int M = g.Nc;
    const int nbx = (M + BW - 1) / BW;
    const int b = (int)xcd_logical_block();
    const int T0[3] = {(b % nbx) * BW, ((b / nbx) % nbx) * BW, (b / (nbx * nbx)) * BW};
    const int bw[3] = {min(BW, M - T0[0]), min(BW, M - T0[1]), min(BW, M - T0[2])};
    static_assert(PW * PW * PW % 2 == 0, "accumulators are cleared 16 bytes at a time");
    for (int i = threadIdx.x; i < PW * PW * PW / 2; i += NT)
        reinterpret_cast<uint4*>(acc)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < 3 * SW) {
        const int k = threadIdx.x / SW, r = threadIdx.x % SW;
        const int c = wrapi(T0[k] - 1 + r, M);
        s_axis[k][r] = (int)(k == 0 ? canon(g, c, 0, 0) : k == 1 ? canon(g, 0, c, 0) : canon(g, 0, 0, c));
    }
    __syncthreads();
    // particle range of window cell s = r (storage cell T0 - 1 + r; empty past
    // a partial cube's reach) and the padded cell of its first slot
    auto range = [&](int s, int& st, int& en, int& at) {
        const int row = s / SW, rz = s / (SW * SW), ry = row - rz * SW, rx = s - row * SW;
        st = en = 0;
        at = s + 2 * row + 2 * PW * rz;
        if (s < NS && rx <= bw[0] + 1 && ry <= bw[1] + 1 && rz <= bw[2] + 1) {
            const int c = s_axis[0][rx] + s_axis[1][ry] + s_axis[2][rz];
            st = offsets[c];
            en = offsets[c + 1];
        }
    };
    // the planes are followed by others, so a load may pass the last
    // particle by up to three bytes
    auto load = [&](int q, unsigned mm[3]) {
#pragma unroll
        for (int k = 0; k < 3; ++k) __builtin_memcpy(&mm[k], p.m[k] + q, U);
    };
    const int lane = L == 1 ? 0 : threadIdx.x % L;
    int s = threadIdx.x / L, q, en, at, q_n, en_n, at_n;
    range(s, q, en, at);
    range(s + CELLS, q_n, en_n, at_n);
    unsigned mm[3];
    load(min(q + U * lane, (int)g.n), mm);
    unsigned a[27];
#pragma unroll
    for (int k = 0; k < 27; ++k) a[k] = 0u;
    int left = ROUND;
    // every lane steps through its own cells: a wave is as long as the lane
    // with the most particles, not the sum of each step's fullest cells
    while (s < NS) {
        const int q0 = q, e0 = en, at0 = at;
        const bool done = q + U * L >= en;
        q += U * L;
        if (done) {
            s += CELLS;
            q = q_n;
            en = en_n;
            at = at_n;
            range(s + CELLS, q_n, en_n, at_n);
        }
        unsigned mn[3];
        load(min(q + U * lane, (int)g.n), mn);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            unsigned w[3][3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const unsigned m2 = 2u * ((mm[k] >> (8 * u)) & 255u);
                w[k][0] = __builtin_elementwise_sub_sat(255u, m2);
                w[k][2] = __builtin_elementwise_sub_sat(m2, 255u);
                w[k][1] = 512u - (w[k][0] | w[k][2]);     // one of them is zero
            }
            const bool live = q0 + U * lane + u < e0;
#pragma unroll
            for (int k = 0; k < 3; ++k) w[2][k] = live ? w[2][k] : 0u;
            unsigned wxy[9];
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int i = 0; i < 3; ++i) wxy[3 * j + i] = (unsigned)__umul24(w[0][i], w[1][j]);
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int j = 0; j < 9; ++j) a[9 * k + j] += (unsigned)__umul24(wxy[j], w[2][k]);
        }
        if (done || --left == 0) {
            if (q0 < e0) {
                // slot (i, j, k) is padded cell r + (i, j, k)
                auto add = [&](int off, unsigned v) { atomicAdd(&acc[at0 + off], (unsigned long long)v); };
                if constexpr (L == 1) {
#pragma unroll
                    for (int k = 0; k < 3; ++k)
#pragma unroll
                        for (int j = 0; j < 9; ++j) add((k * PW + j / 3) * PW + j % 3, a[9 * k + j]);
                } else {
                    // sum over the pair of lanes that differ in a bit: of x in
                    // the lane whose bit is clear, of y in the other
                    const bool b0 = lane & 1, b1 = lane & 2;
                    auto half0 = [&](unsigned x, unsigned y) { return (b0 ? y : x) + quad_xor<1>(b0 ? x : y); };
                    auto half1 = [&](unsigned x, unsigned y) { return (b1 ? y : x) + quad_xor<2>(b1 ? x : y); };
                    unsigned h[14];           // slots 2t and 2t + 1 (the 28th is nothing)
#pragma unroll
                    for (int t = 0; t < 14; ++t) h[t] = half0(a[2 * t], 2 * t + 1 < 27 ? a[2 * t + 1] : 0u);
#pragma unroll
                    for (int t = 0; t < 7; ++t) {
                        // slots 4t .. 4t + 3 on lanes 0 .. 3
                        const unsigned v = half1(h[2 * t], h[2 * t + 1]);
                        int off[4];
#pragma unroll
                        for (int l = 0; l < 4; ++l) {
                            const int m = 4 * t + l;
                            off[l] = ((m / 9) * PW + m / 3 % 3) * PW + m % 3;
                        }
                        if (t < 6 || lane < 3) add(b1 ? (b0 ? off[3] : off[2]) : (b0 ? off[1] : off[0]), v);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 27; ++k) a[k] = 0u;
            left = ROUND;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) mm[k] = mn[k];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < BW * BW * BW; i += NT) {
        const int ix = i % BW, iy = (i / BW) % BW, iz = i / (BW * BW);
        if (ix >= bw[0] || iy >= bw[1] || iz >= bw[2]) continue;
        const float v = (float)((double)acc[((iz + 2) * PW + iy + 2) * PW + ix + 2] * scale - 1.0);
        out[(int64_t)(T0[0] + ix) + (int64_t)M * ((T0[1] + iy) + (int64_t)M * (T0[2] + iz))] = make_float2(v, 0.0f);
    }
}

int ilog2(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

}  // namespace

template <int BW, int NT, int L>
void coarse_deposit_cubes(const Geom& g, const int32_t* offsets, Planes p, float2* mesh, double scale,
                          hipStream_t s) {
    const int nb = (g.Nc + BW - 1) / BW;
    hipLaunchKernelGGL((k_coarse_deposit<BW, NT, L>), dim3(nb * nb * nb), dim3(NT), 0, s, g, offsets, p, mesh, scale);
}

void launch_coarse_deposit(const Geom& g, const int32_t* offsets, Planes p, float2* mesh, hipStream_t s) {
    // acc in units of 2^-27 particle; density = mass / H^3 with H = r / f
    const double scale = std::ldexp(1.0, -27) * ((double)g.f * g.f * g.f) / ((double)g.r * g.r * g.r);
    // Cubes of 16 cells re-read least (1.42x), but a small mesh has too few of
    // them to fill the chip: at 64 cells a side 70 us against 35 with cubes of
    // 8 (8 particles per cell), at 32 a side 60 against 13 with cubes of 4.
    // Quads pay where a cell is a long walk (64 particles per cell: 590
    // against 1592 us at 128 a side, a lane per cell also thrashing its cache
    // lines) and cost nothing on small meshes; with 8 particles per cell on a
    // large mesh most of a quad would idle (1.37 against 0.80 ms at 256).
    if (g.Nc >= 128) {
        if (g.r >= 4 * g.f) coarse_deposit_cubes<16, 512, 4>(g, offsets, p, mesh, scale, s);
        else coarse_deposit_cubes<16, 512, 1>(g, offsets, p, mesh, scale, s);
    } else if (g.Nc >= 64) {
        coarse_deposit_cubes<8, 512, 4>(g, offsets, p, mesh, scale, s);
    } else {
        coarse_deposit_cubes<4, 256, 4>(g, offsets, p, mesh, scale, s);
    }
}

namespace {

// Parts that a column is cut in.  A part of n chunks takes about n + 2 phases
// (its first chunk is another part's last, and the pipeline fills); the chip
// holds `slots` workgroups at a time, and beyond one round of them the last
// one is on average little more than half full.  Timed alone, with columns of
// 40 chunks on 768 slots: 1600 columns (64 tiles of 160^3) 445, 404, 400, 406, 420 us in 1,
// 2, 3, 4, 6 parts; 200 columns 98, 65, 57, 66, 60; 25 columns 86 us in one
// part, 21 in 14.
int column_parts(int64_t columns, int chunks, int slots) {
    int best = 1;
    double least = 0.0;
    for (int s = 1; s <= chunks / 2 && s <= 16; ++s) {
        const double rounds = (double)(columns * s) / slots;
        const double cost = (rounds <= 1.0 ? 1.0 : rounds + 0.6) * ((double)chunks / s + 2.0);
        if (s == 1 || cost < least) {
            least = cost;
            best = s;
        }
    }
    return best;
}

template <int BW, int CZ, int U, class ACC, int MAXSRC>
void fine_deposit_columns(const Geom& g, const int32_t* offsets, Planes p, int tile0, int ntiles, float* mesh,
                          double scale, hipStream_t s) {
    constexpr int NT = 512, MAPCAP = 3072;
    constexpr bool TWO = CZ == 8;
    const int nb = (g.F + BW - 1) / BW, chunks = g.F / CZ;
    // workgroups per CU: ten planes of accumulators each, and the tables
    constexpr int lds = 10 * (BW + 1) * (BW + 4) * (int)sizeof(ACC) + 6 * 1024;
    const int slots = device_cus() * std::max(1, 160 * 1024 / lds);
    const int parts = column_parts((int64_t)nb * nb * ntiles, chunks, slots);
    hipLaunchKernelGGL((k_deposit_zm<BW, CZ, NT, U, TWO, ACC, MAXSRC, MAPCAP>), dim3(nb * nb * parts, ntiles),
                       dim3(NT), 0, s, g, offsets, p, mesh, g.r, g.log2D, scale, tile0, parts);
}

}  // namespace

void launch_fine_deposit(const Geom& g, const int32_t* offsets, Planes p, int tile0, int ntiles,
                         float* mesh, bool wide, hipStream_t s) {
    // every box has r = 4 or r = 8 (the gather's bricks need it)
    const int log2D = g.log2D;
    // acc in units of D^-3 fine-cell masses; density = mass / h^3 = mass * f^3
    const double scale = std::ldexp(1.0, -3 * log2D) * ((double)g.f * g.f * g.f);
    if (g.periodic) {
        // the single periodic tile: 16^3 bricks over (16 / r + 2)^3 <= 6^3 source cells
        const int nb = (g.F + 15) / 16;
        const dim3 grid(nb * nb * nb), block(kDepThreads);
        if (wide)
            hipLaunchKernelGGL((k_deposit<16, false, unsigned long long, 216, 2048>), grid, block, 0, s, g, offsets, p,
                               mesh, g.F, g.r, log2D, scale, 0);
        else
            hipLaunchKernelGGL((k_deposit<16, false, unsigned int, 216, 2048>), grid, block, 0, s, g, offsets, p, mesh,
                               g.F, g.r, log2D, scale, 0);
        return;
    }
    // tile meshes: z-marching columns of 32 x 32 cells, a coarse layer per chunk
    if (g.r == 4) {
        if (wide) fine_deposit_columns<32, 4, 2, unsigned long long, 100>(g, offsets, p, tile0, ntiles, mesh, scale, s);
        else fine_deposit_columns<32, 4, 2, unsigned int, 100>(g, offsets, p, tile0, ntiles, mesh, scale, s);
    } else {
        if (wide) fine_deposit_columns<32, 8, 4, unsigned long long, 36>(g, offsets, p, tile0, ntiles, mesh, scale, s);
        else fine_deposit_columns<32, 8, 4, unsigned int, 36>(g, offsets, p, tile0, ntiles, mesh, scale, s);
    }
}

bool fine_deposit_needs_wide(const Geom& g, int max_block8) {
    // a fine cell gathers the particles of at most one 2 x 2 x 2 block of
    // coarse cells, each weighing at most D^3 units: stay below 2^32
    return (double)max_block8 * std::ldexp(1.0, 3 * g.log2D) >= 4294967296.0;
}

bool fp16_density_fits(const Geom& g, int max_block8) {
    // a fine cell's density is at most f^3 times the particles of one 2 x 2 x 2
    // block of coarse cells; the plane transform's gain is divided out
    return (double)g.f * g.f * g.f * (double)max_block8 + 1.0 < 32768.0;
}

namespace {

template <int BW, class ACC, int MAXSRC, int MAPCAP>
void diag_bricks(const Geom& g, const int32_t* offsets, Planes p, float2* mesh, int full, hipStream_t s) {
    const int H = g.r / g.f;                       // diagnostic cells per coarse cell
    const int nb = (g.ns + BW - 1) / BW;
    const int log2D = ilog2(512 / H);
    hipLaunchKernelGGL((k_deposit<BW, true, ACC, MAXSRC, MAPCAP>), dim3(nb * nb * nb), dim3(kDepThreads), 0, s, g,
                       offsets, p, reinterpret_cast<float*>(mesh), g.ns, H, log2D, std::ldexp(1.0, -3 * log2D), full);
}

// Bricks of 16 cells re-read less than bricks of 8 (1.95x against 3.4x at
// H = 2, 3.4x against 8x at H = 4): 488 against 786 us for all of P(k) of 256^3
// particles at H = 4.  But a mesh below 128 has fewer of them than twice the
// CUs (64: 96 us against 65, 111 against 72 at H = 4), and where the particles
// are concentrated the bricks that hold them are few (256^3 in 1/64 of the
// volume: 3.8 ms against 2.9): a large brick whose window holds more than
// three times the average, and more than 0.6 of a CU's share of all windows
// (below that the others hide it), is left to small ones: 2.6 ms.  That second
// launch is skipped where no window can be that full.
template <class ACC, int SRC8, int MAP8, int SRC16, int MAP16>
void diag_deposit(const Geom& g, const int32_t* offsets, Planes p, float2* mesh, int max_block8, hipStream_t s) {
    const int H = g.r / g.f;
    const int64_t nb = (g.ns + kDiagBrick - 1) / kDiagBrick, cus = device_cus();
    if (nb * nb * nb < 2 * cus) {
        diag_bricks<kDiagPart, ACC, SRC8, MAP8>(g, offsets, p, mesh, 0, s);
        return;
    }
    const int64_t w = kDiagBrick / H + 2;          // window side; even, so blocks of 2 cells cover it
    const double window = (double)(w * w * w) * g.n / g.ncells;
    const double limit = std::max(3.0 * window, 0.6 * window * (double)(nb * nb * nb) / (double)cus);
    const bool even = (double)max_block8 * (double)(w / 2 * (w / 2) * (w / 2)) <= limit;
    const int full = even ? 0 : (int)std::min(limit, 2147483647.0);
    diag_bricks<kDiagBrick, ACC, SRC16, MAP16>(g, offsets, p, mesh, full, s);
    if (full) diag_bricks<kDiagPart, ACC, SRC8, MAP8>(g, offsets, p, mesh, full, s);
}

}  // namespace

void launch_diag_deposit(const Geom& g, const int32_t* offsets, Planes p, float2* mesh, int max_block8,
                         hipStream_t s) {
    const int H = g.r / g.f;
    if (H == 1) {
        diag_bricks<kDiagPart, unsigned long long, 1000, 10240>(g, offsets, p, mesh, 0, s);
        return;
    }
    // a cell is at most half a coarse cell wide and gathers the particles of
    // at most one 2 x 2 x 2 block of coarse cells, as on the fine mesh, so
    // 32-bit accumulators are exact below the same kind of bound; they take
    // half of the LDS (594 -> 278 us with bricks of 16 for 256^3 particles at
    // H = 4)
    const bool wide = (double)max_block8 * std::ldexp(1.0, 27) / ((double)H * H * H) >= 4294967296.0;
    if (H == 2) {
        if (wide) diag_deposit<unsigned long long, 216, 8192, 1000, 8192>(g, offsets, p, mesh, max_block8, s);
        else diag_deposit<unsigned int, 216, 8192, 1000, 8192>(g, offsets, p, mesh, max_block8, s);
    } else {
        if (wide) diag_deposit<unsigned long long, 64, 8192, 216, 4096>(g, offsets, p, mesh, max_block8, s);
        else diag_deposit<unsigned int, 64, 8192, 216, 4096>(g, offsets, p, mesh, max_block8, s);
    }
}

}  // namespace cube
