// Extended PP force (Sec. II, optional PP module; Sec. III-B, pair distances
// from the compressed integer positions).
//
// Every pair of particles closer than r_pp = n_pp fine cells attracts by
//     F_pp(r) = F_G(r) - F_l(r; r_pp),
// F_l(r; D) the attraction of two S2 clouds of diameter D (Hockney &
// Eastwood's reference force), which equals F_G from r = D on; the fine
// mesh's kernel leaves this part out (green.hip).  With xi = 2 r / D:
//     4 pi D^2 F_l = (224 xi - 224 xi^3 + 70 xi^4 + 48 xi^5 - 21 xi^6) / 35,  xi <= 1
//                  = (12/xi^2 - 224 + 896 xi - 840 xi^2 + 224 xi^3 + 70 xi^4
//                     - 48 xi^5 + 7 xi^6) / 35,                            1 <= xi <= 2.
// r_pp <= H, so a particle's partners lie in its own or the adjacent coarse
// cells.  Positions stay in the fixed-point format: per axis the separation
// is 256 (cell' - cell) + m' - m quanta (|.| < 512), the squared distance is
// an exact integer from a packed 16-bit dot product (the CDNA analogue of
// the paper's 8-bit VNNI distances), and only pairs inside r_pp reach the
// FP32 force polynomial.  Coincident particles (and a particle with itself)
// exert nothing.
//
// One workgroup per x-row of Tc coarse cells of a tile (a contiguous run of
// the canonical order), a particle per thread, 256 consecutive ones at a time.
// The packed positions of the 3 x 3 neighbouring rows are staged in LDS (a
// row's middle Tc cells are one particle range); a thread then walks, per row
// its r_pp sphere reaches, the contiguous run of the cells it reaches along x.
// All nine rows at their full length where they fit the kPPCap particles of
// the stage; else for every 256 particles the cells around theirs, as many
// rows at a time as fit.  64^3 particles, r = 4, r_pp = 4 fine cells, 60 / 115 /
// 160 / 300 particles in every filled cell: 1.36 / 3.6 / 5.8 / 14 ms; all pairs
// from global memory 1.6 / 4.0 / 6.3 / 17; pieces of whole cells, which leave
// lanes idle, and a cell that does not fit by itself, 1.6 / 5.8 / 8.7 / 24.
//
// Pairs come from global memory where a row's range alone exceeds the stage
// and, when the reach is less than a cell, where the rows would take more than
// kPPGroups stages: most lanes then need half of the rows at most and wait
// while the others are walked.  460 particles a cell, reaches of 1/4 to 3/4
// cell: 0.87 to 0.93 of the time above, 1.11 to 1.23 of it in five stages; 300
// a cell, three stages: 0.4 to 0.9.  With a whole cell's reach every lane needs
// every row, and staging is faster at any number (0.87 at 600 a cell).
//
// Bound by instruction issue (1.19 vector instructions per clock and CU on
// 1024^3 particles, 26 of 64 lanes at work).  One particle in six of a neighbourhood is in reach,
// yet some lane of a wave is at almost every step, so a single loop computes
// the weight at every step.  Here the loop over partners only measures
// distances and lists the pairs in reach; the weights are computed from the
// lists, in the order the pairs were met (96^3 particles, r_pp = 4 fine cells:
// 240 us -> 207; with lists of 24 or 32 pairs 4 and 13 % more; 197 with the
// staging loads in flight together).
//
// The accelerations go to three FP32 planes in canonical order, which the
// gather adds to the mesh force before the kick.
#include <cmath>

#include "common.h"

namespace cube {

namespace {

typedef short v2i16 __attribute__((ext_vector_type(2)));

constexpr int kPPThreads = 256;
constexpr int kPPCap = 4096;     // neighbour particles a workgroup stages in LDS
constexpr int kPPList = 16;      // pairs a thread lists before their weights are computed
constexpr int kPPPad = 3;        // out-of-reach entries behind each staged row
constexpr int kPPGroups = 3;     // stages for one batch's rows, at most, where the reach is less than a cell
static_assert(16 * kPPCap == 65536, "a list entry holds the row and the place in LDS");

struct PPParams {
    int reach;        // r_pp in position quanta: 256 n_pp / r
    int reach2;       // its square
    float two_over;   // 2 / reach: xi per quantum
    float amp;        // (256 / H)^2 / (4 pi) / 140: quanta to spacings, 4 pi G = 1
};

// F_pp / r per quantum of separation, in units of amp, for 0 < u < reach:
// F_pp = F_G R(xi) / 140 with R = 140 - 35 xi^2 (4 pi D^2 F_l), i.e.
//     R = 140 - xi^3 (224 - 224 xi^2 + 70 xi^3 + 48 xi^4 - 21 xi^5)   (xi <= 1)
//     R = t^5 (168 - 182 t + 64 t^2 - 7 t^3),  t = 2 - xi           (1 <= xi < 2)
// The second line is the outer branch rewritten about xi = 2, where the pair
// force vanishes to fifth order: evaluated in t it has no FP32 cancellation.
__device__ __forceinline__ float pp_weight(int r2, const PPParams& P) {
    const float u2 = (float)r2;                   // exact: 1 <= r2 < 2^24
    const float inv_u = __builtin_amdgcn_rsqf(u2);
    const float x = u2 * inv_u * P.two_over;
    float R;
    if (x <= 1.0f) {
        R = 140.0f - x * x * x * (224.0f + x * x * (-224.0f + x * (70.0f + x * (48.0f - 21.0f * x))));
    } else {
        const float t = 2.0f - x, t2 = t * t;
        R = t2 * t2 * t * (168.0f + t * (-182.0f + t * (64.0f - 7.0f * t)));
    }
    return R * inv_u * inv_u * inv_u;
}

// partner loop of one neighbour cell in global memory: accumulate the pair
// accelerations of the particles [q0, q1) whose cell sits dx, dy, dz coarse
// cells away
__device__ __forceinline__ void pp_cell(int q0, int q1, int dx, int dy, int dz, const int m[3], const Planes& in,
                                        const PPParams& P, float& a0, float& a1, float& a2) {
    for (int q = q0; q < q1; ++q) {
        const int sx = 256 * dx + in.m[0][q] - m[0];
        const int sy = 256 * dy + in.m[1][q] - m[1];
        const int sz = 256 * dz + in.m[2][q] - m[2];
        const v2i16 xy = {(short)sx, (short)sy};
        const int r2 = __builtin_amdgcn_sdot2(xy, xy, sz * sz, false);
        if (r2 == 0 || r2 >= P.reach2) continue;
        const float w = pp_weight(r2, P);
        a0 += w * (float)sx;
        a1 += w * (float)sy;
        a2 += w * (float)sz;
    }
}

// Dynamic LDS: own row offsets [Tc + 1], per neighbour row the particles in
// front of its Tc + 2 cells [9][Tc + 3], up to kPPCap packed positions, the
// threads' pair lists [kPPList][threads].
__global__ __launch_bounds__(kPPThreads) void k_pp(Geom g, const int32_t* __restrict__ offsets, Planes in,
                                                  float* __restrict__ ax_out, float* __restrict__ ay_out,
                                                  float* __restrict__ az_out, PPParams P) {
    extern __shared__ int lds[];
    const int Tc = g.Tc, RW = Tc + 3;
    int* offs = lds;
    int* s_off = offs + (Tc + 1);
    uint32_t* s_pos = reinterpret_cast<uint32_t*>(s_off + 9 * RW);
    uint16_t* s_list = reinterpret_cast<uint16_t*>(s_pos + kPPCap) + threadIdx.x;
    // per neighbour row (dy, dz) = (r % 3 - 1, r / 3 - 1): its first middle
    // cell and the global particle ranges of the middle cells and of the
    // cells just left and right of them
    __shared__ int64_t s_cm[9];
    __shared__ int s_rng[9][6];
    __shared__ int s_base[10];
    const Chunk ch = chunk_of(g, blockIdx.x);
    const int Nc = g.Nc;
    for (int j = threadIdx.x; j <= Tc; j += blockDim.x) offs[j] = offsets[ch.c0 + j];
    if (threadIdx.x < 9) {
        const int r = threadIdx.x;
        const int y = wrapi(ch.cy + r % 3 - 1, Nc), z = wrapi(ch.cz + r / 3 - 1, Nc);
        const int64_t cm = canon(g, ch.cx0, y, z);      // Tc consecutive cells from here
        const int64_t cl = canon(g, wrapi(ch.cx0 - 1, Nc), y, z);
        const int64_t cr = canon(g, wrapi(ch.cx0 + Tc, Nc), y, z);
        s_cm[r] = cm;
        s_rng[r][0] = offsets[cm];
        s_rng[r][1] = offsets[cm + Tc];
        s_rng[r][2] = offsets[cl];
        s_rng[r][3] = offsets[cl + 1];
        s_rng[r][4] = offsets[cr];
        s_rng[r][5] = offsets[cr + 1];
    }
    __syncthreads();
    // s_off: per row, the particles in front of each of its Tc + 2 cells (left
    // cell, middle cells, right cell)
    for (int e = threadIdx.x; e < 9 * RW; e += blockDim.x) {
        const int r = e / RW, i = e - r * RW;
        const int nl = s_rng[r][3] - s_rng[r][2], nr = s_rng[r][5] - s_rng[r][4];
        int v = 0;
        if (i > 0) v = nl + (offsets[s_cm[r] + min(i - 1, Tc)] - s_rng[r][0]) + (i == Tc + 2 ? nr : 0);
        s_off[e] = v;
    }
    __syncthreads();
    const int p_begin = offs[0], p_end = offs[Tc];
    int around = 9 * kPPPad;
    for (int r = 0; r < 9; ++r) around += s_off[r * RW + Tc + 2];
    const bool whole = around <= kPPCap;                     // one stage serves the whole row

    // the neighbours of the row's cells [x0, x1) in rows [g0, g1), staged: four
    // particles of the rows' concatenation at a time, their loads in flight
    // together: 256 i + m along x (i the cell within the row), the bytes along
    // y and z
    auto stage = [&](int g0, int g1, int x0, int x1) {
        __syncthreads();                                     // the last stage has been read
        if (threadIdx.x == 0) {
            int b = 0;
            for (int r = 0; r < 10; ++r) {
                s_base[r] = r <= g1 ? b : 1 << 30;
                if (r >= g0 && r < g1) b += s_off[r * RW + x1 + 2] - s_off[r * RW + x0] + kPPPad;
            }
        }
        __syncthreads();
        const int all = s_base[g1], step = (int)blockDim.x;
        for (int e0 = threadIdx.x; e0 < all; e0 += 4 * step) {
            uint32_t b0[4], b1[4], b2[4];
            int row[4], at[4];
            bool pad[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = min(e0 + u * step, all - 1);
                int r = 0;
#pragma unroll
                for (int i = 1; i < 9; ++i) r += e >= s_base[i];
                const int k = e - s_base[r] + s_off[r * RW + x0];
                const int nl = s_rng[r][3] - s_rng[r][2], nm = s_rng[r][1] - s_rng[r][0];
                const int ql = s_rng[r][2] + k, qm = s_rng[r][0] + (k - nl), qr = s_rng[r][4] + (k - nl - nm);
                pad[u] = e >= s_base[r + 1] - kPPPad;
                row[u] = r;
                at[u] = k;
                // (no branches: the loads of all four are in flight together)
                const int q = pad[u] ? 0 : k < nl ? ql : k < nl + nm ? qm : qr;
                b0[u] = in.m[0][q];
                b1[u] = in.m[1][q];
                b2[u] = in.m[2][q];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * step;
                // the cell: largest i with s_off[i] <= at, i < Tc + 2 < 128
                const int* o = s_off + row[u] * RW;
                int i = 0;
#pragma unroll
                for (int half = 64; half > 0; half >>= 1) {
                    const int v = o[min(i + half, Tc + 2)];
                    i = (i + half < Tc + 2) & (v <= at[u]) ? i + half : i;
                }
                const uint32_t w = (uint32_t)(256 * i) + b0[u] | b1[u] << 16 | b2[u] << 24;
                if (e < all) s_pos[e] = pad[u] ? 0xffffu : w;
            }
        }
        __syncthreads();
    };

    // A particle per thread: the loops and their barriers are uniform over the
    // workgroup.
    for (int p0 = p_begin; p0 < p_end; p0 += kPPThreads) {
        int x0 = 0, x1 = Tc;
        if (!whole) {
            x0 = find_cell(offs, Tc, p0);
            x1 = find_cell(offs, Tc, min(p0 + kPPThreads, p_end) - 1) + 1;
        }
        const int p = p0 + (int)threadIdx.x;
        const bool live = p < p_end;
        const int j = find_cell(offs, Tc, live ? p : p0);
        const int c[3] = {ch.cx0 + j, ch.cy, ch.cz};
        int m[3], lo[3], hi[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            m[k] = live ? in.m[k][p] : 0;
            lo[k] = m[k] < P.reach ? -1 : 0;            // the sphere crosses the lower face
            hi[k] = m[k] + P.reach > 255 ? 1 : 0;       // ... the upper face
            if (!live) hi[k] = lo[k] - 1;               // no rows
        }
        float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f;
        // rows that fit the stage together form a group; bit r: one begins at row r
        unsigned cuts = 0;
        bool staged = true;
        if (!whole) {
            int n = 0;
#pragma unroll
            for (int r = 0; r < 9; ++r) {
                const int len = s_off[r * RW + x1 + 2] - s_off[r * RW + x0] + kPPPad;
                staged = staged && len <= kPPCap;
                n += len;
                if (n > kPPCap) {
                    cuts |= 1u << r;
                    n = len;
                }
            }
            staged = staged && (__popc(cuts) < kPPGroups || P.reach == 256);
        }
        if (staged) {
            for (int g0 = 0, g1; g0 < 9; g0 = g1) {
                const unsigned later = cuts >> (g0 + 1);
                g1 = later ? g0 + __ffs(later) : 9;
                if (!whole || p0 == p_begin) stage(g0, g1, x0, x1);
                const int xp = 256 * (j + 1) + m[0];
                const uint32_t lim = (uint32_t)(P.reach2 - 1);
                int n = 0;
                // the weights of the pairs listed so far, in the order they were met
                const int yp = m[1] + 256, zp = m[2] + 256;       // (dy + 1 and dz + 1 are kept)
                auto flush = [&]() {
                    int e = s_list[0];
                    uint32_t w = s_pos[e & (kPPCap - 1)];
                    for (int i = 0; i < n;) {
                        const int sx = (int)(w & 0xffffu) - xp;
                        const int sy = (int)((w >> 16) & 255u) - yp + 256 * ((e >> 12) & 3);
                        const int sz = (int)(w >> 24) - zp + 256 * (e >> 14);
                        ++i;                                      // the next pair's reads in flight
                        e = s_list[(i & (kPPList - 1)) * kPPThreads];
                        w = s_pos[e & (kPPCap - 1)];
                        const float f = pp_weight(__mul24(sx, sx) + __mul24(sy, sy) + __mul24(sz, sz), P);
                        a0 += f * (float)sx;
                        a1 += f * (float)sy;
                        a2 += f * (float)sz;
                    }
                    n = 0;
                };
                for (int dz = lo[2]; dz <= hi[2]; ++dz) {
                    const int zd = zp - 256 * (dz + 1);
                    for (int dy = lo[1]; dy <= hi[1]; ++dy) {
                        const int r = (dz + 1) * 3 + (dy + 1);
                        if (r < g0 || r >= g1) continue;
                        const int* row = s_off + r * RW + j;
                        const int shift = s_base[r] - s_off[r * RW + x0];
                        const int tag = ((dz + 1) * 4 + (dy + 1)) * kPPCap;
                        const int q1 = row[2 + hi[0]] + shift;
                        const v2i16 own = {(short)xp, (short)(yp - 256 * (dy + 1))};
                        // (what a group reads past q1 is out of reach: farther
                        // cells of the row or its padding)
                        for (int q = row[1 + lo[0]] + shift; q < q1; q += 4) {
                            uint32_t w[4];
#pragma unroll
                            for (int k = 0; k < 4; ++k) w[k] = s_pos[q + k];
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const v2i16 d = __builtin_bit_cast(v2i16, w[k] & 0x00ffffffu) - own;
                                const int sz = (int)(w[k] >> 24) - zd;
                                // 0 < r^2 < reach^2 as one comparison
                                const uint32_t r2 = (uint32_t)__builtin_amdgcn_sdot2(d, d, __mul24(sz, sz) - 1, false);
                                if (r2 < lim) s_list[n++ * kPPThreads] = (uint16_t)(q + k + tag);
                            }
                            if (__any(n > kPPList - 4)) flush();
                        }
                    }
                }
                flush();
            }
        } else {
            for (int dz = lo[2]; dz <= hi[2]; ++dz)
                for (int dy = lo[1]; dy <= hi[1]; ++dy)
                    for (int dx = lo[0]; dx <= hi[0]; ++dx) {
                        const int64_t cn = canon(g, wrapi(c[0] + dx, Nc), wrapi(c[1] + dy, Nc), wrapi(c[2] + dz, Nc));
                        pp_cell(offsets[cn], offsets[cn + 1], dx, dy, dz, m, in, P, a0, a1, a2);
                    }
        }
        if (live) {
            ax_out[p] = a0 * P.amp;
            ay_out[p] = a1 * P.amp;
            az_out[p] = a2 * P.amp;
        }
    }
}

}  // namespace

void launch_pp(const Geom& g, const int32_t* offsets, Planes in, float* const acc[3], hipStream_t s) {
    PPParams P;
    P.reach = 256 * g.npp / g.r;
    P.reach2 = P.reach * P.reach;
    P.two_over = 2.0f / (float)P.reach;
    const double q_per_spacing = 256.0 * g.f / g.r;          // 256 / H
    P.amp = (float)(q_per_spacing * q_per_spacing / (4.0 * M_PI * 140.0));
    const int64_t chunks = g.ncells / g.Tc;
    const size_t lds = sizeof(int) * ((size_t)(g.Tc + 1) + 9 * (size_t)(g.Tc + 3) + kPPCap) +
                       sizeof(uint16_t) * (size_t)kPPList * kPPThreads;
    hipLaunchKernelGGL(k_pp, dim3((unsigned)chunks), dim3(kPPThreads), lds, s, g, offsets, in, acc[0], acc[1], acc[2],
                       P);
}

}  // namespace cube
