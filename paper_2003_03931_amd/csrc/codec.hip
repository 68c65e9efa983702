// Fixed-point particle codec (Sec. III-A, Eq. (2)).
//
// Positions: per axis the global quantum Q = floor(x * 256 / H) mod 256 N_c,
// stored as the byte m = Q mod 256 in canonical cell order; decoding gives the
// bin centre (Q + 1/2) H / 256, exact in FP32.  Velocities: one signed byte
// per axis, u = clamp(rint(v / s), -127, 127) with a power-of-two scale s, or
// (cell-mean codec) the FP32 velocities are placed in cell order here and
// encoded by vcodec.hip.
#include <algorithm>

#include "common.h"

namespace cube {

namespace {

// Four consecutive particles' rows of three floats: as three float4s where
// the caller's arrays are aligned for it.
template <bool VEC>
__device__ __forceinline__ void load_rows(const float* __restrict__ p, int64_t i4, float r[12]) {
    if constexpr (VEC) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const float4 v = reinterpret_cast<const float4*>(p)[3 * i4 + j];
            r[4 * j] = v.x;
            r[4 * j + 1] = v.y;
            r[4 * j + 2] = v.z;
            r[4 * j + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 12; ++j) r[j] = p[12 * i4 + j];
    }
}

// Cell keys and in-cell bytes of the positions, and the largest |velocity
// component| (as bits: non-negative floats order like them).  Four particles
// per thread (their number is a multiple of 64); memory-bound.
template <bool VEC>
__global__ __launch_bounds__(256) void k_encode_keys(Geom g, const float* __restrict__ pos,
                                                     const float* __restrict__ vel, uint32_t* __restrict__ key,
                                                     uint32_t* __restrict__ qpack, uint32_t* __restrict__ vmax,
                                                     int64_t n4) {
    __shared__ int red[256 / kWave];
    const double scale = 256.0 * g.f / g.r;          // 256 / H, a power of two
    const int64_t nq = 256 * (int64_t)g.Nc;
    const float inv_tc = 1.0f / (float)g.Tc;
    uint32_t m = 0;
    for (int64_t i4 = (int64_t)blockIdx.x * 256 + threadIdx.x; i4 < n4; i4 += (int64_t)gridDim.x * 256) {
        float x[12], v[12];
        load_rows<VEC>(pos, i4, x);
        load_rows<VEC>(vel, i4, v);
        uint32_t kk[4], qq[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            int q[3], t[3], l[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                int64_t w = (int64_t)floor((double)x[3 * u + k] * scale);
                if (w < 0 || w >= nq) {              // outside the box: wrap
                    w %= nq;
                    w = w < 0 ? w + nq : w;
                }
                q[k] = (int)w;
                const int c = q[k] >> 8;
                t[k] = (int)(((float)c + 0.5f) * inv_tc);    // c / Tc: exact for c < 2^10
                l[k] = c - t[k] * g.Tc;
                m = max(m, __float_as_uint(fabsf(v[3 * u + k])));
            }
            const int tile = t[0] + g.nt * (t[1] + g.nt * t[2]);
            kk[u] = (uint32_t)(tile * (g.Tc * g.Tc * g.Tc) + l[0] + g.Tc * (l[1] + g.Tc * l[2]));
            qq[u] = (uint32_t)(q[0] & 255) | ((uint32_t)(q[1] & 255) << 8) | ((uint32_t)(q[2] & 255) << 16);
        }
        reinterpret_cast<uint4*>(key)[i4] = make_uint4(kk[0], kk[1], kk[2], kk[3]);
        reinterpret_cast<uint4*>(qpack)[i4] = make_uint4(qq[0], qq[1], qq[2], qq[3]);
    }
    const int mw = wave_max((int)m);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = mw;
    __syncthreads();
    if (threadIdx.x == 0) {
        int mb = red[0];
        for (int w = 1; w < 256 / kWave; ++w) mb = max(mb, red[w]);
        // one address for the whole grid: skip the atomic the maximum covers
        if ((uint32_t)mb > *(volatile uint32_t*)vmax) atomicMax(vmax, (uint32_t)mb);
    }
}

// Fresh step scalars; the velocity scale is the power of two at or above
// headroom * max|v| / 127 (1 when nothing moves).
__global__ __launch_bounds__(256) void k_compress_scalars(StepScalars* sc, const uint32_t* __restrict__ vmax,
                                                          double headroom) {
    for (int i = threadIdx.x; i < (int)(sizeof(StepScalars) / sizeof(int32_t)); i += 256)
        reinterpret_cast<int32_t*>(sc)[i] = 0;
    __syncthreads();
    if (threadIdx.x != 0) return;
    const float v = __uint_as_float(*vmax);
    double s = 1.0;
    if (v > 0.0f && !isinf(v)) {
        int e;
        const double m = frexp(headroom * (double)v / 127.0, &e);
        s = ldexp(1.0, m == 0.5 ? e - 1 : e);
    }
    sc->s = s;
    sc->s_next = s;
}

// First index in the sorted keys [lo, hi) whose key is at least c.
__device__ __forceinline__ int lower_bound(const uint32_t* __restrict__ key, int lo, int hi, uint32_t c) {
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (key[mid] < c) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Offsets and counts of 256 cells from the sorted keys: the workgroup narrows
// the keys to its cells' range with 256 probes a round, then finds where they
// change: all of the range's keys are read, or, in a range longer than
// kWalkKeys, each cell's first key is searched.  (Counting 11.2 million keys
// one by one took 396 us of atomics, this takes 43 to 49.)
constexpr int kWalkKeys = 1 << 14;

__global__ __launch_bounds__(256) void k_key_offsets(const uint32_t* __restrict__ key, int64_t n, int64_t ncells,
                                                      int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                      int32_t* __restrict__ max_out) {
    __shared__ int below[2][256 / kWave];
    __shared__ int s_off[257];
    const int64_t c0 = (int64_t)blockIdx.x * 256;
    const int nc = (int)min((int64_t)256, ncells - c0);
    // keys below c0 and below c0 + nc
    int64_t lo[2] = {0, 0}, hi[2] = {n, n};
    const uint32_t want[2] = {(uint32_t)c0, (uint32_t)(c0 + nc)};
    while (hi[0] - lo[0] > 0 || hi[1] - lo[1] > 0) {
        // probes split [lo, hi) in 257 parts; those below the wanted key count
        int64_t step[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            step[e] = (hi[e] - lo[e]) / 257 + 1;
            const int64_t at = lo[e] + (int64_t)(threadIdx.x + 1) * step[e] - 1;
            const bool b = at < hi[e] && key[at] < want[e];
            const int c = __popcll(__ballot(b));
            if ((threadIdx.x & (kWave - 1)) == 0) below[e][threadIdx.x / kWave] = c;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            int64_t c = 0;
            for (int w = 0; w < 256 / kWave; ++w) c += below[e][w];
            const int64_t a = lo[e] + c * step[e], z = min(hi[e], a + step[e] - 1);
            lo[e] = min(a, hi[e]);
            hi[e] = max(z, lo[e]);
        }
        __syncthreads();
    }
    const int t = threadIdx.x;
    const int st = (int)lo[0], en = (int)lo[1];
    if (en - st > kWalkKeys) {
        if (t < nc) s_off[t] = t == 0 ? st : lower_bound(key, st, en, (uint32_t)(c0 + t));
    } else {
        if (t < nc) s_off[t] = en;                  // cells past the last key
        __syncthreads();
        for (int e = st + t; e < en; e += 256) {
            const int c = (int)((int64_t)key[e] - c0), prev = e > st ? (int)((int64_t)key[e - 1] - c0) : -1;
            for (int x = prev + 1; x <= c; ++x) s_off[x] = e;
        }
    }
    if (t == 0) s_off[nc] = en;
    __syncthreads();
    int mx = 0;
    if (t < nc) {
        const int c = s_off[t + 1] - s_off[t];
        counts[c0 + t] = c;
        offsets[c0 + t] = s_off[t];
        if (c0 + t == ncells - 1) offsets[ncells] = en;
        mx = c;
    }
    mx = wave_max(mx);
    if ((t & (kWave - 1)) == 0 && mx > *(volatile int32_t*)max_out) atomicMax(max_out, mx);
}

// Four consecutive output particles per thread: gathers of the sorted rows,
// one 4-byte (velocities: 16-byte) store per plane.
__global__ __launch_bounds__(256) void k_scatter_compressed(const uint32_t* __restrict__ perm,
                                                            const uint32_t* __restrict__ qpack,
                                                            const float* __restrict__ vel, Planes out, StepScalars* sc,
                                                            int64_t n4) {
    __shared__ int red[2][256 / kWave];
    int sat = 0, umax = 0;
    const double inv_s = 1.0 / sc->s;                // exact: s is a power of two
    const int64_t j4 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j4 < n4) {
        const uint4 src4 = reinterpret_cast<const uint4*>(perm)[j4];
        const uint32_t src[4] = {src4.x, src4.y, src4.z, src4.w};
        uint32_t qp[4];
        float v[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            qp[u] = qpack[src[u]];
#pragma unroll
            for (int k = 0; k < 3; ++k) v[u][k] = vel[3 * (int64_t)src[u] + k];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            uint32_t w = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) w |= ((qp[u] >> (8 * k)) & 255u) << (8 * u);
            reinterpret_cast<uint32_t*>(out.m[k])[j4] = w;
        }
        if (out.v[0]) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                reinterpret_cast<float4*>(out.v[k])[j4] = make_float4(v[0][k], v[1][k], v[2][k], v[3][k]);
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                uint32_t b = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    double w = rint((double)v[u][k] * inv_s);
                    sat += fabs(w) > 127.0;
                    w = fmin(fmax(w, -127.0), 127.0);
                    const int c = (int)w;
                    umax = max(umax, abs(c));
                    b |= (uint32_t)(uint8_t)(int8_t)c << (8 * u);
                }
                reinterpret_cast<uint32_t*>(out.u[k])[j4] = b;
            }
        }
        if (out.ids) reinterpret_cast<uint4*>(out.ids)[j4] = src4;
    }
    if (out.v[0]) return;                    // codes are written by the cell-mean encoder
    sat = wave_sum(sat);
    umax = wave_max(umax);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[0][threadIdx.x / kWave] = sat;
        red[1][threadIdx.x / kWave] = umax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / kWave; ++w) {
            sat += red[0][w];
            umax = max(umax, red[1][w]);
        }
        if (sat) atomicAdd((unsigned long long*)&sc->saturations, (unsigned long long)sat);
        // one address for the whole grid: skip the atomic when the (monotone)
        // maximum already covers this workgroup
        if (umax > *(volatile int32_t*)&sc->max_u) atomicMax(&sc->max_u, umax);
    }
}

// A workgroup decodes the particles of up to kDecodeCells consecutive cells,
// four consecutive ones per thread (whole 4-byte loads of the planes, float4
// stores of the rows where the caller's arrays allow them; at the ends of the
// range, which may split such a four, one at a time).  Store-bound: 24 bytes
// out per particle for 6 in.  (A particle per thread, a row of cells per
// workgroup: 176 us for 11.2 million; this: 92.)  The launch sizes the groups
// for one round of 1024 particles.  In a concentrated state the few groups that
// hold the particles need many rounds and are too few to hide their latency, so
// four rounds' loads are issued together (2.1 million particles in 1/64 of the
// cells, 64 a cell on average: 402 us round by round, 69 so), and the launch may
// share a group among `gridDim.y` workgroups.
constexpr int kDecodeCells = 128;
constexpr int kDecodeRound = 4 * 256;        // particles
constexpr int kDecodeSet = 4;                // rounds loaded together

template <bool VEC>
__global__ __launch_bounds__(256) void k_decode(Geom g, const int32_t* __restrict__ offsets, int cells, Planes in,
                                                const StepScalars* __restrict__ sc, VelCells vcell,
                                                float* __restrict__ pos, float* __restrict__ vel) {
    __shared__ int offs[kDecodeCells + 1];
    __shared__ int cell[3][kDecodeCells];
    const int64_t c0 = (int64_t)blockIdx.x * cells;
    const int nc = (int)min((int64_t)cells, g.ncells - c0);
    const int lo = offsets[c0], hi = offsets[c0 + nc];
    // this workgroup's part of the fours that hold [lo, hi), whole rounds
    const int all4 = (hi + 3) / 4 - lo / 4, parts = (int)gridDim.y;
    const int part4 = (all4 + 256 * parts - 1) / (256 * parts) * 256;
    const int first4 = lo / 4 + (int)blockIdx.y * part4, end4 = min((hi + 3) / 4, first4 + part4);
    if (first4 >= end4) return;
    for (int j = threadIdx.x; j <= nc; j += 256) offs[j] = offsets[c0 + j];
    if ((int)threadIdx.x < nc) {
        const int64_t c = c0 + threadIdx.x, tc3 = (int64_t)g.Tc * g.Tc * g.Tc;
        const int tile = (int)(c / tc3), l = (int)(c - tile * tc3);
        cell[0][threadIdx.x] = tile % g.nt * g.Tc + l % g.Tc;
        cell[1][threadIdx.x] = tile / g.nt % g.nt * g.Tc + l / g.Tc % g.Tc;
        cell[2][threadIdx.x] = tile / (g.nt * g.nt) * g.Tc + l / (g.Tc * g.Tc);
    }
    __syncthreads();
    const float H256 = (float)g.r / (float)(256 * g.f);   // H / 256, a power of two
    const double s = sc->s;
    struct Four {
        uint32_t m[3], u[3];
    };
    auto load = [&](int p4) {
        Four f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            f.m[k] = reinterpret_cast<const uint32_t*>(in.m[k])[p4];
            f.u[k] = reinterpret_cast<const uint32_t*>(in.u[k])[p4];
        }
        return f;
    };
    auto put = [&](int p4, const Four& f) {
        const int p = 4 * p4;
        int j = find_cell_fixed<7>(offs, nc, max(p, lo));
        int next = offs[j + 1], at[3];           // the cell's end and coordinates
#pragma unroll
        for (int k = 0; k < 3; ++k) at[k] = cell[k][j] * 256;
        float x[12], v[12];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (next <= p + e && j + 1 < nc) {
                do next = offs[++j + 1]; while (next <= p + e && j + 1 < nc);
#pragma unroll
                for (int k = 0; k < 3; ++k) at[k] = cell[k][j] * 256;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int q = at[k] + (int)((f.m[k] >> (8 * e)) & 255u);
                x[3 * e + k] = ((float)q + 0.5f) * H256;
                const int c = (int)(int8_t)(f.u[k] >> (8 * e));
                v[3 * e + k] = g.vcodec ? (float)vc_decode(vcell.vc[k][c0 + j], s, vcell.tab, c) : (float)c * (float)s;
            }
        }
        if (p >= lo && p + 4 <= hi) {
            if constexpr (VEC) {
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    reinterpret_cast<float4*>(pos)[3 * (int64_t)p4 + e] =
                        make_float4(x[4 * e], x[4 * e + 1], x[4 * e + 2], x[4 * e + 3]);
                    reinterpret_cast<float4*>(vel)[3 * (int64_t)p4 + e] =
                        make_float4(v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 12; ++e) {
                    pos[3 * (int64_t)p + e] = x[e];
                    vel[3 * (int64_t)p + e] = v[e];
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (p + e >= lo && p + e < hi)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        pos[3 * ((int64_t)p + e) + k] = x[3 * e + k];
                        vel[3 * ((int64_t)p + e) + k] = v[3 * e + k];
                    }
        }
    };
    int p4 = first4 + (int)threadIdx.x;
    // whole sets of rounds, every load within the range
    constexpr int step = kDecodeSet * 256;
    for (int at = first4; at + step <= end4; at += step, p4 += step) {
        Four f[kDecodeSet];
#pragma unroll
        for (int u = 0; u < kDecodeSet; ++u) f[u] = load(p4 + 256 * u);
#pragma unroll
        for (int u = 0; u < kDecodeSet; ++u) put(p4 + 256 * u, f[u]);
    }
    for (; p4 < end4; p4 += 256) put(p4, load(p4));
}

bool aligned16(const void* a, const void* b) {
    return ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0;
}

}  // namespace

void launch_encode_keys(const Geom& g, const float* pos, const float* vel, uint32_t* key, uint32_t* qpack,
                        uint32_t* vmax, int64_t n, hipStream_t s) {
    launch_fill_i32(reinterpret_cast<int32_t*>(vmax), 0, 1, s);
    const unsigned blocks = std::min(grid1d(n / 4, 256), 8192u);
    if (aligned16(pos, vel))
        hipLaunchKernelGGL(k_encode_keys<true>, dim3(blocks), dim3(256), 0, s, g, pos, vel, key, qpack, vmax, n / 4);
    else
        hipLaunchKernelGGL(k_encode_keys<false>, dim3(blocks), dim3(256), 0, s, g, pos, vel, key, qpack, vmax, n / 4);
}

void launch_compress_scalars(StepScalars* sc, const uint32_t* vmax, float headroom, hipStream_t s) {
    hipLaunchKernelGGL(k_compress_scalars, dim3(1), dim3(256), 0, s, sc, vmax, (double)headroom);
}

void launch_key_offsets(const uint32_t* sorted_key, int64_t n, int64_t ncells, int32_t* counts, int32_t* offsets,
                        int32_t* max_out, hipStream_t s) {
    hipLaunchKernelGGL(k_key_offsets, dim3(grid1d(ncells, 256)), dim3(256), 0, s, sorted_key, n, ncells, counts,
                       offsets, max_out);
}

void launch_scatter_compressed(const uint32_t* perm, const uint32_t* qpack, const float* vel, Planes out,
                               StepScalars* sc, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_scatter_compressed, dim3(grid1d(n / 4, 256)), dim3(256), 0, s, perm, qpack, vel, out, sc,
                       n / 4);
}

void launch_decode(const Geom& g, const int32_t* offsets, Planes in, const StepScalars* sc,
                   const VelCells& vcell, float* pos, float* vel, int max_count, hipStream_t s) {
    // As many cells as hold one round's particles on average (with 128 whatever
    // they hold, 4096 cells of 64 particles took 39 us, 25 now), and few enough
    // for eight workgroups per CU, but not below 16: a row of cells per
    // workgroup was faster than 128 cells in boxes too small to fill the chip.
    const int64_t round = std::max<int64_t>(1, kDecodeRound * g.ncells / g.n);
    const int64_t fill = std::max<int64_t>(16, g.ncells / (8 * device_cus()));
    const int cells = (int)std::min({round, fill, (int64_t)kDecodeCells});
    // Few groups of which some may hold many rounds' particles: up to eight
    // workgroups each (2.1 million particles in 1/64 of the cells, 8 a cell on
    // average: 123 us undivided, 68 shared by eight).  In a large box the extra
    // workgroups, mostly idle, would cost more than the longest group.
    const unsigned groups = grid1d(g.ncells, cells);
    const bool heavy = (int64_t)cells * max_count > 8 * kDecodeRound;
    const dim3 grid(groups, heavy ? std::min(8u, std::max(1u, 16384 / groups)) : 1), block(256);
    if (aligned16(pos, vel))
        hipLaunchKernelGGL(k_decode<true>, grid, block, 0, s, g, offsets, cells, in, sc, vcell, pos, vel);
    else
        hipLaunchKernelGGL(k_decode<false>, grid, block, 0, s, g, offsets, cells, in, sc, vcell, pos, vel);
}

}  // namespace cube
