// Per-step scalar bookkeeping and FP64 diagnostics.
//
// Velocity scale update before each kick: s' = pow2ceil(h_v M s / 127) with M
// the max |u| left by the previous kick (kept at s when M = 0); evaluated in
// FP64 on the device so a multi-step call never waits for the host.
// Diagnostics: momentum and kinetic energy of the decoded velocities summed in
// FP64 in a fixed order (per-chunk partials, then one ordered reduction);
// power-spectrum shells binned in FP64.
#include <algorithm>
#include <cmath>

#include "common.h"

namespace cube {

namespace {

__device__ double pow2ceil_d(double x) {
    int e;
    const double m = frexp(x, &e);      // x = m 2^e, m in [0.5, 1)
    return m == 0.5 ? ldexp(1.0, e - 1) : ldexp(1.0, e);
}

__device__ __forceinline__ bool halted(const StepScalars* sc) { return *(volatile const int32_t*)&sc->halt != 0; }

// Begin of a step: counters of the running step, the coming kick's scale, the
// new counts cleared, the tiles' record cursors set.
__global__ __launch_bounds__(256) void k_step_begin(StepScalars* sc, double hv, int4* __restrict__ counts_new,
                                                    int64_t n4, const int32_t* __restrict__ offsets, int64_t tile_cells,
                                                    int32_t* __restrict__ tcursor, int ntiles) {
    if (halted(sc)) return;
    const int64_t stride = (int64_t)gridDim.x * 256, first = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t i = first; i < n4; i += stride) counts_new[i] = make_int4(0, 0, 0, 0);
    for (int64_t i = first; i < ntiles; i += stride) tcursor[i] = offsets[i * tile_cells];
    if (blockIdx.x != 0) return;
    if (threadIdx.x < 64) sc->umax_slot[threadIdx.x] = 0;
    else if (threadIdx.x < 128) sc->cmax_slot[threadIdx.x - 64] = 0;
    if (threadIdx.x != 0) return;
    const int M = sc->max_u;
    const double s = sc->s;
    sc->s_next = (M == 0) ? s : pow2ceil_d((hv * (double)M) * s / 127.0);
    sc->max_u_next = 0;
    sc->far_count = 0;
    sc->max_carry = 0;
    sc->overflow = 0;
    sc->sat_step = 0;
    sc->new_max_count = 0;
    sc->new_max_block8 = 0;
    sc->scan_ticket = 0;
    sc->commit_ticket = 0;
}

struct PlanCheck {
    int vcodec, planned_wide, planned_f16;
    double wide_cut, f16_cut, f3;
};

__device__ void epilogue(StepScalars* sc, const PlanCheck& pc) {
    int um = sc->max_u_next, cm = sc->max_carry;
    for (int i = 0; i < 64; ++i) {
        um = max(um, sc->umax_slot[i]);
        cm = max(cm, sc->cmax_slot[i]);
    }
    if (!pc.vcodec) {
        sc->s = sc->s_next;
        sc->max_u = um;
    }
    sc->max_carry = cm;
    sc->saturations += sc->sat_step;
    sc->sat_step = 0;
    sc->max_count = sc->new_max_count;
    sc->max_block8 = sc->new_max_block8;
    sc->steps_done += 1;
    // the next step was enqueued for narrower accumulators or FP16 densities
    const double b8 = (double)sc->max_block8;
    if ((!pc.planned_wide && b8 >= pc.wide_cut) || (pc.planned_f16 && pc.f3 * b8 + 1.0 >= pc.f16_cut)) sc->halt = 3;
}

__global__ void k_epilogue(StepScalars* sc, PlanCheck pc) {
    if (threadIdx.x == 0 && !halted(sc)) epilogue(sc, pc);
}

// counts <- counts_new and offsets <- offsets_new, 16 bytes at a time where
// aligned.  `last`: the last workgroup to finish commits the scalars; every
// workgroup has then read the halt flag that this may set.
__global__ __launch_bounds__(256) void k_commit_cells(const int32_t* __restrict__ cn, const int32_t* __restrict__ on,
                                                      int32_t* __restrict__ c, int32_t* __restrict__ o, int64_t ncells,
                                                      StepScalars* sc, int last, PlanCheck pc) {
    if (halted(sc)) return;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t n4 = ncells / 4;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
        reinterpret_cast<int4*>(c)[i] = reinterpret_cast<const int4*>(cn)[i];
        reinterpret_cast<int4*>(o)[i] = reinterpret_cast<const int4*>(on)[i];
    }
    for (int64_t i = 4 * n4 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= ncells; i += stride) {
        if (i < ncells) c[i] = cn[i];
        o[i] = on[i];
    }
    if (!last) return;
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(&sc->commit_ticket, 1) == (int)gridDim.x - 1) epilogue(sc, pc);
}

__global__ void k_fill(int32_t* p, int32_t v, int64_t n, const int32_t* gate) {
    if (gate && *(volatile const int32_t*)gate) return;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

// per chunk: sum v_x, v_y, v_z, v^2 in FP64 (v = u s, or the cell-mean
// decode v_c + sigma tan(u pi / 255))
__global__ __launch_bounds__(256) void k_moments(Geom g, const int32_t* __restrict__ offsets, Planes p,
                                                 const StepScalars* __restrict__ sc, VelCells vcell,
                                                 double* __restrict__ partial) {
    extern __shared__ int offs[];
    __shared__ double red[4][256 / kWave];
    const int64_t c0 = (int64_t)blockIdx.x * g.Tc;
    for (int j = threadIdx.x; j <= g.Tc; j += blockDim.x) offs[j] = offsets[c0 + j];
    __syncthreads();
    const int lo = offs[0], hi = offs[g.Tc];
    const double s = sc->s;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = lo + threadIdx.x; i < hi; i += blockDim.x) {
        const int64_t c = g.vcodec ? c0 + find_cell(offs, g.Tc, i) : 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double v = g.vcodec ? vc_decode(vcell.vc[k][c], s, vcell.tab, p.u[k][i]) : (double)p.u[k][i] * s;
            a[k] += v;
            a[3] += v * v;
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double v = wave_sum_d(a[k]);
        if ((threadIdx.x & (kWave - 1)) == 0) red[k][threadIdx.x / kWave] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        double t = 0.0;
        for (int w = 0; w < (int)(blockDim.x / kWave); ++w) t += red[threadIdx.x][w];
        partial[(int64_t)blockIdx.x * 4 + threadIdx.x] = t;
    }
}

// The same sums for linear codes v = u s: u and u^2 are summed as integers,
// four codes per load, and scaled once per workgroup.  Every partial sum is an
// integer (below 3 x 128^2 x 2^31 < 2^47, and doubles hold those below 2^53)
// times a power of two, so the result is the exact one.
// particles: how many the cells hold, all (a multiple of 4) or, in an empty
// box, none: its planes hold anything.
constexpr int kMomentThreads = 256;

__global__ __launch_bounds__(kMomentThreads) void k_moments_linear(Planes p, const int32_t* __restrict__ particles,
                                                                   const StepScalars* __restrict__ sc,
                                                                   double* __restrict__ partial) {
    __shared__ long long red[4][kMomentThreads / kWave];
    const int n4 = *particles / 4;
    long long t[4] = {0, 0, 0, 0};
    for (int i = (int)blockIdx.x * kMomentThreads + (int)threadIdx.x; i < n4; i += (int)gridDim.x * kMomentThreads) {
        int sq = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t w = reinterpret_cast<const uint32_t*>(p.u[k])[i];
            int sum = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int u = (int)(int8_t)(w >> (8 * e));
                sum += u;
                sq += u * u;
            }
            t[k] += sum;
        }
        t[3] += sq;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) t[k] += __shfl_xor(t[k], d, kWave);
        if ((threadIdx.x & (kWave - 1)) == 0) red[k][threadIdx.x / kWave] = t[k];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        long long v = 0;
        for (int w = 0; w < kMomentThreads / kWave; ++w) v += red[threadIdx.x][w];
        const double s = sc->s;
        partial[(int64_t)blockIdx.x * 4 + threadIdx.x] = (double)v * (threadIdx.x < 3 ? s : s * s);
    }
}

// out[c] (+)= sum_b partial[b * width + c], fixed order
__global__ __launch_bounds__(1024) void k_reduce_partials(const double* __restrict__ partial, int nblocks, int width,
                                                          double* __restrict__ out, int add) {
    __shared__ double red[1024 / kWave];
    const int c = blockIdx.x;
    double acc = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) acc += partial[(int64_t)b * width + c];
    acc = wave_sum_d(acc);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < (int)(blockDim.x / kWave); ++w) t += red[w];
        out[c] = add ? out[c] + t : t;
    }
}

// floor(sqrt(v)) of a non-negative integer, exactly
__device__ __forceinline__ long isqrt_floor(long v) {
    long q = (long)sqrt((double)v);
    while (q * q > v) --q;
    while ((q + 1) * (q + 1) <= v) ++q;
    return q;
}

// Shell sums of |dk|^2 / n^3, mode counts and |k| sums, a wave per z-plane and
// shell.  A mode with integer |m|^2 = r2 falls in shell j = floor(sqrt(r2) +
// 1/2) exactly when j^2 - j + 1 <= r2 <= j^2 + j, so a wave walks its shell's
// modes of the plane: a row m_y per lane, |m_x| ascending, + before -, and
// the lanes are added in a fixed order: the sums do not depend on scheduling,
// and the spectrum is reproducible bit for bit.  (A thread per shell left most
// of the chip idle: 355 us at 256^3, this takes 31.)
constexpr int kBinWaves = 4;

__global__ __launch_bounds__(kBinWaves* kWave) void k_power_bins(const float2* __restrict__ dk, int n, int nbins,
                                                                 double* __restrict__ partial) {
    const int z = blockIdx.y;
    const int j = (int)blockIdx.x * kBinWaves + (int)threadIdx.x / kWave + 1;
    if (j > nbins) return;
    const int lane = threadIdx.x & (kWave - 1);
    const long mz = z <= n / 2 - 1 ? z : z - n;
    const int half = n / 2;
    const double inv_n3 = 1.0 / ((double)n * n * n);
    const double kf = 2.0 * M_PI / n;
    double ps = 0.0, ks = 0.0, cs = 0.0;
    const long A0 = (long)j * j - j + 1 - mz * mz, B0 = (long)j * j + j - mz * mz;
    if (B0 >= 0) {
        const long ymax = isqrt_floor(B0);
        for (long my = -ymax + lane; my <= ymax; my += kWave) {
            if (my < -half || my > half - 1) continue;
            const long A = A0 - my * my, B = B0 - my * my;
            if (B < 0) continue;
            long lo = 0;
            if (A > 0) {
                lo = isqrt_floor(A - 1) + 1;                        // ceil(sqrt(A))
            }
            const long hi = isqrt_floor(B);
            const int y = (int)(my >= 0 ? my : my + n);
            for (long mx = lo; mx <= hi; ++mx) {
                const double r = sqrt((double)(mx * mx + my * my + mz * mz));
#pragma unroll
                for (int sgn = 0; sgn < 2; ++sgn) {
                    if (sgn == 1 && mx == 0) break;
                    const long sx = sgn ? -mx : mx;
                    if (sx < -half || sx > half - 1) continue;
                    const int x = (int)(sx >= 0 ? sx : sx + n);
                    const float2 v = dk[((int64_t)z * n + y) * n + x];
                    ps += ((double)v.x * v.x + (double)v.y * v.y) * inv_n3;
                    ks += r * kf;
                    cs += 1.0;
                }
            }
        }
    }
    ps = wave_sum_d(ps);
    ks = wave_sum_d(ks);
    cs = wave_sum_d(cs);
    if (lane == 0) {
        partial[(int64_t)z * 3 * nbins + (j - 1)] = ps;
        partial[(int64_t)z * 3 * nbins + nbins + (j - 1)] = ks;
        partial[(int64_t)z * 3 * nbins + 2 * nbins + (j - 1)] = cs;
    }
}

// out[i] = sum over z of partial[z][i], a wave per i, fixed order
__global__ __launch_bounds__(kBinWaves* kWave) void k_sum_planes(const double* __restrict__ partial, int n, int width,
                                                                 double* __restrict__ out) {
    const int i = (int)blockIdx.x * kBinWaves + (int)threadIdx.x / kWave;
    if (i >= width) return;
    double t = 0.0;
    for (int z = threadIdx.x & (kWave - 1); z < n; z += kWave) t += partial[(int64_t)z * width + i];
    t = wave_sum_d(t);
    if ((threadIdx.x & (kWave - 1)) == 0) out[i] = t;
}

}  // namespace

void launch_step_begin(const Geom& g, StepScalars* sc, float v_headroom, const int32_t* offsets, int32_t* counts_new,
                       int32_t* tcursor, hipStream_t s) {
    // a side of the coarse mesh is a multiple of 4
    const unsigned blocks = std::min(grid1d(g.ncells / 4, 256), 4096u);
    hipLaunchKernelGGL(k_step_begin, dim3(blocks), dim3(256), 0, s, sc, (double)v_headroom,
                       reinterpret_cast<int4*>(counts_new), g.ncells / 4, offsets, (int64_t)g.Tc * g.Tc * g.Tc, tcursor,
                       g.ntiles);
}

void launch_step_commit(const Geom& g, StepScalars* sc, const int32_t* counts_new, const int32_t* offsets_new,
                        int32_t* counts, int32_t* offsets, bool planned_wide, bool planned_f16, hipStream_t s) {
    // 32-bit fine accumulators hold D^3 units per particle of a 2x2x2 block of
    // coarse cells; FP16 density spectra hold f^3 per particle of such a block
    const PlanCheck pc{g.vcodec, planned_wide ? 1 : 0, planned_f16 ? 1 : 0, std::ldexp(1.0, 32 - 3 * g.log2D), 32768.0,
                       (double)g.f * g.f * g.f};
    const unsigned blocks = std::min(grid1d(g.ncells / 4 + 1, 256), 8192u);
    // the workgroups' atomics on one address take 12 ns each: above some
    // hundreds of them a launch costs less
    const bool last = blocks <= 256;
    hipLaunchKernelGGL(k_commit_cells, dim3(blocks), dim3(256), 0, s, counts_new, offsets_new, counts, offsets,
                       g.ncells, sc, last ? 1 : 0, pc);
    if (!last) hipLaunchKernelGGL(k_epilogue, dim3(1), dim3(64), 0, s, sc, pc);
}

void launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s, const int32_t* gate) {
    unsigned blocks = grid1d(n, 256);
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill, dim3(blocks), dim3(256), 0, s, p, v, n, gate);
}

void launch_moments(const Geom& g, const int32_t* offsets, Planes p, const StepScalars* sc,
                    const VelCells& vcell, double* partial, double* out, hipStream_t s) {
    int blocks = (int)(g.ncells / g.Tc);
    if (g.vcodec) {
        hipLaunchKernelGGL(k_moments, dim3(blocks), dim3(256), (g.Tc + 1) * sizeof(int), s, g, offsets, p, sc, vcell,
                           partial);
    } else {
        // (the number of particles is a multiple of 64)
        blocks = (int)std::min<int64_t>(std::min(blocks, 1024), (int64_t)grid1d(g.n / 4, kMomentThreads));
        hipLaunchKernelGGL(k_moments_linear, dim3(blocks), dim3(kMomentThreads), 0, s, p, offsets + g.ncells, sc,
                           partial);
    }
    launch_reduce_partials(partial, blocks, 4, out, false, s);
}

void launch_reduce_partials(const double* partial, int nblocks, int width, double* out, bool add, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_partials, dim3(width), dim3(1024), 0, s, partial, nblocks, width, out, add ? 1 : 0);
}

void launch_power_bins(const float2* dk, int n, int nbins, double* partial, double* out, hipStream_t s) {
    const int width = 3 * nbins;
    hipLaunchKernelGGL(k_power_bins, dim3((nbins + kBinWaves - 1) / kBinWaves, n), dim3(kBinWaves * kWave), 0, s, dk, n,
                       nbins, partial);
    hipLaunchKernelGGL(k_sum_planes, dim3((width + kBinWaves - 1) / kBinWaves), dim3(kBinWaves * kWave), 0, s, partial,
                       n, width, out);
}

}  // namespace cube
