// The strip sweep's kernels for the serving pool's simulations (see strip.hpp).
#pragma once

#include "pool_job.hpp"

namespace vplbm {

// A strip, or one of its blocks where the simulation ends (final_step), for KK <= K steps.
template <int S, int K, int KK>
__device__ __forceinline__ void pool_strip(const StripJob &job, int form, PoolSim *sim, int block, bool final_step,
                                           StripLastShared<typename Codec<S>::real, K> &shared)
{
    using T = typename Codec<S>::real;
    constexpr int V = strip_width<S, 1, K>();
    const int lane = threadIdx.x;
    for (int i = lane; i < 64 * kRingWidth; i += 64) (&shared.part[0][0])[i] = 0.0;
    double mass[KK];
#pragma unroll
    for (int k = 0; k < KK; k++) mass[k] = 0.0;
    bool bad;
    if (form == kPlain) bad = strip_sweep<S, 1, KK, false, K>(job, mass, shared);
    else bad = strip_sweep<S, 1, KK, true, K>(job, mass, shared);
    if (__ballot(bad) && lane == 0) atomicOr(&sim->status, 1u);
    if (final_step) {
        const int w = job.g.nx - job.x0 < V ? job.g.nx - job.x0 : V;
        const double m = wave_sum<wave_sum_dpp<T>()>(mass[KK - 1]);
        if (lane == 0) shared.part[0][0] = double(w) * double(job.y1 - job.y0) + m;
        __syncthreads();
        if (lane < sim->width) {
            double v = 0.0;
            for (int q = 0; q < 64; q++) v += shared.part[q][lane];   // fixed order
            sim->partials[(size_t)block * sim->width + lane] = v;
        }
        __syncthreads();
    }
}

// K steps of every resident simulation of one format, a strip per wave.
// W: waves per SIMD that the registers are allotted for.
template <int S, int K, int W>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(W))) void pool_strip_kernel(PoolLaunch a)
{
    using T = typename Codec<S>::real;
    __shared__ StripShared<T, K> shared;
    const int n = *a.ntiles;
    const TileRef tr = a.tiles[blockIdx.x];                   // the table spans the grid
    if ((int)blockIdx.x >= n) return;
    PoolSim *sim = a.sims + tr.slot;
    const long long start = *a.t_base - sim->t0, left = sim->target - start;
    if (!sim->active || start < 0 || left <= 0 || a.t_off >= pool_body(*sim, left)) return;
    const StripJob job = pool_job(sim, (pool_buf(*sim, start) + a.t_off / K) & 1, start + a.t_off, tr.x0, tr.y0, tr.y1);
    double mass[K];
#pragma unroll
    for (int k = 0; k < K; k++) mass[k] = 0.0;
    bool bad;
    if (tr.form == kPlain) bad = strip_sweep<S, 1, K, false, K, false>(job, mass, shared);
    else bad = strip_sweep<S, 1, K, true, K, false>(job, mass, shared);
    if (__ballot(bad) && threadIdx.x == 0) atomicOr(&sim->status, 1u);
}

// The end of a replay: the steps that the main launches (these strips' or patches') leave.  Simulations
// that end go block by block, and each block's FP64 sums go to its place in the partials.  (A kernel of
// its own: in the one above, the loop and the cases would cost 38 registers' spills on every launch.)
template <int S, int K, int W>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(W))) void pool_strip_tail_kernel(PoolLaunch a)
{
    using T = typename Codec<S>::real;
    __shared__ StripLastShared<T, K> shared;
    const int n = *a.ntiles;
    const TileRef tr = a.tiles[blockIdx.x];
    if ((int)blockIdx.x >= n) return;
    PoolSim *sim = a.sims + tr.slot;
    const long long start = *a.t_base - sim->t0, left = sim->target - start;
    if (!sim->active || start < 0 || left <= 0) return;
    const bool final_step = left <= sim->spl;
    const int body = pool_body(*sim, left), k = int(final_step ? left : sim->spl) - body;
    if (k == 0) return;
    const int buf = (pool_buf(*sim, start) + (body + sim->spk - 1) / sim->spk) & 1;
    const int rows = final_step ? pool_block_rows(tr.form) : tr.y1 - tr.y0;
    static_assert(K >= 3 && K <= 5, "the cases below");
    for (int y0 = tr.y0, block = tr.tile; y0 < tr.y1; y0 += rows, block++) {
        const StripJob job = pool_job(sim, buf, start + body, tr.x0, y0, y0 + rows < tr.y1 ? y0 + rows : tr.y1);
        if (k == 1) pool_strip<S, K, 1>(job, tr.form, sim, block, final_step, shared);
        else if (k == 2) pool_strip<S, K, 2>(job, tr.form, sim, block, final_step, shared);
        else if (k == 3) pool_strip<S, K, 3>(job, tr.form, sim, block, final_step, shared);
        else if constexpr (K >= 4) {
            if (k == 4) pool_strip<S, K, 4>(job, tr.form, sim, block, final_step, shared);
            else if constexpr (K >= 5) pool_strip<S, K, 5>(job, tr.form, sim, block, final_step, shared);
        }
    }
}

// The main launches of one replay of `steps` steps (a.t_off is set here).
template <int S, int K, int W> hipError_t pool_strip_launch(PoolLaunch a, int steps, int grid, hipStream_t st)
{
    for (a.t_off = 0; a.t_off + K <= steps; a.t_off += K) {
        pool_strip_kernel<S, K, W><<<dim3(grid), dim3(64), 0, st>>>(a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <int S, int K, int W> hipError_t pool_strip_tail(PoolLaunch a, int grid, hipStream_t st)
{
    pool_strip_tail_kernel<S, K, W><<<dim3(grid), dim3(64), 0, st>>>(a);
    return hipGetLastError();
}

template <int S, int K, int W> constexpr PoolStrips pool_strips_form()
{
    return {K, strip_width<S, 1, K>(), strip_halo<S, 1, K>(), W, &pool_strip_launch<S, K, W>, &pool_strip_tail<S, K, W>};
}

}  // namespace vplbm
