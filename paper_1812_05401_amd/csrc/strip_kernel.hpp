// The strip sweep's kernel for a single simulation (see strip.hpp).
#pragma once

#include "reduce.hpp"
#include "strip.hpp"

namespace vplbm {

// W: waves per SIMD that the registers are allotted for.
template <int S, int C, int K, int W>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(W))) void strip_kernel(StepArgs a, const StripTile *strips)
{
    using T = typename Codec<S>::real;
    constexpr int V = strip_width<S, C, K>();
    __shared__ StripShared<T, K> shared;
    const int lane = threadIdx.x;
    const long long t = *a.t_base + a.t_off;
    if ((int)blockIdx.x >= work_blocks(a)) {
        fold_block(a, t, K);
        return;
    }
    const StripTile tile = strips[blockIdx.x];
    if (tile.y1 <= tile.y0) return;                    // an empty entry (uniform)
    if (a.reduce) {
        // a plain strip sums no force, and its mass goes to the first slot
        const int rows = tile.form == kPlain ? 1 : kForceSlots;
        for (int k = 0; k < K; k++)
            for (int q = lane; q < rows * kRingWidth; q += 64) (&shared.part[k][0][0])[q] = 0.0;
    }
    const StripJob job{a.src, a.dst, a.mask, a.mask_step, a.bodies, a.state_step, a.g, a.p, a.outlet.prev, a.outlet.next,
                       a.outlet.u, tile.x0, tile.y0, tile.y1, a.reduce != 0, (unsigned)t};
    double mass[K];
#pragma unroll
    for (int k = 0; k < K; k++) mass[k] = 0.0;
    bool bad;
    if (tile.form == kPlain) bad = strip_sweep<S, C, K, false>(job, mass, shared);
    else bad = strip_sweep<S, C, K, true>(job, mass, shared);
    if (a.reduce) {
        const int w = a.g.nx - job.x0 < V ? a.g.nx - job.x0 : V;
        const double nodes = double(w) * double(job.y1 - job.y0);
#pragma unroll
        for (int k = 0; k < K; k++) {
            const double m = wave_sum<wave_sum_dpp<T>()>(mass[k]);
            if (lane == 0) shared.part[k][0][0] = nodes + m;
        }
        if (__ballot(bad) && lane == 0) atomicOr(a.status, 1u);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; k++) add_partials(a, t + k, &shared.part[k][0][0], tile.form == kPlain ? 1 : kForceSlots);
    }
}

template <int S, int C, int K, int W> void strip_launch(const StepArgs &a, const StripTile *strips, int n, hipStream_t st)
{
    strip_kernel<S, C, K, W><<<dim3(all_blocks(a, n)), dim3(64), 0, st>>>(a, strips);
}

template <int S, int C, int K, int W> hipError_t strip_load()
{
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(&strip_kernel<S, C, K, W>));
}

template <int S, int C, int K, int W> constexpr StripShape strip_form(int rows = 36)
{
    return {C, K, W, strip_width<S, C, K>(), strip_halo<S, C, K>(), rows, &strip_launch<S, C, K, W>, &strip_load<S, C, K, W>};
}

}  // namespace vplbm
