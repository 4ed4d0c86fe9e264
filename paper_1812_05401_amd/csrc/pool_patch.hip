// Patches in LDS (see patch.hpp) over the serving pool's simulations, where few nodes are resident.
#include "patch.hpp"
#include "pool_job.hpp"

namespace vplbm {

template <int S, int TW, int TH, int K, int THREADS> __global__ __launch_bounds__(THREADS) void pool_patch_kernel(PoolLaunch a)
{
    __shared__ PatchShared<S, TW, TH, K, false> sh;
    const int n = *a.ntiles;
    const TileRef tr = a.tiles[blockIdx.x];                   // the table spans the grid
    if ((int)blockIdx.x >= n) return;                         // uniform over the workgroup
    PoolSim *sim = a.sims + tr.slot;
    const long long start = *a.t_base - sim->t0, left = sim->target - start;
    if (!sim->active || start < 0 || left <= 0) return;
    const int body = pool_body(*sim, left);
    if (a.t_off >= body) return;
    const StripJob job = pool_job(sim, (pool_buf(*sim, start) + a.t_off / K) & 1, start + a.t_off, tr.x0, tr.y0, tr.y1);
    const bool bad = patch_steps<S, TW, TH, K, THREADS, false>(job, body - a.t_off < K ? body - a.t_off : K, sh);
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(&sim->status, 1u);
}

template <int S, int TW, int TH, int K, int THREADS> struct Patches {
    // the main launches of one replay of `steps` steps (a.t_off is set here)
    static hipError_t launch(PoolLaunch a, int steps, int grid, hipStream_t st)
    {
        for (a.t_off = 0; a.t_off < steps; a.t_off += K) {
            pool_patch_kernel<S, TW, TH, K, THREADS><<<dim3(grid), dim3(THREADS), 0, st>>>(a);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    static constexpr PoolPatches form{K, TW, TH, launch};
};

// Two of the forms of patch.hip, for the same reasons: 24 x 16 while it leaves every CU at most one
// workgroup, larger above.
template <int S> static const PoolPatches &patches_of(int kernel)
{
    constexpr bool narrow = sizeof(typename Codec<S>::real) == 4;
    if (kernel >= kPoolSmall) return Patches<S, 24, 16, 5, 768>::form;
    return Patches<S, narrow ? 26 : 20, narrow ? 18 : 17, narrow ? 4 : 3, narrow ? 768 : 512>::form;
}

const PoolPatches &pool_patches(int kernel)
{
    switch (pool_storage(kernel)) {
    case kF64: return patches_of<kF64>(kernel);
    case kF32: return patches_of<kF32>(kernel);
    case kF32D: return patches_of<kF32D>(kernel);
    case kF16S: return patches_of<kF16S>(kernel);
    case kBF16S: return patches_of<kBF16S>(kernel);
    case kF16SR: return patches_of<kF16SR>(kernel);
    default: return patches_of<kBF16SR>(kernel);
    }
}

// Patches while few nodes are resident.  us per step at 0.64 and 1.28 million nodes (800 x 800, one and two),
// patches and strips: f32 5.9, 10.4 and 8.1, 10.4; f64 11.2, 19.5 and 11.8, 16.5; f32d 9.4, 16.5 and 10.1, 12.9;
// f16s 6.1, 11.0 and 7.9, 10.8; bf16s 6.2, 11.5 and 8.5, 11.8; bf16sr 6.9, 12.2 and 9.2, 11.7.  (On one lattice of
// 96 x 96: f32 2.1, two- or three-step tiles 5.3, strips 7.5; f64 2.9, 4.7 and 9.8.)  f16sr takes
// tiles between the two: at 0.4, 0.48, 2.6 and 5.1 million nodes patches 8.3, 9.3, 39, 76, tiles 9.3, 8.9, 28.2, 53,
// strips 13.2, 12.0, 29.1, 48.9.
int pool_choose(int storage, long long nodes)
{
    long long most = 0, tiles = 0;
    switch (storage) {
    case kF64: most = 800000; break;
    case kF32: most = 1200000; break;
    case kF32D: most = 680000; break;
    case kF16S: most = 1100000; break;
    case kBF16S: most = 1250000; break;
    case kF16SR: most = 420000; tiles = 3800000; break;
    case kBF16SR: most = 950000; break;
    }
    if (nodes <= most) return storage + (nodes <= 256 * 384 ? kPoolSmall : kPoolPatches);
    return nodes <= tiles ? kPoolTiles32 : kPoolStrips + storage;
}

// A strip that takes one step of its three to five still has a window and rows for all of them.  us per
// replay of one and two steps, 14 simulations of 800 x 800, strips and two-step tiles: f32 256, 262 and 180,
// 226 (three: 265 in strips); f64 379, 388 and 298, 375, but of four simulations two steps 130 and 138; f32d
// 257, 271 and 216, 302; f16s 151, 159 and 161, 216; bf16sr 147, 166 and 164, 231; f16sr 150, 179 and 167, 239.
int pool_least(int storage) { return storage == kF32 ? 3 : storage == kF64 || storage == kF32D ? 2 : 1; }

}  // namespace vplbm
