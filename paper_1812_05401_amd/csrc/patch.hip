// The patch kernel for a single simulation (see patch.hpp).
#include "patch.hpp"
#include "reduce.hpp"

namespace vplbm {

template <int S, int TW, int TH, int K, int THREADS>
__global__ __launch_bounds__(THREADS) void patch_kernel(StepArgs a, int nsteps)
{
    __shared__ PatchShared<S, TW, TH, K, true> sh;
    const long long t = *a.t_base + a.t_off;
    if ((int)blockIdx.x >= work_blocks(a)) {
        fold_block(a, t, nsteps);
        return;
    }
    const int ntx = (a.g.nx + TW - 1) / TW;
    const int tile = xcd_tile(blockIdx.x, work_blocks(a));
    const int x0 = (tile % ntx) * TW, y0 = (tile / ntx) * TH;
    const StripJob job{a.src, a.dst, a.mask, a.mask_step, a.bodies, a.state_step, a.g, a.p, a.outlet.prev, a.outlet.next,
                       a.outlet.u, x0, y0, y0 + TH, a.reduce != 0, (unsigned)t};
    const bool bad = patch_steps<S, TW, TH, K, THREADS, true>(job, nsteps, sh);
    if (a.reduce) {
        if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(a.status, 1u);
        __syncthreads();
        for (int i = threadIdx.x; i < nsteps * kRingWidth; i += THREADS) {
            const int k = i / kRingWidth, q = i % kRingWidth;
            double v = 0.0;
#pragma unroll
            for (int w = 0; w < kPatchSlots; w++) v += sh.part[k][w][q];
            if (v != 0.0) unsafeAtomicAdd(acc_set(a, t + k) + (blockIdx.x & (kSub - 1)) * kRingWidth + q, v);
        }
    }
}

template <int S, int TW, int TH, int K, int THREADS> struct Patch {
    static void launch(const StepArgs &a, int nsteps, hipStream_t st)
    {
        const int tiles = ((a.g.nx + TW - 1) / TW) * ((a.g.ny + TH - 1) / TH);
        patch_kernel<S, TW, TH, K, THREADS><<<dim3(all_blocks(a, tiles)), dim3(THREADS), 0, st>>>(a, nsteps);
    }
    static_assert(K <= kMaxSteps, "reduction sets");
    static constexpr PatchShape shape{K, launch};
};

// The first two keep the grid within about one workgroup per CU (256) with the most steps the halo can
// pay for; 24 x 16 carries that to 98,304 nodes.  Above, every CU has several workgroups and the halo's
// work counts: 16 x 16 and four steps while two of its workgroups share a CU, then a larger patch
// (of FP32 arithmetic, FP64 values of that size would leave one workgroup per CU; they take one of
// three steps).  us per step, this form and the one to either side:
//   160 x 160   f32 1.89 (8 x 8: 1.89)                           f64 2.84 (8 x 8: 2.89)
//   300 x 300   f32 2.15 (16 x 16, six: 3.28; four: 2.67)        f64 3.30 (5.06; 3.98)
//   256 x 512   f32 2.72 (24 x 16: 3.12; 26 x 18: 2.97)          f64 3.98 (5.41; 20 x 17: 4.29)
//   512 x 400   f32 3.06 (16 x 16: 3.95; 24 x 16: 3.52)          f64 5.90 (16 x 16: 5.96; 26 x 18: 5.99)
//   768 x 640   f32 5.62 (16 x 16: 7.03; 28 x 20, three: 5.70)   f64 9.83 (10.57; 11.78)
template <int S> static const PatchShape *patch_forms(long long nodes)
{
    constexpr bool narrow = sizeof(typename Codec<S>::real) == 4;
    if (nodes <= 24000) return &Patch<S, 8, 8, 8, 512>::shape;
    if (nodes <= 256 * 256) return &Patch<S, 16, 16, 6, 704>::shape;
    if (nodes <= 256 * 384) return &Patch<S, 24, 16, 5, 768>::shape;
    if (nodes <= 150000) return &Patch<S, 16, 16, 4, 512>::shape;
    return &Patch<S, narrow ? 26 : 20, narrow ? 18 : 17, narrow ? 4 : 3, narrow ? 768 : 512>::shape;
}

// The largest lattice that patches still win: the two- and three-step kernels (which f32 leaves to the
// strip sweep) fill the chip at 0.7 million nodes.  us per step, patches and those kernels:
//   1000 x 601   f32 6.60, 7.65   f64 12.11, 12.75   f32d 10.89, 11.36   f16 9.29, 10.73   f16s 6.80, 8.16
//   1024 x 768   f32 7.80, 8.61   f64 14.98, 14.42   f32d 13.38, 12.68   f16 11.10, 10.89  f16s 8.17, 8.28
const PatchShape *patch_shape(int storage, long long nodes, long long most)
{
    if (most < 0) most = storage == kF32 ? 799999 : 650000;
    if (nodes > most) return nullptr;
    switch (storage) {
    case kF64: return patch_forms<kF64>(nodes);
    case kF32: return patch_forms<kF32>(nodes);
    case kF32D: return patch_forms<kF32D>(nodes);
    case kF16S: return patch_forms<kF16S>(nodes);
    case kBF16S: return patch_forms<kBF16S>(nodes);
    case kF16SR: return patch_forms<kF16SR>(nodes);
    case kBF16SR: return patch_forms<kBF16SR>(nodes);
    }
    return nullptr;
}

}  // namespace vplbm
