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

// The largest lattice that patches still win (a long run): the two- and three-step kernels (which f32 leaves
// to the strip sweep) fill the chip at 0.7 million nodes, with FP64 arithmetic before that, and stochastic
// rounding makes the halo's nodes dear, in f16 most.  us per step, patches and those kernels:
//   640 x 470    f32 4.08, 5.58  f64 6.96, 7.52    f32d 6.06, 6.46    f16 7.10, 7.67   bf16 4.68, 6.35
//   800 x 500    f32 4.82, 5.57  f64 8.71, 9.12    f32d 7.46, 7.78    f16 8.25, 7.67   bf16 5.65, 6.43
//   768 x 640    f32 5.62, 6.31  f64 9.90, 10.14   f32d 8.97, 8.91    f16 9.75, 7.84   bf16 6.56, 6.56
//   840 x 715    f32 6.55, 6.68  f64 11.72, 11.43  f32d 10.56, 10.04  f16s 6.72, 7.54  bf16 7.71, 8.34
const PatchShape *patch_shape(int storage, long long nodes, long long most)
{
    if (most < 0) most = storage == kF32 ? 799999 : storage == kF64 ? 550000 : storage == kF32D ? 450000 : storage == kF16SR ? 350000 : 650000;
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

// What remains of a call takes the one- and two-step kernels where those are faster: a patch loads and
// computes its halo for any number of steps.  us per launch of one step, patches and tiles:
//   200 x 200    f32 6.71, 7.23   f64 7.68, 8.45    f16 7.20, 7.38
//   256 x 256    f32 8.80, 7.37   f64 9.92, 8.74    f16 9.08, 7.41
//   768 x 640    f32 13.8, 10.3   f64 20.0, 16.5    bf16 14.0, 10.1
// and of two (of three, patches are faster or within 2%):
//   320 x 192    f32 9.4, 12.6    f64 10.9, 11.6   f32d 10.3, 10.9   f16 10.1, 14.6   bf16 9.8, 13.0
//   384 x 256    f32 8.6, 13.5    f64 12.3, 12.0   f32d 11.4, 11.2   f16 10.9, 15.8   bf16 8.9, 14.1
//   512 x 400    f32 10.7, 14.2   f64 15.9, 14.6   f32d 13.9, 13.3   f16 15.2, 16.2   bf16 11.5, 14.5
//   640 x 470    f32 13.4, 14.3   f64 18.7, 17.6   f32d 16.5, 15.3   f16 19.7, 17.7   bf16 14.3, 15.0
//   800 x 500    f32 15.6, 15.2   f64 22.8, 20.3   f32d 19.5, 17.8   f16s 16.0, 14.0  bf16 17.3, 15.0
int patch_least(int storage, long long nodes)
{
    const long long two = storage == kF64 || storage == kF32D ? 90000 : storage == kF16SR ? 250000 : 350000;
    return nodes > two ? 3 : nodes > 50000 ? 2 : 1;
}

}  // namespace vplbm
