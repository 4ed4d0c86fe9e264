// Per-step reductions (mass and body forces) of the single-simulation step kernels: where a launch
// adds its partial sums, and how a later one folds them into the ring.
#pragma once

#include "kernels.hpp"

namespace vplbm {

// Sub-slots [kSub][kRingWidth] of step t: one of kAccSets sets, used round-robin by step.
__device__ __forceinline__ double *acc_set(const StepArgs &a, long long t)
{
    return a.acc + (size_t)(t & (kAccSets - 1)) * kSub * kRingWidth;
}

// Sum value q of the sub-slots of steps t - kMaxSteps .. t - 1 (those that exist) into their ring
// entries, with one wave, or the steps spread over WAVES of them: lane l adds sub-slots l, l + 64, ... in
// order, then a fixed butterfly adds the lanes, so a result does not depend on which workgroup folds or
// when.  One memory round trip for all of them.  Nothing is cleared, so folding a step again gives the same value: a step
// is folded by the next launch, and again by later ones while it is among their last kMaxSteps.
// The fold always takes the shuffle form of the wave sum, so that every fold of a step (by any
// kernel class, or by an observation) writes the same value.
template <int WAVES = 1> __device__ __forceinline__ void fold_recent(const StepArgs &a, long long t, int q)
{
    constexpr int N = kMaxSteps / WAVES;
    static_assert(N * WAVES == kMaxSteps, "as many steps for every wave");
    const int lane = threadIdx.x & 63, first = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * N;
    double v[N];
#pragma unroll
    for (int d = 0; d < N; d++) v[d] = 0.0;
    for (int b = lane; b < kSub; b += 64) {
#pragma unroll
        for (int d = 0; d < N; d++) v[d] += acc_set(a, t - 1 - (first + d))[b * kRingWidth + q];
    }
#pragma unroll
    for (int i = 0; i < N; i++) {
        const int d = first + i;
        const double sum = wave_sum<false>(v[i]);
        if (lane == 0 && t >= 1 + d && d < a.ring_len) a.ring[(size_t)((t - 1 - d) % a.ring_len) * kRingWidth + q] = sum;
    }
}

// Strips and patches: workgroups of a launch that only do its share of the reductions, after those that compute: they run
// beside them, so no tile waits for a fold.  (In the tiles' own workgroups the fold's two memory round
// trips were a tenth of a launch on a 128 x 128 lattice.)
constexpr int kFoldBlocks = kRingWidth;

// The number of computing workgroups of this launch.
__device__ __forceinline__ int work_blocks(const StepArgs &a) { return int(gridDim.x) - (a.reduce ? kFoldBlocks : 0); }
inline int all_blocks(const StepArgs &a, int work) { return work + (a.reduce ? kFoldBlocks : 0); }

// Workgroup work_blocks + q of a launch that computes steps t .. t + n - 1 (1 <= n <= kMaxSteps): its
// first wave folds value q of steps t - kMaxSteps .. t - 1, and it zeroes sub-slots q, q + kFoldBlocks,
// ... of the sets of steps t + n .. t + n + kMaxSteps - 1, which the next launch accumulates into.  The
// sets one launch folds, writes and clears span at most 3 kMaxSteps consecutive steps, so with
// kAccSets >= 3 kMaxSteps they are distinct.  Step s is first folded by a launch starting at most
// kMaxSteps steps after s; the launch that clears its set for step s + kAccSets starts at least
// kAccSets - 2 kMaxSteps + 1 steps after s, later in stream order, so every fold of s sees its
// complete sums.
__device__ __forceinline__ void fold_block(const StepArgs &a, long long t, int n)
{
    const int q = int(blockIdx.x) - work_blocks(a);
    if (threadIdx.x < 64) fold_recent(a, t, q);
    for (int i = threadIdx.x; i < kMaxSteps * kRingWidth; i += blockDim.x) {
        double *set = acc_set(a, t + n + i / kRingWidth);
        for (int b = q; b < kSub; b += kFoldBlocks) set[b * kRingWidth + i % kRingWidth] = 0.0;
    }
}

// The same in the first workgroups of a tiled kernel, before their tiles (the fold on all of their WAVES
// waves).  Workgroups of its own are better for small lattices, but those take patches; and with that
// branch the FP64 kernels take 85 and 114 VGPRs, not 79 and 92, which is one wave per SIMD less.  us per
// launch of one and two steps at 4096 x 1024, with the branch and here: f64 117.7, 140.6 and 112.9, 129.1;
// f32d 90.2, 110.2 and 73.1, 94.2.
template <int WAVES> __device__ __forceinline__ void reduction_prologue(const StepArgs &a, long long t, int n)
{
    for (int q = blockIdx.x; q < kRingWidth; q += gridDim.x) fold_recent<WAVES>(a, t, q);
    if (threadIdx.x < kMaxSteps * kRingWidth) {
        double *set = acc_set(a, t + n + threadIdx.x / kRingWidth);
        const int q = threadIdx.x % kRingWidth;
        for (int b = blockIdx.x; b < kSub; b += gridDim.x) set[b * kRingWidth + q] = 0.0;
    }
}

// A workgroup's partial sums of step t (rows of per-wave partials, added in a fixed order) into
// its sub-slot of the step's set: threads 0 .. kRingWidth - 1, after the barrier that completes
// the rows.
__device__ __forceinline__ void add_partials(const StepArgs &a, long long t, const double *rows, int nrows)
{
    if (threadIdx.x < kRingWidth) {
        double v = 0.0;
        for (int w = 0; w < nrows; w++) v += rows[w * kRingWidth + threadIdx.x];   // fixed order
        double *slot = acc_set(a, t) + (blockIdx.x & (kSub - 1)) * kRingWidth;
        if (v != 0.0) unsafeAtomicAdd(slot + threadIdx.x, v);
    }
}

}  // namespace vplbm
