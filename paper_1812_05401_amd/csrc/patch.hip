// Several steps of a small lattice per launch: patches in LDS.
//
// Below about half a million nodes a launch is not bound by arithmetic or memory but by its own
// latency: on 128 x 128 nodes the two-step kernel takes 11 us, on 32 of 256 CUs.  So a patch is made
// small enough that every CU has one, and the idle arithmetic goes into a wide halo: a workgroup loads
// its patch with K - 1 nodes around it once and takes all the steps in LDS, each on one ring of nodes
// less, the last on the patch's own nodes, which are stored.  A step reads its pulls, then (barrier)
// overwrites the same slots.  A thread has the same few nodes throughout, so coordinates, ids and edge
// tests are made once.  f32, 128 x 128: 5.55 -> 1.54 us per step; f64 5.43 -> 2.20.
//
// Values in LDS are rounded as a store to global memory would round them, and the node update is
// node.hpp's: the populations are bitwise those of one-step launches.
#include "reduce.hpp"
#include "strip.hpp"

namespace vplbm {

constexpr int kPatchSlots = 16;   // rows of partial sums per step

template <int S, int TW, int TH, int K, int THREADS>
__global__ __launch_bounds__(THREADS) void patch_kernel(StepArgs a, int nsteps)
{
    using P = Cols<S, 1>;
    using E = typename Codec<S>::elem;
    using T = typename Codec<S>::real;
    constexpr int EW = TW + 2 * (K - 1), EH = TH + 2 * (K - 1), EN = EW * EH;
    constexpr int R = (EN + THREADS - 1) / THREADS;
    constexpr int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    constexpr int cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    constexpr int mirror_y[9] = {0, 1, 4, 3, 2, 8, 7, 6, 5};
    constexpr int odirs[3] = {3, 6, 7};                // the directions entering from x = nx
    static_assert(THREADS / 64 <= kPatchSlots, "a row of partials per wave");
    __shared__ E mid[9 * EN];
    __shared__ double part[K][kPatchSlots][kRingWidth];
    __shared__ T body[K][kMaxBodies][5];
    __shared__ T record[K][EH][3];                     // convective outlet records, by region row
    const Geom &g = a.g;
    const long long t = *a.t_base + a.t_off;
    if ((int)blockIdx.x >= work_blocks(a)) {
        fold_block(a, t, nsteps);
        return;
    }
    const Rates<T> rates(a.p);
    const T out_u = uniform(T(a.outlet.u));
    const bool conv = a.outlet.prev != nullptr;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ntx = (g.nx + TW - 1) / TW;
    const int tile = xcd_tile(blockIdx.x, work_blocks(a));
    const int x0 = (tile % ntx) * TW, y0 = (tile / ntx) * TH;
    const int skip = K - nsteps;                       // rings of the region that fewer steps do not need
    const E *__restrict__ src = static_cast<const E *>(a.src);
    E *__restrict__ dst = static_cast<E *>(a.dst);
    if (a.reduce)
        for (int i = threadIdx.x; i < K * kPatchSlots * kRingWidth; i += THREADS) (&part[0][0][0])[i] = 0.0;
    for (int i = threadIdx.x; i < nsteps * kMaxBodies; i += THREADS) {
        const BodyState &s = a.bodies[i / kMaxBodies * a.state_step + i % kMaxBodies];
        T *o = body[i / kMaxBodies][i % kMaxBodies];
        o[0] = T(s.cx);
        o[1] = T(s.cy);
        o[2] = T(s.vx);
        o[3] = T(s.vy);
        o[4] = T(s.omega);
    }
    // This thread's nodes: region position, lattice node, the ring they lie on (a step takes the rings
    // from its own on; the patch's own nodes are ring K - 1 and further in).
    int ex[R], ey[R], x[R], y[R], ring[R];
    bool own[R], plain[R];
    unsigned id[R];
    const bool moves = a.mask_step != 0;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int e = threadIdx.x + r * THREADS;
        ex[r] = e % EW;
        ey[r] = e / EW;
        const int ux = x0 + ex[r] - (K - 1), uy = y0 + ey[r] - (K - 1);
        x[r] = ux;
        y[r] = uy;
        bool live = e < EN;
        if (g.xper) {
            x[r] %= g.nx;
            if (x[r] < 0) x[r] += g.nx;
        } else {
            live &= ux >= 0 && ux < g.nx;
        }
        if (g.yper) {
            y[r] %= g.ny;
            if (y[r] < 0) y[r] += g.ny;
        } else {
            live &= uy >= 0 && uy < g.ny;
        }
        const int h = ex[r] < EW - 1 - ex[r] ? ex[r] : EW - 1 - ex[r], v = ey[r] < EH - 1 - ey[r] ? ey[r] : EH - 1 - ey[r];
        ring[r] = live ? (h < v ? h : v) : -1;
        own[r] = ring[r] >= K - 1 && ux < g.nx && uy < g.ny;
        plain[r] = (g.xper || (x[r] > 0 && x[r] < g.nx - 1)) && (g.yper || (y[r] > 0 && y[r] < g.ny - 1));
        id[r] = ring[r] >= skip ? a.mask[y[r] * g.pitch + x[r]] : 0u;
    }
    bool bad = false;
    __syncthreads();                                   // the tables are complete
    for (int k = 0; k < nsteps; k++) {
        const bool last = k == nsteps - 1;
        P res[R][9];
        double mass = 0.0;
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (ring[r] < skip + k) continue;
            T f[9];
            if (k == 0) {
                pull<S>(src, x[r], y[r], g, Outlet{nullptr, nullptr, 0.0}, f);
            } else if (plain[r]) {
#pragma unroll
                for (int d = 0; d < 9; d++)
                    f[d] = Codec<S>::load(mid + d * EN, unsigned((ey[r] - cy[d]) * EW + ex[r] - cx[d]), weight<T>(d));
            } else {
                const int ux = x0 + ex[r] - (K - 1), uy = y0 + ey[r] - (K - 1);
#pragma unroll
                for (int d = 0; d < 9; d++) {
                    const bool low = uy - cy[d] < 0 || uy - cy[d] >= g.ny, side = ux - cx[d] < 0 || ux - cx[d] >= g.nx;
                    const bool mirror = !g.yper && low;
                    const int px = !g.xper && side ? ex[r] : ex[r] - cx[d];
                    const int py = mirror ? ey[r] : ey[r] - cy[d];
                    f[d] = Codec<S>::load(mid + (mirror ? mirror_y[d] : d) * EN, unsigned(py * EW + px), weight<T>(d));
                }
            }
            if (conv && x[r] == g.nx - 1) {
                // the outlet rule, with the values the step before recorded here
                T *next = static_cast<T *>(a.outlet.next);
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    const T prev = k == 0 ? static_cast<const T *>(a.outlet.prev)[q * g.ny + y[r]] : record[k - 1][ey[r]][q];
                    f[odirs[q]] = outlet_value(prev, f[odirs[q]], out_u);
                    if (!last) record[k][ey[r]][q] = f[odirs[q]];
                    else if (own[r]) next[q * g.ny + y[r]] = f[odirs[q]];
                }
            }
            if (g.inlet && x[r] == 0) inlet_west(f, rates.uin_x, rates.uin_y);
            if (moves && k > 0) id[r] = a.mask[k * a.mask_step + y[r] * g.pitch + x[r]];
            T drho;
            if (id[r]) {
                T usx, usy, fx, fy;
                body_velocity(body[k][id[r] - 1], x[r], y[r], usx, usy);
                drho = relax_solid(f, true, usx, usy, rates, fx, fy);
                if (a.reduce && own[r]) {
                    double *slot = part[k][lane % kPatchSlots] + 2 * id[r];
                    unsafeAtomicAdd(slot - 1, -double(fx));
                    unsafeAtomicAdd(slot, -double(fy));
                }
            } else {
                drho = relax_fluid(f, rates);
            }
            if (own[r]) {
                const double rho = 1.0 + double(drho);
                mass += rho;
                bad |= !(rho > 0.0 && rho < 1e30);
            }
            const unsigned hash = Codec<S>::stochastic ? mix32(unsigned(t + k) * 0x9e3779b9u + 0x7f4a7c15u) : 0u;
            round_cols<S, 1>(res[r], 0, f, unsigned(y[r] * g.pitch + x[r]), hash, ~0ull);
        }
        if (a.reduce) {
            const double m = wave_sum<wave_sum_dpp<T>()>(mass);
            if (lane == 0) part[k][wave][0] = m;
        }
        if (last) {
#pragma unroll
            for (int r = 0; r < R; r++)
                if (own[r]) {
#pragma unroll
                    for (int d = 0; d < 9; d++) res[r][d].put(dst + d * g.plane, unsigned(y[r] * g.pitch + x[r]));
                }
        } else {
            __syncthreads();                           // every pull has read the step before
#pragma unroll
            for (int r = 0; r < R; r++)
                if (ring[r] >= skip + k) {
#pragma unroll
                    for (int d = 0; d < 9; d++) res[r][d].put(mid + d * EN, unsigned(ey[r] * EW + ex[r]));
                }
            __syncthreads();
        }
    }
    if (a.reduce) {
        if (__ballot(bad) && lane == 0) atomicOr(a.status, 1u);
        __syncthreads();
        for (int i = threadIdx.x; i < nsteps * kRingWidth; i += THREADS) {
            const int k = i / kRingWidth, q = i % kRingWidth;
            double v = 0.0;
#pragma unroll
            for (int w = 0; w < kPatchSlots; w++) v += part[k][w][q];
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
