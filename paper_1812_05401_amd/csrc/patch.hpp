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
#pragma once

#include "strip.hpp"

namespace vplbm {

// Rows of partial sums per step: a wave's mass is in its own, forces go to row lane % kPatchSlots.  Waves meet
// there, in no fixed order: the last bits of a force may differ from run to run (populations do not).
constexpr int kPatchSlots = 16;

// LDS of a patch.  SUMS: with the observables' partial sums.
template <int S, int TW, int TH, int K, bool SUMS> struct PatchShared {
    using T = typename Codec<S>::real;
    static constexpr int EW = TW + 2 * (K - 1), EH = TH + 2 * (K - 1), EN = EW * EH;
    typename Codec<S>::elem mid[9 * EN];
    double part[SUMS ? K : 1][kPatchSlots][kRingWidth];
    T body[K][kMaxBodies][5];
    T record[K][EH][3];                                // convective outlet records, by region row
};

// nsteps (1 to K) steps of the patch of TW x TH nodes at (job.x0, job.y0), by a workgroup of THREADS.
// Returns whether an own node of this thread had a non-finite or non-positive density.
template <int S, int TW, int TH, int K, int THREADS, bool SUMS>
__device__ __forceinline__ bool patch_steps(const StripJob &job, int nsteps, PatchShared<S, TW, TH, K, SUMS> &sh)
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
    const Geom &g = job.g;
    const Rates<T> rates(job.p);
    const T out_u = uniform(T(job.out_u));
    const bool conv = job.out_prev != nullptr;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int x0 = job.x0, y0 = job.y0;
    const int skip = K - nsteps;                       // rings of the region that fewer steps do not need
    const E *__restrict__ src = static_cast<const E *>(job.src);
    E *__restrict__ dst = static_cast<E *>(job.dst);
    if (SUMS && job.reduce)
        for (int i = threadIdx.x; i < K * kPatchSlots * kRingWidth; i += THREADS) (&sh.part[0][0][0])[i] = 0.0;
    for (int i = threadIdx.x; i < nsteps * kMaxBodies; i += THREADS) {
        const BodyState &s = job.bodies[i / kMaxBodies * job.state_step + i % kMaxBodies];
        T *o = sh.body[i / kMaxBodies][i % kMaxBodies];
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
    const bool moves = job.mask_step != 0;
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
        id[r] = ring[r] >= skip ? job.mask[y[r] * g.pitch + x[r]] : 0u;
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
                    f[d] = Codec<S>::load(sh.mid + d * EN, unsigned((ey[r] - cy[d]) * EW + ex[r] - cx[d]), weight<T>(d));
            } else {
                const int ux = x0 + ex[r] - (K - 1), uy = y0 + ey[r] - (K - 1);
#pragma unroll
                for (int d = 0; d < 9; d++) {
                    const bool low = uy - cy[d] < 0 || uy - cy[d] >= g.ny, side = ux - cx[d] < 0 || ux - cx[d] >= g.nx;
                    const bool mirror = !g.yper && low;
                    const int px = !g.xper && side ? ex[r] : ex[r] - cx[d];
                    const int py = mirror ? ey[r] : ey[r] - cy[d];
                    f[d] = Codec<S>::load(sh.mid + (mirror ? mirror_y[d] : d) * EN, unsigned(py * EW + px), weight<T>(d));
                }
            }
            if (conv && x[r] == g.nx - 1) {
                // the outlet rule, with the values the step before recorded here
                T *next = static_cast<T *>(job.out_next);
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    const T prev = k == 0 ? static_cast<const T *>(job.out_prev)[q * g.ny + y[r]] : sh.record[k - 1][ey[r]][q];
                    f[odirs[q]] = outlet_value(prev, f[odirs[q]], out_u);
                    if (!last) sh.record[k][ey[r]][q] = f[odirs[q]];
                    else if (own[r]) next[q * g.ny + y[r]] = f[odirs[q]];
                }
            }
            if (g.inlet && x[r] == 0) inlet_west(f, rates.uin_x, rates.uin_y);
            if (moves && k > 0) id[r] = job.mask[k * job.mask_step + y[r] * g.pitch + x[r]];
            T drho;
            if (id[r]) {
                T usx, usy, fx, fy;
                body_velocity(sh.body[k][id[r] - 1], x[r], y[r], usx, usy);
                drho = relax_solid(f, true, usx, usy, rates, fx, fy);
                if (SUMS && job.reduce && own[r]) {
                    double *slot = sh.part[k][lane % kPatchSlots] + 2 * id[r];
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
            const unsigned hash = Codec<S>::stochastic ? mix32((job.step + unsigned(k)) * 0x9e3779b9u + 0x7f4a7c15u) : 0u;
            round_cols<S, 1>(res[r], 0, f, unsigned(y[r] * g.pitch + x[r]), hash, ~0ull);
        }
        if (SUMS && job.reduce) {
            const double m = wave_sum<wave_sum_dpp<T>()>(mass);
            if (lane == 0) sh.part[k][wave][0] = m;
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
                    for (int d = 0; d < 9; d++) res[r][d].put(sh.mid + d * EN, unsigned(ey[r] * EW + ex[r]));
                }
            __syncthreads();
        }
    }
    return bad;
}

}  // namespace vplbm
