// Serving pool: many resident VP-LBM simulations advanced together by a batched step kernel
// replayed from a captured HIP graph (see the pool section of include/vplbm.h).
//
// Device side.  A descriptor per slot (buffers, geometry, parameters, admission step, target) and for
// every kernel a table that covers the resident simulations it advances, one entry per workgroup.  While
// few nodes are resident these are patches in LDS (patch.hpp), three to five steps per launch, then the
// strip sweep (strip.hpp), three to five steps too: see pool_choose.  f16sr between the two, and lattices
// of very few rows or of planes beyond 4 GB, take two steps per launch on 64 x 8 tiles, the first kept
// in LDS as in the two-step kernel.  All run the same per-node update as the single-simulation step, so
// a simulation's fields do not depend on its co-residents or on the launch shape, and the kernel may
// change at any replay boundary.  All resident simulations advance together, so a simulation's steps
// done are the pool's step counter (on the device) minus its admission step: no per-step bookkeeping
// launch is needed.  Whatever took the steps before, a simulation's last steps are taken by strips, block
// by block (of those that have no strips, by tiles), and each block writes its FP64 partial sums of the
// final step (mass, body forces) to its own place, summed in a fixed order; at retirement a fold kernel
// adds them in order, so the final observables are bitwise independent of the mix.
//
// Early stop: for simulations that ask for it, the graph ends with a residual check (a kernel per entry
// and a per-slot fold) that lowers the simulation's target on the device once its
// velocity change is below the tolerance.
//
// Host side.  Between graph replays: retire finished, failed and cancelled simulations (fold), admit
// queued requests first come first served while the memory budget, the slots and the resident-node cap
// allow, write the tables anew if anything changed.  The retired simulations' fields go to the host, and
// their memory back, before admissions where requests wait, else beside the next replay.  The graph reads the
// tables from device memory; it is captured again when a table outgrows its part of them or fills little
// of it, when the kernels that residents need change, and when the residual check is switched on or off.
#include <math.h>
#include <stddef.h>
#include <string.h>

#include <algorithm>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <unordered_set>
#include <vector>

#include "host_copy.hpp"
#include "internal.hpp"
#include "pool.hpp"
#include "pool_policy.hpp"
#include "strip_plan.hpp"

using namespace vplbm;

namespace vplbm {

// The final step's per-tile sums (mass, body forces): wave shuffles, then the waves in order,
// into the tile's slot of the simulation's partials.  Called by every thread of the workgroup.
template <bool DPP>
__device__ __forceinline__ void pool_tile_partials(const PoolSim &d, int tile, double rho, double fx,
                                                   double fy, int id, double (*part)[kRingWidth])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane < kRingWidth) part[wave][lane] = 0.0;
    const double mw = wave_sum<DPP>(rho);
    if (lane == 0) part[wave][0] = mw;
    unsigned long long solid = __ballot(id != 0);
    while (solid) {
        const int lead = __ffsll((unsigned long long)solid) - 1;
        const int b = __shfl(id, lead, 64);
        const bool mine = id == b;
        const double sx = wave_sum<DPP>(mine ? -fx : 0.0);
        const double sy = wave_sum<DPP>(mine ? -fy : 0.0);
        if (lane == 0) {
            part[wave][1 + 2 * (b - 1)] = sx;
            part[wave][2 + 2 * (b - 1)] = sy;
        }
        solid &= ~__ballot(mine);
    }
    __syncthreads();
    if ((int)threadIdx.x < d.width) {
        double v = 0.0;
        for (int w = 0; w < kBlock2 / 64; w++) v += part[w][threadIdx.x];
        d.partials[(size_t)tile * d.width + threadIdx.x] = v;
    }
}

// One tile of one simulation for `nsteps` (1 or 2) steps from `done`: the node arithmetic of the
// single-simulation kernels (update_node, or the two-step form with the first step kept in LDS),
// so a simulation's fields do not depend on the launch shape or its co-residents.  CONV: the
// simulation has a convective outlet; as in the single-simulation two-step kernel, the first step
// reads the previous values from global memory and keeps what it records for the tile's rows in
// LDS (outl, 3 x kPoolTileH values), and the second applies the outlet rule with them and records
// its own for the next launch.
template <int S, bool CONV>
__device__ __forceinline__ void pool_tile(const PoolSim &d, int tile, long long done, int nsteps, int b,
                                          unsigned char *lds, double (*part)[kRingWidth],
                                          double *outl_lds, unsigned *status)
{
    using C = Codec<S>;
    using T = typename C::real;
    using E = typename C::elem;
    constexpr int odirs[3] = {3, 6, 7};           // the directions entering from x = nx
    const Geom &g = d.g;
    // selects rather than indexing: the kernel holds d in registers, not in memory
    const E *__restrict__ src = static_cast<const E *>(b ? d.buf[1] : d.buf[0]);
    E *__restrict__ dst = static_cast<E *>(b ? d.buf[0] : d.buf[1]);
    const Outlet none{nullptr, nullptr, 0.0};
    void *const oprev = b ? d.outlet[1] : d.outlet[0];
    void *const onext = b ? d.outlet[0] : d.outlet[1];
    const Outlet one{CONV ? oprev : nullptr, CONV ? onext : nullptr, d.ou};
    const Outlet out1{CONV ? oprev : nullptr, nullptr, d.ou};
    T *outl = reinterpret_cast<T *>(outl_lds);
    const int x0 = (tile % d.ntx) * kPoolTileW, y0 = (tile / d.ntx) * kPoolTileH;
    const int x = x0 + (threadIdx.x % kPoolTileW), y = y0 + (threadIdx.x / kPoolTileW);
    const bool active = (x < g.nx) & (y < g.ny);
    double rho = 0.0, fx = 0.0, fy = 0.0;
    int id = 0;
    bool bad = false;
    if (nsteps == 1) {
        if (active) {
            const auto m = update_node<S>(src, dst, d.mask, d.bodies, g, CONV ? one : none, d.p, x, y, id,
                                          (unsigned)done);
            rho = 1.0 + double(m.drho);
            fx = double(m.fx);
            fy = double(m.fy);
            bad = !(rho > 0.0 && rho < 1e30);
        }
    } else {
        E *mid = reinterpret_cast<E *>(lds);
        for (int it = 0; it < (kPoolEN + kBlock2 - 1) / kBlock2; it++) {
            const int e = threadIdx.x + it * kBlock2;
            const int lx = e % kPoolEW - 1, ly = e / kPoolEW - 1;
            int hx = x0 + lx, hy = y0 + ly;
            bool live = e < kPoolEN;
            if (hx < 0 || hx >= g.nx) {
                if (g.xper && hx >= -1 && hx <= g.nx) hx += hx < 0 ? g.nx : -g.nx;
                else live = false;
            }
            if (hy < 0 || hy >= g.ny) {
                if (g.yper && hy >= -1 && hy <= g.ny) hy += hy < 0 ? g.ny : -g.ny;
                else live = false;
            }
            if (live) {
                T f[9];
                int hid;
                const bool own = (lx >= 0) & (lx < kPoolTileW) & (ly >= 0) & (ly < kPoolTileH) &
                                 (x0 + lx < g.nx) & (y0 + ly < g.ny);
                pull<S>(src, hx, hy, g, CONV ? out1 : none, f);
                if (CONV && hx == g.nx - 1 && own)
                    for (int k = 0; k < 3; k++) outl[k * kPoolTileH + ly] = f[odirs[k]];
                const auto m = relax_node(f, d.mask, d.bodies, g, d.p, hx, hy, hid);
                store_node<S>(mid, kPoolEN, unsigned(e), f, unsigned(hy * g.pitch + hx), (unsigned)done);
                const double r1 = 1.0 + double(m.drho);
                bad |= own && !(r1 > 0.0 && r1 < 1e30);
            }
        }
        __syncthreads();
        if (active) {
            T f[9];
            pull_tile<S>(mid, kPoolEN, kPoolEW, x, y, x0, y0, g, f);
            if (CONV && x == g.nx - 1) {
                // the outlet rule of pull, with the first step's values from LDS
                const T u = T(d.ou);
                T *next = static_cast<T *>(onext);
                for (int k = 0; k < 3; k++) {
                    int pa;
                    const unsigned jn = tile_source(odirs[k], g.nx - 2, y, x0, y0, kPoolEW, g, pa);
                    const T nb = C::load(mid + pa * kPoolEN, jn, weight<T>(odirs[k]));
                    f[odirs[k]] = (outl[k * kPoolTileH + (y - y0)] + u * nb) / (T(1) + u);
                }
                for (int k = 0; k < 3; k++) next[k * g.ny + y] = f[odirs[k]];
            }
            const auto m = relax_node(f, d.mask, d.bodies, g, d.p, x, y, id);
            const unsigned i = y * g.pitch + x;
            store_node<S>(dst, g.plane, i, f, i, (unsigned)(done + 1));
            rho = 1.0 + double(m.drho);
            fx = double(m.fx);
            fy = double(m.fy);
            bad |= !(rho > 0.0 && rho < 1e30);
        }
    }
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(status, 1u);
    if (done + nsteps == d.target) pool_tile_partials<wave_sum_dpp<T>()>(d, tile, rho, fx, fy, id, part);
}

// pool_tile with or without the convective outlet (a separate instantiation, as in the
// single-simulation two-step kernel).
template <int S>
__device__ __forceinline__ void pool_tile2(const PoolSim &d, int tile, long long done, int nsteps, int b,
                                           unsigned char *lds, double (*part)[kRingWidth], double *outl,
                                           unsigned *status)
{
    if (d.conv) pool_tile<S, true>(d, tile, done, nsteps, b, lds, part, outl, status);
    else pool_tile<S, false>(d, tile, done, nsteps, b, lds, part, outl, status);
}

// One or two steps of every resident simulation that KERNEL (kPoolTiles32: FP32 arithmetic, kPoolTiles64:
// FP64) takes.  Two kernels, so the FP32 formats are
// not held to the FP64 path's registers and LDS: measured 4 waves per SIMD with one for all.  The host
// writes the table in XCD order (upload_tables), so the entry is found without first reading the
// tile count: the two loads are issued together, and a workgroup starts with two dependent loads
// (its entry, then its simulation's descriptor) before its populations.
template <int KERNEL> __global__ __launch_bounds__(kBlock2) void pool_step_kernel(PoolLaunch a)
{
    // the LDS tile in the kernel's widest storage format
    __shared__ __align__(16) unsigned char lds[9 * kPoolEN * (KERNEL == kPoolTiles64 ? 8 : 4)];
    __shared__ double part[kBlock2 / 64][kRingWidth];
    __shared__ double outl[3 * kPoolTileH];                   // convective outlet records
    const int n = *a.ntiles;
    const TileRef tr = a.tiles[blockIdx.x];                   // the table spans the grid
    if ((int)blockIdx.x >= n) return;                         // uniform over the workgroup
    // A local copy of the descriptor: its fields are read once into scalar registers (read through
    // the pointer, they were read again after stores that might alias it: measured 16% of the
    // kernel's time).  The status flag is written through the pointer.
    const PoolSim d = a.sims[tr.slot];
    unsigned *status = &a.sims[tr.slot].status;
    const long long start = *a.t_base - d.t0, left = d.target - start;
    if (!d.active || start < 0 || left <= 0) return;          // uniform over the workgroup
    const int body = pool_body(d, left), k = body - a.t_off < 2 ? body - a.t_off : 2;
    if (k <= 0) return;
    const long long done = start + a.t_off;
    const int b = (pool_buf(d, start) + a.t_off / 2) & 1;
    if constexpr (KERNEL == kPoolTiles64) {
        if (d.storage == kF64) pool_tile2<kF64>(d, tr.tile, done, k, b, lds, part, outl, status);
        else pool_tile2<kF32D>(d, tr.tile, done, k, b, lds, part, outl, status);
    } else {
        switch (d.storage) {
        case kF32: pool_tile2<kF32>(d, tr.tile, done, k, b, lds, part, outl, status); break;
        case kF16S: pool_tile2<kF16S>(d, tr.tile, done, k, b, lds, part, outl, status); break;
        case kF16SR: pool_tile2<kF16SR>(d, tr.tile, done, k, b, lds, part, outl, status); break;
        case kBF16SR: pool_tile2<kBF16SR>(d, tr.tile, done, k, b, lds, part, outl, status); break;
        default: pool_tile2<kBF16S>(d, tr.tile, done, k, b, lds, part, outl, status); break;
        }
    }
}

// Final observables of the simulation in `slot`: value q (workgroup q) of its tiles' partial
// sums.  Thread j adds tiles j, j + 256, ... in order, a fixed butterfly adds each wave's lanes and
// thread 0 the four waves in order, so the result depends only on the simulation's own tiles.
constexpr int kFoldBlock = 256;
__global__ __launch_bounds__(kFoldBlock) void pool_fold_kernel(PoolSim *sims, int slot)
{
    __shared__ double ws[kFoldBlock / 64];
    const int q = blockIdx.x, width = sims[slot].width;
    const int nt = q < width ? sims[slot].ntiles : 0;
    const double *part = sims[slot].partials;
    double v = 0.0;
    for (int t = threadIdx.x; t < nt; t += kFoldBlock) v += part[(size_t)t * width + q];
    v = wave_sum<false>(v);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) sims[slot].obs[q] = ((ws[0] + ws[1]) + ws[2]) + ws[3];
}

// Whether a simulation checks its residual after this launch (the same test in both kernels).
__device__ __forceinline__ bool residual_due(const PoolSim &d, long long done)
{
    return d.active && d.tol > 0.0 && done >= d.next_check && done < d.target;
}

// Residual check, node part, on the state after the launch's steps: |u - u_snap|^2 and |u|^2 at
// a fluid node; the snapshot becomes u.
template <int S>
__device__ __forceinline__ void pool_residual_node(const PoolSim &d, int parity, int x, int y,
                                                   double &d2, double &u2)
{
    using E = typename Codec<S>::elem;
    const Outlet o{d.conv ? d.outlet[parity] : nullptr, nullptr, d.ou};   // read, not recorded
    int id;
    const auto m = observe_node<S>(static_cast<const E *>(d.buf[parity]), d.mask, d.bodies, d.g, o, d.p, x, y, id);
    const size_t n = (size_t)d.g.nx * d.g.ny, i = (size_t)y * d.g.nx + x;
    const double ux = double(m.ux), uy = double(m.uy);
    if (id == 0) {
        const double dx = ux - d.snap[i], dy = uy - d.snap[n + i];
        d2 = dx * dx + dy * dy;
        u2 = ux * ux + uy * uy;
    }
    d.snap[i] = ux;
    d.snap[n + i] = uy;
}

// One workgroup per table entry; sums per tile or block (waves in a fixed order).  A simulation's check
// goes through one table: that of its strips if it has them, whichever kernel advances it (a second pass
// would compare the state with the snapshot that the first one just took).
__global__ __launch_bounds__(kBlock2) void pool_residual_kernel(PoolSim *sims, const TileRef *tiles,
                                                                const int *ntiles,
                                                                const long long *t_base, int t_off)
{
    __shared__ double part[kBlock2 / 64][2];
    const int n = *ntiles;
    if ((int)blockIdx.x >= n) return;                         // uniform over the workgroup
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const TileRef tr = tiles[blockIdx.x];                     // the table is in XCD order
    const PoolSim &d = sims[tr.slot];
    const long long done = *t_base + t_off - d.t0;
    if (!residual_due(d, done) || (d.tail && tr.kernel < kPoolStrips)) return;   // uniform over the workgroup
    const int x = tr.x0 + lane, width = tr.w;
    const int parity = pool_buf(d, done);
    const int rows = tr.kernel >= kPoolStrips ? pool_block_rows(tr.form) : tr.y1 - tr.y0;
    for (int y0 = tr.y0, block = tr.tile; y0 < tr.y1; y0 += rows, block++) {   // a strip's blocks
        const int y1 = y0 + rows < tr.y1 ? y0 + rows : tr.y1;
        double d2 = 0.0, u2 = 0.0;
        for (int y = y0 + wave; y < y1; y += kBlock2 / 64) {   // rows, in order
            if (lane >= width || x >= d.g.nx) continue;
            double a2 = 0.0, b2 = 0.0;
            switch (d.storage) {
            case kF64: pool_residual_node<kF64>(d, parity, x, y, a2, b2); break;
            case kF32: pool_residual_node<kF32>(d, parity, x, y, a2, b2); break;
            case kF16S: pool_residual_node<kF16S>(d, parity, x, y, a2, b2); break;
            case kF32D: pool_residual_node<kF32D>(d, parity, x, y, a2, b2); break;
            case kF16SR: pool_residual_node<kF16SR>(d, parity, x, y, a2, b2); break;
            case kBF16SR: pool_residual_node<kBF16SR>(d, parity, x, y, a2, b2); break;
            default: pool_residual_node<kBF16S>(d, parity, x, y, a2, b2); break;
            }
            d2 += a2;
            u2 += b2;
        }
        d2 = wave_sum(d2);
        u2 = wave_sum(u2);
        __syncthreads();                                      // the block before is written
        if (lane == 0) {
            part[wave][0] = d2;
            part[wave][1] = u2;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            double v = 0.0;
            for (int w = 0; w < kBlock2 / 64; w++) v += part[w][threadIdx.x];
            d.rpart[2 * block + threadIdx.x] = v;
        }
    }
}

// Residual check, decision: workgroup s (one wave) folds slot s's tile sums in a fixed order;
// below the tolerance the simulation gets one more step, whose observables the step kernel
// reduces.
__global__ void pool_residual_fold_kernel(PoolSim *sims, const long long *t_base, int t_off)
{
    PoolSim &d = sims[blockIdx.x];
    const long long done = *t_base + t_off - d.t0;
    if (!residual_due(d, done)) return;                       // uniform over the workgroup
    double d2 = 0.0, u2 = 0.0;
    for (int t = threadIdx.x; t < d.ntiles; t += 64) {
        d2 += d.rpart[2 * t];
        u2 += d.rpart[2 * t + 1];
    }
    d2 = wave_sum(d2);
    u2 = wave_sum(u2);
    if (threadIdx.x == 0) {
        double r = u2 > 0.0 ? sqrt(d2 / u2) : (d2 > 0.0 ? INFINITY : 0.0);
        if (!d.have_snap) r = INFINITY;
        d.residual = r;
        d.have_snap = 1;
        d.next_check = done + d.every;
        if (r < d.tol) d.target = done + 1;
    }
}

__global__ void pool_advance_kernel(long long *t, long long n) { *t += n; }

}  // namespace vplbm

namespace {

struct Request {
    int64_t id = -1;
    vplbm_config cfg{};
    std::vector<vplbm_body> bodies;
    int64_t nsteps = 0;
    int keep_fields = 0;
    double tol = 0.0;
    int64_t every = 0;
    bool cancel = false;
    double residual = INFINITY;
    int state = VPLBM_QUEUED;
    int slot = -1;
    uint64_t bytes = 0;
    int64_t done = 0;
    vplbm_obs obs{};
    std::unique_ptr<double[]> fields;     // rho, ux, uy
    // device memory while resident
    void *buf[2] = {nullptr, nullptr};
    uint8_t *mask = nullptr;
    BodyParams *params = nullptr;
    BodyState *state_dev = nullptr;
    double *partials = nullptr;
    double *snap = nullptr;
    double *rpart = nullptr;
    void *outlet[2] = {nullptr, nullptr};
};

Geom pool_geometry(const vplbm_config &c)
{
    Geom g{};
    g.nx = c.nx;
    g.ny = c.ny;
    g.pitch = (c.nx + 63) / 64 * 64;
    g.plane = g.pitch * c.ny;
    g.xper = c.bc_xlo == VPLBM_PERIODIC;
    g.yper = c.bc_ylo == VPLBM_PERIODIC;
    g.inlet = c.bc_xlo == VPLBM_VELOCITY;
    return g;
}

// The kernel for a simulation in replays of spl steps.  The strip sweep needs the planes within its 32-bit
// offsets and a row of the lattice for every step.
int pool_kernel(int storage, const Geom &g, int spl)
{
    const PoolStrips *strips = pool_strips(storage);
    if (strips && spl >= pool_least(storage) && 9ull * (unsigned long long)g.plane * elem_bytes(storage) <= 0xFFFFFFFFull && g.ny >= strips->steps) return kPoolStrips + storage;
    return storage == kF64 || storage == kF32D ? kPoolTiles64 : kPoolTiles32;
}

const PoolStrips &strips_of(int kernel) { return *pool_strips(pool_storage(kernel)); }

// Kernel `kernel` for the main launches of d, `done` steps done, at a replay boundary.
void set_kernel(PoolSim &d, int kernel, long long done)
{
    const int buf = d.spk ? pool_buf(d, done) : 0;
    const bool strips = kernel >= kPoolStrips && kernel < kPoolPatches;
    d.kernel = kernel;
    d.from = done;
    d.from_buf = buf;
    d.spk = kernel < kPoolStrips ? 2 : strips ? strips_of(kernel).steps : pool_patches(kernel).steps;
    d.body = strips ? d.spl / d.tail * d.tail : d.spl;
    d.launches = (d.body + d.spk - 1) / d.spk + (d.body < d.spl);
}

// Tiles that vplbm_pool_bytes_needed counts, with sums of eight bodies each: those of 64 x 8 nodes, for
// binary32 64 x 14.  There are more blocks of strips than that, but their sums are of the bodies that a
// request has: only one with several bodies over much of the lattice takes more (charge).
int count_tiles(const Geom &g, int storage)
{
    const int th = storage == kF32 ? 14 : kPoolTileH;
    return (g.nx + kPoolTileW - 1) / kPoolTileW * ((g.ny + th - 1) / th);
}

// What the strips of a simulation are made of (StripPlan's segments): nothing but the simulation
// decides on them.
std::vector<StripTile> pool_segments(const Request &r, const Geom &g, int kernel)
{
    const PoolStrips &shape = strips_of(kernel);
    int box[kMaxBodies][4], nbox = 0;
    for (const vplbm_body &b : r.bodies) nbox += body_box(g, b, box[nbox]);
    return strip_segments({g.nx, g.ny, g.xper != 0, g.yper != 0, shape.own + 2 * shape.halo, shape.halo, shape.steps, nbox, box});
}

int segment_blocks(const StripTile &s) { return (s.y1 - s.y0 + pool_block_rows(s.form) - 1) / pool_block_rows(s.form); }

uint64_t bytes_needed(const vplbm_config &c, bool stop = false)
{
    const Geom g = pool_geometry(c);
    const int ntiles = count_tiles(g, c.storage);
    const uint64_t pop = (uint64_t)9 * g.plane * elem_bytes(c.storage);
    const uint64_t residual = stop ? 2 * (uint64_t)g.nx * g.ny * sizeof(double) + (uint64_t)ntiles * 2 * sizeof(double) : 0;
    const uint64_t outlet = c.bc_xhi == VPLBM_CONVECTIVE ? 2 * 3 * (uint64_t)g.ny * sizeof(double) : 0;
    return 2 * pop + (uint64_t)g.pitch * g.ny + sizeof(BodyParams) * kMaxBodies +
           sizeof(BodyState) * kMaxBodies + (uint64_t)ntiles * kRingWidth * sizeof(double) + residual +
           outlet;
}

// The kernel that a request is admitted with, what its strips are made of, and the tiles or blocks whose
// sums it takes memory for.
struct Parts {
    int kernel, ntiles, width;
    std::vector<StripTile> segments;
};
Parts parts_of(const Request &r, int spl)
{
    Parts p;
    const Geom g = pool_geometry(r.cfg);
    p.kernel = pool_kernel(r.cfg.storage, g, spl);
    p.width = 1 + 2 * (int)r.bodies.size();
    p.ntiles = (g.nx + kPoolTileW - 1) / kPoolTileW * ((g.ny + kPoolTileH - 1) / kPoolTileH);
    if (p.kernel >= kPoolStrips) {
        p.segments = pool_segments(r, g, p.kernel);
        p.ntiles = 0;
        for (const StripTile &s : p.segments) p.ntiles += segment_blocks(s);
    }
    return p;
}

size_t sum_bytes(int ntiles, int width, bool stop) { return (size_t)ntiles * (width + (stop ? 2 : 0)) * sizeof(double); }

// What a request that needs `need` bytes by the count above is charged: the memory it takes.  One that may
// run by that count always may: where the difference is all that is missing, alone.
uint64_t charge(const Request &r, uint64_t need, const vplbm_pool_config &cfg)
{
    const bool stop = r.tol > 0.0;
    const Parts p = parts_of(r, cfg.steps_per_launch);
    const uint64_t counted = sum_bytes(count_tiles(pool_geometry(r.cfg), r.cfg.storage), kRingWidth, stop), taken = sum_bytes(p.ntiles, p.width, stop);
    return taken <= counted ? need : std::min(need + (taken - counted), cfg.budget_bytes);
}

std::mutex g_pool_mu;
std::unordered_set<const void *> g_pools;

}  // namespace

// A simulation out of its slot, its memory not yet released.
struct Leaving {
    int64_t id;
    PoolSim sim;
    int state;                            // its request's, once its fields are on the host
};

struct vplbm_pool_s {
    vplbm_pool_config cfg{};
    hipStream_t stream = nullptr;
    bool own_stream = false;
    hipStream_t cap_stream = nullptr;
    hipGraphExec_t graph = nullptr;
    bool graph_checks = false;            // the graph ends with the residual-check kernels
    int graph_kernels = 0;                // step kernels in the graph (bits)
    PoolSim *d_sims = nullptr;
    TileRef *d_tiles = nullptr;           // the kernels' tables, one after the other
    int *d_ntiles = nullptr;              // entries of each
    long long *d_t = nullptr;             // pool step counter (steps every resident sim has run)
    long long *d_zero = nullptr;
    double *staging = nullptr;
    size_t staging_bytes = 0;
    HostCopy host_copy;                   // results to host memory
    int tile_cap = 0;
    // Of each kernel's table: where it begins, its workgroups per launch in the captured graph (as many
    // entries are there), and the entries that count.
    int table_at[kPoolKernels] = {}, table_cap[kPoolKernels] = {}, table_n[kPoolKernels] = {};
    long long t_host = 0;                 // host copy of *d_t after the last finished chunk
    std::vector<PoolSim> h_sims;
    std::vector<int64_t> slot_req;        // request id per slot (-1 free)
    std::vector<std::vector<StripTile>> segments;   // per slot: what its strips are made of
    std::map<int64_t, Request> reqs;
    std::deque<int64_t> queue;
    std::deque<Leaving> leaving;          // retired, in the order they are released
    hipStream_t copy_stream = nullptr;    // their fields, beside the next replay
    int64_t next_id = 0;
    uint64_t used = 0;
    bool in_flight = false;
    bool stale = false;                   // the device's tables are not those of h_sims (an upload is due)
    int32_t finished = 0;
    uint64_t max_nodes = 0;               // admission cap on resident lattice nodes (0: none)
    uint64_t resident_nodes = 0;
};

namespace {

bool pool_valid(const void *p)
{
    if (!p) return false;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    return g_pools.count(p) != 0;
}

void free_request_memory(vplbm_pool p, Request &r)
{
    void *ptrs[] = {r.buf[0], r.buf[1], r.mask, r.params, r.state_dev, r.partials, r.snap, r.rpart,
                    r.outlet[0], r.outlet[1]};
    for (void *q : ptrs)
        if (q) (void)hipFreeAsync(q, p->stream);
    r.outlet[0] = r.outlet[1] = nullptr;
    r.snap = nullptr;
    r.rpart = nullptr;
    r.buf[0] = r.buf[1] = nullptr;
    r.mask = nullptr;
    r.params = nullptr;
    r.state_dev = nullptr;
    r.partials = nullptr;
}

int ensure_pool_staging(vplbm_pool p, size_t bytes)
{
    if (p->staging_bytes >= bytes) return VPLBM_OK;
    HIP_TRY(hipStreamSynchronize(p->stream));
    if (p->staging) HIP_TRY(hipFree(p->staging));
    p->staging = nullptr;
    p->staging_bytes = 0;
    if (hipMalloc(&p->staging, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return fail(VPLBM_ENOMEM, "cannot allocate %zu bytes of staging memory", bytes);
    }
    p->staging_bytes = bytes;
    return VPLBM_OK;
}

long long steps_done(const vplbm_pool p, const PoolSim &d)
{
    const long long n = p->t_host - d.t0;
    return n < d.target ? n : d.target;
}

// Take a finished (or failed) simulation out of its slot: its observables and state.  Its memory stays
// (release).  Launches and copies on the pool's stream, and waits for them.
int retire(vplbm_pool p, int slot)
{
    Request &r = p->reqs[p->slot_req[slot]];
    PoolSim &d = p->h_sims[slot];
    const long long done = steps_done(p, d);
    r.done = done;
    r.residual = d.residual;
    memset(&r.obs, 0, sizeof r.obs);
    r.obs.step = done - 1;
    r.obs.nbodies = (int32_t)r.bodies.size();
    r.obs.status = (d.status & 1u) ? 1 : 0;
    const bool cancelled = r.cancel && done < d.target && !r.obs.status;
    if (done == d.target) {
        pool_fold_kernel<<<kRingWidth, kFoldBlock, 0, p->stream>>>(p->d_sims, slot);
        HIP_TRY(hipGetLastError());
        const char *dev_obs = reinterpret_cast<const char *>(p->d_sims + slot) + offsetof(PoolSim, obs);
        HIP_TRY(hipMemcpyAsync(d.obs, dev_obs, sizeof d.obs, hipMemcpyDeviceToHost, p->stream));
        HIP_TRY(hipStreamSynchronize(p->stream));
        r.obs.mass = d.obs[0];
        for (int k = 0; k < kMaxBodies; k++) {
            r.obs.fx[k] = d.obs[1 + 2 * k];
            r.obs.fy[k] = d.obs[2 + 2 * k];
        }
    }
    const int state = r.obs.status ? VPLBM_FAILED : (cancelled ? VPLBM_CANCELLED : VPLBM_DONE);
    host_log("pool %p: retire request %lld (%s) after %lld steps", (void *)p, (long long)r.id,
        state == VPLBM_DONE ? "done" : state == VPLBM_FAILED ? "failed" : "cancelled", done);
    p->stale = true;                      // until the upload the device steps it still
    p->leaving.push_back({r.id, d, state});
    p->resident_nodes -= (uint64_t)r.cfg.nx * r.cfg.ny;
    r.slot = -1;
    p->slot_req[slot] = -1;
    memset(&p->h_sims[slot], 0, sizeof(PoolSim));
    return VPLBM_OK;
}

// The retired simulations' fields to the host, and their memory back.  st: the pool's stream, or one
// beside it, after whatever touches their buffers or the staging memory has ended.
int release(vplbm_pool p, hipStream_t st)
{
    while (!p->leaving.empty()) {
        const Leaving &l = p->leaving.front();
        Request &r = p->reqs[l.id];
        const PoolSim &d = l.sim;
        if (r.keep_fields) {
            const size_t n = (size_t)d.g.nx * d.g.ny;
            int rc = ensure_pool_staging(p, 3 * n * sizeof(double));
            if (rc) return rc;
            r.fields.reset(new (std::nothrow) double[3 * n]);
            if (!r.fields) return fail(VPLBM_ENOMEM, "cannot allocate the host arrays of a result");
            StepArgs a{};
            const int pb = pool_buf_after(d, r.done);
            a.src = d.buf[pb];                          // the state after the steps done
            a.outlet.prev = d.conv ? d.outlet[pb] : nullptr;
            a.outlet.u = d.ou;
            a.mask = d.mask;
            a.bodies = d.bodies;
            a.t_base = p->d_zero;
            a.g = d.g;
            a.p = d.p;
            HIP_TRY(launch_readback(d.storage, a, p->staging, p->staging + n, p->staging + 2 * n, st));
            void *const dst[1] = {r.fields.get()};
            HIP_TRY(p->host_copy.read(st, p->staging, 3 * n * sizeof(double), dst, 1));
        }
        free_request_memory(p, r);
        p->used -= r.bytes;
        p->finished++;
        r.state = l.state;
        p->leaving.pop_front();
    }
    return VPLBM_OK;
}

// Allocate and initialise a queued request in a free slot.  Returns 1 if admitted, 0 if it does
// not fit the budget now, 2 if the device refused its memory, < 0 on error.
int admit(vplbm_pool p, Request &r, int slot)
{
    const uint64_t nodes = (uint64_t)r.cfg.nx * r.cfg.ny;
    const AdmissionState st{p->used, p->cfg.budget_bytes, p->resident_nodes, p->max_nodes, 1};
    if (!may_admit(st, r.bytes, nodes)) return 0;
    PoolSim d{};
    d.g = pool_geometry(r.cfg);
    Parts parts = parts_of(r, p->cfg.steps_per_launch);
    d.spl = p->cfg.steps_per_launch;
    d.tail = parts.kernel >= kPoolStrips ? strips_of(parts.kernel).steps : 0;
    set_kernel(d, parts.kernel, 0);
    d.ntx = (d.g.nx + kPoolTileW - 1) / kPoolTileW;
    d.ntiles = parts.ntiles;
    d.width = parts.width;
    const int conv = r.cfg.bc_xhi == VPLBM_CONVECTIVE ? 1 : 0;
    const size_t pop = (size_t)9 * d.g.plane * elem_bytes(r.cfg.storage);
    struct { void **ptr; size_t n; } allocs[] = {
        {&r.buf[0], pop}, {&r.buf[1], pop}, {(void **)&r.mask, (size_t)d.g.pitch * d.g.ny},
        {(void **)&r.params, sizeof(BodyParams) * kMaxBodies},
        {(void **)&r.state_dev, sizeof(BodyState) * kMaxBodies},
        {(void **)&r.partials, sum_bytes(d.ntiles, d.width, false)},
        {(void **)&r.snap, r.tol > 0.0 ? 2 * (size_t)d.g.nx * d.g.ny * sizeof(double) : 0},
        {(void **)&r.rpart, r.tol > 0.0 ? sum_bytes(d.ntiles, 0, true) : 0},
        {&r.outlet[0], conv ? 3 * (size_t)d.g.ny * sizeof(double) : 0},
        {&r.outlet[1], conv ? 3 * (size_t)d.g.ny * sizeof(double) : 0},
    };
    for (auto &a : allocs) {
        if (a.n == 0) continue;
        if (hipMallocAsync(a.ptr, a.n, p->stream) != hipSuccess) {
            (void)hipGetLastError();
            free_request_memory(p, r);
            return 2;   // the device is fuller than the budget says
        }
    }
    BodyParams hp[kMaxBodies];
    memset(hp, 0, sizeof hp);
    const int nb = (int)r.bodies.size();
    for (int k = 0; k < nb; k++) {
        const vplbm_body &b = r.bodies[k];
        hp[k].kind = b.kind; hp[k].cx = b.cx; hp[k].cy = b.cy; hp[k].r = b.r; hp[k].hx = b.hx;
        hp[k].hy = b.hy; hp[k].ux = b.ux; hp[k].uy = b.uy; hp[k].omega = b.omega;
    }
    HIP_TRY(hipMemcpyAsync(r.params, hp, sizeof hp, hipMemcpyHostToDevice, p->stream));
    HIP_TRY(launch_bodies(r.params, r.state_dev, nb, p->d_zero, 0, p->stream));
    HIP_TRY(launch_mask(r.mask, d.g, r.params, r.state_dev, nb, 0, 0, d.g.nx, d.g.ny, p->stream));
    d.buf[0] = r.buf[0];
    d.buf[1] = r.buf[1];
    d.mask = r.mask;
    d.bodies = r.state_dev;
    d.partials = r.partials;
    d.p = node_params(r.cfg);
    d.storage = r.cfg.storage;
    d.conv = conv;
    d.ou = r.cfg.u_in_x;
    d.outlet[0] = r.outlet[0];
    d.outlet[1] = r.outlet[1];
    d.active = 1;
    d.t0 = p->t_host;
    d.target = r.nsteps;
    d.tol = r.tol;
    d.every = r.every;
    d.next_check = r.every;
    d.residual = INFINITY;
    d.snap = r.snap;
    d.rpart = r.rpart;
    StepArgs a{};
    a.dst = d.buf[0];
    a.mask = d.mask;
    a.bodies = d.bodies;
    a.g = d.g;
    a.p = d.p;
    HIP_TRY(launch_init(d.storage, a, nullptr, nullptr, nullptr, r.cfg.rho0, r.cfg.ux0, r.cfg.uy0, p->stream));
    if (conv) {   // the previous-step outlet values start as the initial state's last column
        a.src = d.buf[0];
        HIP_TRY(launch_outlet_init(d.storage, a, d.outlet[0], p->stream));
    }
    // the body table copy above reads `hp` from the stack: let it land before returning
    HIP_TRY(hipStreamSynchronize(p->stream));
    p->stale = true;
    p->h_sims[slot] = d;
    p->segments[slot] = std::move(parts.segments);
    r.slot = slot;
    r.state = VPLBM_RUNNING;
    p->used += r.bytes;
    p->resident_nodes += nodes;
    host_log("pool %p: admit request %lld (%dx%d, %lld steps) in slot %d, %llu bytes; resident %llu nodes",
        (void *)p, (long long)r.id, r.cfg.nx, r.cfg.ny, (long long)r.nsteps, slot,
        (unsigned long long)r.bytes, (unsigned long long)p->resident_nodes);
    return 1;
}

int ensure_pool_graph(vplbm_pool p)
{
    bool checks = false;
    int kernels = 0;                      // bit k: a simulation of kernel k is resident
    for (const PoolSim &d : p->h_sims) {
        checks |= d.active && d.tol > 0.0;
        if (d.active) kernels |= 1 << d.kernel;
    }
    if (p->graph && p->graph_checks == checks && p->graph_kernels == kernels) return VPLBM_OK;
    if (p->graph) {
        HIP_TRY(hipGraphExecDestroy(p->graph));
        p->graph = nullptr;
    }
    int cap = 0;
    for (int kernel = 0; kernel < kPoolKernels; kernel++) cap += p->table_cap[kernel];
    host_log("pool %p: capture the step graph (%d workgroups per launch, %d steps, residual checks %d)",
        (void *)p, cap, p->cfg.steps_per_launch, (int)checks);
    if (!p->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&p->cap_stream, hipStreamNonBlocking));
    hipGraph_t graph = nullptr;
    HIP_TRY(hipStreamBeginCapture(p->cap_stream, hipStreamCaptureModeThreadLocal));
    hipError_t e = hipSuccess;
    // Each kernel's launches from the replay's start: its steps each (PoolSim::spk), what remains
    // last (pool_buf counts launches this way).  The kernels advance the same steps.
    const int spl = p->cfg.steps_per_launch;
    auto launch_on = [&](int table) { return PoolLaunch{p->d_sims, p->d_tiles + p->table_at[table], p->d_ntiles + table, p->d_t, 0}; };
    for (int kernel = 0; kernel < kPoolKernels; kernel++) {
        if (!(kernels >> kernel & 1)) continue;
        const int cap = p->table_cap[kernel];
        PoolLaunch a = launch_on(kernel);
        if (kernel >= kPoolStrips) {
            const auto launch = kernel < kPoolPatches ? strips_of(kernel).launch : pool_patches(kernel).launch;
            if (e == hipSuccess) e = launch(a, spl, cap, p->cap_stream);
            continue;
        }
        for (int j = 0; j < spl && e == hipSuccess; j += 2) {
            a.t_off = j;
            if (kernel == kPoolTiles32) pool_step_kernel<kPoolTiles32><<<dim3(cap), dim3(kBlock2), 0, p->cap_stream>>>(a);
            else pool_step_kernel<kPoolTiles64><<<dim3(cap), dim3(kBlock2), 0, p->cap_stream>>>(a);
            e = hipGetLastError();
        }
    }
    for (int table = kPoolStrips; table < kPoolPatches; table++)   // every format's strips: the tails
        if (e == hipSuccess && p->table_cap[table]) e = strips_of(table).tail(launch_on(table), p->table_cap[table], p->cap_stream);
    if (e == hipSuccess && checks) {
        const int n = p->cfg.steps_per_launch;
        for (int table = 0; table < kPoolPatches && e == hipSuccess; table++) {
            if (!p->table_cap[table]) continue;
            const PoolLaunch a = launch_on(table);
            pool_residual_kernel<<<dim3(p->table_cap[table]), dim3(kBlock2), 0, p->cap_stream>>>(a.sims, a.tiles, a.ntiles, a.t_base, n);
            e = hipGetLastError();
        }
        if (e == hipSuccess) {
            pool_residual_fold_kernel<<<dim3(p->cfg.max_slots), dim3(64), 0, p->cap_stream>>>(p->d_sims, p->d_t, n);
            e = hipGetLastError();
        }
    }
    if (e == hipSuccess) {
        pool_advance_kernel<<<1, 1, 0, p->cap_stream>>>(p->d_t, p->cfg.steps_per_launch);
        e = hipGetLastError();
    }
    p->graph_checks = checks;
    p->graph_kernels = kernels;
    hipError_t e2 = hipStreamEndCapture(p->cap_stream, &graph);
    if (e != hipSuccess) {
        if (graph) (void)hipGraphDestroy(graph);
        return fail(VPLBM_EHIP, "pool graph capture failed: %s", hipGetErrorString(e));
    }
    HIP_TRY(e2);
    e = hipGraphInstantiate(&p->graph, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    HIP_TRY(e);
    return VPLBM_OK;
}

// The strips of every resident simulation of a format, sorted by rows and columns (patches leave the
// tail of a replay to them): blocks of a segment
// together until all of them make as many strips as the GPU holds waves.  14 simulations of 4.9 million
// nodes, us per step: 41 with half as many strips, 33.7 with 0.8, 32.7, 34.5 with 1.2, 32.2 with twice as
// many; the last five of them, 1.6 million: 13.8, 13.1, 12.8, 12.5, 12.4.
void pool_strip_entries(vplbm_pool p, int storage, std::vector<TileRef> &out)
{
    const PoolStrips &shape = *pool_strips(storage);
    auto takes = [&](const PoolSim &d) { return d.active && d.tail && d.storage == storage; };
    int most = 0;
    for (const PoolSim &d : p->h_sims)
        if (takes(d)) most = std::max(most, d.g.ny);
    if (!most) return;
    auto pieces = [&](const StripTile &s, double t) {   // strips of a segment
        const int m = std::max(1, strip_rows(t, s.form, shape.steps) / pool_block_rows(s.form));
        return (segment_blocks(s) + m - 1) / m;
    };
    const double t = strip_time(shape.steps, most, 1024 * shape.waves * 39 / 40, [&](double t) {
        long long n = 0;
        for (int s = 0; s < p->cfg.max_slots; s++)
            if (takes(p->h_sims[s]))
                for (const StripTile &g : p->segments[s]) n += pieces(g, t);
        return n;
    });
    for (int s = 0; s < p->cfg.max_slots; s++) {
        if (!takes(p->h_sims[s])) continue;
        const size_t first = out.size();
        int tile = 0;
        for (const StripTile &g : p->segments[s]) {
            const int blocks = segment_blocks(g), rows = pool_block_rows(g.form), n = pieces(g, t);
            for (int i = 0; i < n; i++) {
                const int b0 = (int)((long long)blocks * i / n), b1 = (int)((long long)blocks * (i + 1) / n);
                out.push_back({s, tile + b0, kPoolStrips + storage, g.x0, shape.own, g.y0 + b0 * rows, std::min(g.y0 + b1 * rows, g.y1), g.form});
            }
            tile += blocks;
        }
        std::stable_sort(out.begin() + first, out.end(), [](const TileRef &a, const TileRef &b) {
            return a.y0 != b.y0 ? a.y0 < b.y0 : a.x0 < b.x0;
        });
    }
}

// The kernels of the simulations that strips or patches advance, for what is resident now (at a replay
// boundary): a change goes on from the buffer that holds the state.
void choose_kernels(vplbm_pool p)
{
    for (PoolSim &d : p->h_sims) {
        if (!d.active || !d.tail) continue;
        const int kernel = pool_choose(d.storage, (long long)p->resident_nodes);
        if (kernel != d.kernel) set_kernel(d, kernel, p->t_host - d.t0);
    }
}

int upload_tables(vplbm_pool p)
{
    choose_kernels(p);
    std::vector<TileRef> table[kPoolKernels];
    for (int s = 0; s < p->cfg.max_slots; s++) {
        const PoolSim &d = p->h_sims[s];
        if (!d.active || (d.kernel >= kPoolStrips && d.kernel < kPoolPatches)) continue;
        const bool patches = d.kernel >= kPoolPatches;
        const int w = patches ? pool_patches(d.kernel).w : kPoolTileW, h = patches ? pool_patches(d.kernel).h : kPoolTileH;
        int t = 0;
        for (int y0 = 0; y0 < d.g.ny; y0 += h)
            for (int x0 = 0; x0 < d.g.nx; x0 += w) table[d.kernel].push_back({s, t++, d.kernel, x0, w, y0, std::min(y0 + h, d.g.ny), 0});
    }
    for (int kernel = kPoolStrips; kernel < kPoolPatches; kernel++)
        if (pool_strips(pool_storage(kernel))) pool_strip_entries(p, pool_storage(kernel), table[kernel]);
    // A table that outgrows its part, or fills little of it (workgroups without an entry cost time too:
    // 4096 of 768 threads 4 us), moves all of them, and the graph is captured again.
    bool move = false;
    for (int k = 0; k < kPoolKernels; k++) {
        const int n = (int)table[k].size(), cap = p->table_cap[k];
        move |= n > cap || (n == 0) != (cap == 0) || cap > 4 * std::max(n, 64);
    }
    if (move) {
        int total = 0;
        for (int k = 0; k < kPoolKernels; k++) {
            const int n = (int)table[k].size();
            int cap = n ? 64 : 0;
            while (cap < n) cap *= 2;
            p->table_at[k] = total;
            p->table_cap[k] = cap;
            total += cap;
        }
        HIP_TRY(hipStreamSynchronize(p->stream));
        if (p->graph) {
            HIP_TRY(hipGraphExecDestroy(p->graph));
            p->graph = nullptr;
        }
        if (total > p->tile_cap) {
            if (p->d_tiles) HIP_TRY(hipFree(p->d_tiles));
            p->d_tiles = nullptr;
            p->tile_cap = 0;
            int cap = 4096;
            while (cap < total) cap *= 2;
            if (hipMalloc(&p->d_tiles, sizeof(TileRef) * cap) != hipSuccess) {
                (void)hipGetLastError();
                memset(p->table_cap, 0, sizeof p->table_cap);
                return fail(VPLBM_ENOMEM, "cannot allocate the tile table");
            }
            p->tile_cap = cap;
        }
    }
    std::vector<TileRef> order;
    for (int k = 0; k < kPoolKernels; k++) {
        const int n = p->table_n[k] = (int)table[k].size();
        for (int b = 0; b < n; b++) order.push_back(table[k][xcd_entry(b, n)]);
        order.resize(p->table_at[k] + p->table_cap[k], TileRef{});
    }
    if (!order.empty()) HIP_TRY(hipMemcpyAsync(p->d_tiles, order.data(), sizeof(TileRef) * order.size(), hipMemcpyHostToDevice, p->stream));
    HIP_TRY(hipMemcpyAsync(p->d_ntiles, p->table_n, sizeof p->table_n, hipMemcpyHostToDevice, p->stream));
    HIP_TRY(hipMemcpyAsync(p->d_sims, p->h_sims.data(), sizeof(PoolSim) * p->cfg.max_slots, hipMemcpyHostToDevice, p->stream));
    // The host copies above read memory that changes on the next call: finish them.
    HIP_TRY(hipStreamSynchronize(p->stream));
    p->stale = false;
    return VPLBM_OK;
}

}  // namespace

extern "C" {

int vplbm_pool_bytes_needed(const vplbm_config *cfg, uint64_t *bytes)
{
    int rc = check_config(cfg);
    if (rc) return rc;
    if (!bytes) return fail(VPLBM_EINVAL, "bytes is NULL");
    *bytes = bytes_needed(*cfg);
    return VPLBM_OK;
}

int vplbm_pool_create(const vplbm_pool_config *cfg, vplbm_pool *out)
{
    if (!out) return fail(VPLBM_EINVAL, "out is NULL");
    *out = nullptr;
    if (!cfg) return fail(VPLBM_EINVAL, "config is NULL");
    if (cfg->abi_version != VPLBM_ABI_VERSION) return fail(VPLBM_EINVAL, "abi_version %u, library is %d", cfg->abi_version, VPLBM_ABI_VERSION);
    if (cfg->max_slots < 1 || cfg->max_slots > kPoolMaxSlots) return fail(VPLBM_EINVAL, "max_slots must be in [1, %d]", kPoolMaxSlots);
    if (cfg->steps_per_launch < 1 || cfg->steps_per_launch > 4096) return fail(VPLBM_EINVAL, "steps_per_launch must be in [1, 4096]");
    if (cfg->budget_bytes == 0) return fail(VPLBM_EINVAL, "budget_bytes must be > 0");
    vplbm_pool p = new vplbm_pool_s();
    p->cfg = *cfg;
    if (cfg->stream) {
        p->stream = (hipStream_t)cfg->stream;
    } else {
        if (hipStreamCreateWithFlags(&p->stream, hipStreamNonBlocking) != hipSuccess) {
            delete p;
            return fail(VPLBM_EHIP, "cannot create a stream");
        }
        p->own_stream = true;
    }
    p->h_sims.assign(cfg->max_slots, PoolSim{});
    memset(p->h_sims.data(), 0, sizeof(PoolSim) * cfg->max_slots);
    p->slot_req.assign(cfg->max_slots, -1);
    p->segments.resize(cfg->max_slots);
    hipError_t e = hipMalloc(&p->d_sims, sizeof(PoolSim) * cfg->max_slots);
    if (e == hipSuccess) e = hipMalloc(&p->d_ntiles, sizeof(int) * kPoolKernels);
    if (e == hipSuccess) e = hipMalloc(&p->d_zero, sizeof(long long));
    if (e == hipSuccess) e = hipMalloc(&p->d_t, sizeof(long long));
    if (e == hipSuccess) e = hipMemsetAsync(p->d_zero, 0, sizeof(long long), p->stream);
    if (e == hipSuccess) e = hipMemsetAsync(p->d_t, 0, sizeof(long long), p->stream);
    if (e == hipSuccess) e = hipMemsetAsync(p->d_ntiles, 0, sizeof(int) * kPoolKernels, p->stream);
    if (e == hipSuccess) e = hipMemsetAsync(p->d_sims, 0, sizeof(PoolSim) * cfg->max_slots, p->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(p->stream);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (p->d_sims) (void)hipFree(p->d_sims);
        if (p->d_ntiles) (void)hipFree(p->d_ntiles);
        if (p->d_zero) (void)hipFree(p->d_zero);
        if (p->d_t) (void)hipFree(p->d_t);
        if (p->own_stream) (void)hipStreamDestroy(p->stream);
        delete p;
        return fail(VPLBM_ENOMEM, "cannot allocate the pool tables: %s", hipGetErrorString(e));
    }
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        g_pools.insert(p);
    }
    *out = p;
    return VPLBM_OK;
}

int vplbm_pool_submit(vplbm_pool p, const vplbm_config *cfg, const vplbm_body *bodies,
                      int32_t nbodies, int64_t nsteps, int32_t keep_fields, int64_t *id)
{
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    if (!id) return fail(VPLBM_EINVAL, "id is NULL");
    int rc = check_config(cfg);
    if (rc) return rc;
    rc = check_bodies(bodies, nbodies);
    if (rc) return rc;
    for (int k = 0; k < nbodies; k++)
        if (bodies[k].freq != 0.0 && (bodies[k].ax != 0.0 || bodies[k].ay != 0.0))
            return fail(VPLBM_EINVAL, "pool simulations take static bodies only (body %d moves)", k);
    if (nsteps < 1) return fail(VPLBM_EINVAL, "nsteps must be >= 1");
    const uint64_t need = bytes_needed(*cfg);
    if (need > p->cfg.budget_bytes)
        return fail(VPLBM_EBUDGET, "simulation needs %llu bytes, pool budget is %llu", (unsigned long long)need, (unsigned long long)p->cfg.budget_bytes);
    Request r;
    r.id = p->next_id++;
    r.cfg = *cfg;
    r.bodies.assign(bodies, bodies + nbodies);
    r.nsteps = nsteps;
    r.keep_fields = keep_fields ? 1 : 0;
    r.bytes = charge(r, need, p->cfg);
    *id = r.id;
    p->reqs[r.id] = std::move(r);
    p->queue.push_back(*id);
    return VPLBM_OK;
}

int vplbm_pool_set_stop(vplbm_pool p, int64_t id, double tol, int64_t every)
{
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    auto it = p->reqs.find(id);
    if (it == p->reqs.end()) return fail(VPLBM_EINVAL, "unknown request %lld", (long long)id);
    Request &r = it->second;
    if (r.state != VPLBM_QUEUED) return fail(VPLBM_ESTATE, "request %lld is no longer queued", (long long)id);
    if (!(tol > 0.0) || !isfinite(tol)) return fail(VPLBM_EINVAL, "tol must be finite and > 0");
    if (every < 1) return fail(VPLBM_EINVAL, "every must be >= 1");
    const uint64_t need = bytes_needed(r.cfg, true);
    if (need > p->cfg.budget_bytes)
        return fail(VPLBM_EBUDGET, "simulation with a residual snapshot needs %llu bytes, pool budget is %llu",
                    (unsigned long long)need, (unsigned long long)p->cfg.budget_bytes);
    r.tol = tol;
    r.every = every;
    r.bytes = charge(r, need, p->cfg);
    return VPLBM_OK;
}

int vplbm_pool_cancel(vplbm_pool p, int64_t id)
{
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    auto it = p->reqs.find(id);
    if (it == p->reqs.end()) return fail(VPLBM_EINVAL, "unknown request %lld", (long long)id);
    Request &r = it->second;
    if (r.state == VPLBM_QUEUED) {
        for (auto q = p->queue.begin(); q != p->queue.end(); ++q)
            if (*q == id) {
                p->queue.erase(q);
                break;
            }
        memset(&r.obs, 0, sizeof r.obs);
        r.obs.step = -1;
        r.obs.nbodies = (int32_t)r.bodies.size();
        r.done = 0;
        r.state = VPLBM_CANCELLED;
        r.keep_fields = 0;
        p->finished++;
        return VPLBM_OK;
    }
    if (r.state == VPLBM_RUNNING) {
        r.cancel = true;
        return VPLBM_OK;
    }
    return fail(VPLBM_ESTATE, "request %lld has already finished", (long long)id);
}

int vplbm_pool_set_admission(vplbm_pool p, uint64_t max_resident_nodes)
{
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    p->max_nodes = max_resident_nodes;
    return VPLBM_OK;
}

int vplbm_pool_residual(vplbm_pool p, int64_t id, double *residual)
{
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    if (!residual) return fail(VPLBM_EINVAL, "residual is NULL");
    auto it = p->reqs.find(id);
    if (it == p->reqs.end()) return fail(VPLBM_EINVAL, "unknown request %lld", (long long)id);
    const Request &r = it->second;
    *residual = r.slot >= 0 ? p->h_sims[r.slot].residual : r.residual;
    return VPLBM_OK;
}

int vplbm_pool_advance(vplbm_pool p, int32_t *running, int32_t *queued, int32_t *finished_total)
{
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    if (p->in_flight) {
        HIP_TRY(hipStreamSynchronize(p->stream));
        p->in_flight = false;
        p->t_host += p->cfg.steps_per_launch;
        HIP_TRY(hipMemcpy(p->h_sims.data(), p->d_sims, sizeof(PoolSim) * p->cfg.max_slots, hipMemcpyDeviceToHost));
    }
    for (int s = 0; s < p->cfg.max_slots; s++) {
        PoolSim &d = p->h_sims[s];
        if (!d.active) continue;
        const long long done = steps_done(p, d);
        p->reqs[p->slot_req[s]].done = done;
        if (done >= d.target || (d.status & 1u) || p->reqs[p->slot_req[s]].cancel) {
            int rc = retire(p, s);
            if (rc) return rc;
        }
    }
    // The retired simulations' fields take about 1 ms per 16 MB.  With requests waiting for the memory
    // that comes first; with none it runs beside the next replay (a batch of 14 of 128 to 896 nodes
    // square with fields: 9 of 74 ms).
    const bool beside = p->queue.empty();
    if (beside) {                         // no allocation while the replay runs: it would wait for it
        size_t most = 0;
        for (const Leaving &l : p->leaving)
            if (p->reqs[l.id].keep_fields) most = std::max(most, 3 * (size_t)l.sim.g.nx * l.sim.g.ny * sizeof(double));
        if (most && ensure_pool_staging(p, most) == VPLBM_OK && !p->copy_stream)
            HIP_TRY(hipStreamCreateWithFlags(&p->copy_stream, hipStreamNonBlocking));
    } else {
        int rc = release(p, p->stream);
        if (rc) return rc;
    }
    // First come, first served: the head of the queue waits for room rather than being passed.
    while (!p->queue.empty()) {
        int slot = -1;
        for (int s = 0; s < p->cfg.max_slots; s++)
            if (p->slot_req[s] < 0) { slot = s; break; }
        if (slot < 0) break;
        Request &r = p->reqs[p->queue.front()];
        int rc = admit(p, r, slot);
        if (rc < 0) return rc;
        if (rc == 2) {
            // The device refused the memory.  With simulations resident, retirements will free
            // some: wait.  With none, nothing ever will: the request fails instead of blocking
            // the queue for good.
            bool resident = false;
            for (int s = 0; s < p->cfg.max_slots; s++) resident |= p->h_sims[s].active != 0;
            if (!fail_when_refused(resident)) break;
            memset(&r.obs, 0, sizeof r.obs);
            r.obs.step = -1;
            r.obs.nbodies = (int32_t)r.bodies.size();
            r.obs.status = 2;
            r.done = 0;
            r.state = VPLBM_FAILED;
            r.keep_fields = 0;
            p->finished++;
            host_log("pool %p: request %lld failed: the device refused %llu bytes with nothing resident",
                (void *)p, (long long)r.id, (unsigned long long)r.bytes);
            p->queue.pop_front();
            continue;
        }
        if (rc == 0) break;
        p->slot_req[slot] = r.id;
        p->queue.pop_front();
    }
    int nrun = 0;
    for (int s = 0; s < p->cfg.max_slots; s++) nrun += p->h_sims[s].active ? 1 : 0;
    // Also where an earlier call ended in an error before its upload: what it retired may have given its
    // memory back since.
    if (p->stale) {
        int rc = upload_tables(p);
        if (rc) return rc;
    }
    if (nrun > 0) {
        int rc = ensure_pool_graph(p);
        if (rc) return rc;
        HIP_TRY(hipGraphLaunch(p->graph, p->stream));
        p->in_flight = true;
    }
    if (!p->leaving.empty()) {
        int rc = release(p, p->copy_stream ? p->copy_stream : p->stream);
        if (rc) return rc;
    }
    if (running) *running = nrun;
    if (queued) *queued = (int32_t)p->queue.size();
    if (finished_total) *finished_total = p->finished;
    return VPLBM_OK;
}

int vplbm_pool_status(vplbm_pool p, int64_t id, int32_t *state, int64_t *steps_done)
{
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    auto it = p->reqs.find(id);
    if (it == p->reqs.end()) return fail(VPLBM_EINVAL, "unknown request %lld", (long long)id);
    if (state) *state = it->second.state;
    if (steps_done) *steps_done = it->second.done;
    return VPLBM_OK;
}

int vplbm_pool_result(vplbm_pool p, int64_t id, vplbm_obs *out, double *rho, double *ux, double *uy)
{
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    auto it = p->reqs.find(id);
    if (it == p->reqs.end()) return fail(VPLBM_EINVAL, "unknown request %lld", (long long)id);
    Request &r = it->second;
    if (r.state != VPLBM_DONE && r.state != VPLBM_FAILED && r.state != VPLBM_CANCELLED)
        return fail(VPLBM_ESTATE, "request %lld has not finished", (long long)id);
    if ((rho || ux || uy) && !r.keep_fields) return fail(VPLBM_EINVAL, "request %lld did not keep its fields", (long long)id);
    if (out) *out = r.obs;
    const size_t n = (size_t)r.cfg.nx * r.cfg.ny;
    const double *const field = r.fields.get();   // null: cancelled or refused before it ran
    if (field && rho) host_copy(rho, field, n * sizeof(double));
    if (field && ux) host_copy(ux, field + n, n * sizeof(double));
    if (field && uy) host_copy(uy, field + 2 * n, n * sizeof(double));
    p->reqs.erase(it);
    return VPLBM_OK;
}

int vplbm_pool_destroy(vplbm_pool p)
{
    if (!p) return VPLBM_OK;
    if (!pool_valid(p)) return fail(VPLBM_EINVAL, "invalid pool");
    (void)hipStreamSynchronize(p->stream);
    for (auto &kv : p->reqs) free_request_memory(p, kv.second);
    (void)hipStreamSynchronize(p->stream);
    if (p->graph) (void)hipGraphExecDestroy(p->graph);
    void *ptrs[] = {p->d_sims, p->d_tiles, p->d_ntiles, p->d_zero, p->d_t, p->staging};
    for (void *q : ptrs)
        if (q) (void)hipFree(q);
    if (p->cap_stream) (void)hipStreamDestroy(p->cap_stream);
    if (p->copy_stream) (void)hipStreamDestroy(p->copy_stream);
    if (p->own_stream) (void)hipStreamDestroy(p->stream);
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        g_pools.erase(p);
    }
    delete p;
    return VPLBM_OK;
}

}  // extern "C"
