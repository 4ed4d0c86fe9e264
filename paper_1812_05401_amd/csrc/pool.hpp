// What the serving pool's host side and its kernels share.
#pragma once

#include "kernels.hpp"
#include "strip_plan.hpp"

namespace vplbm {

constexpr int kPoolTileW = 64, kPoolTileH = 8;   // 512 nodes: one per thread of kBlock2
constexpr int kPoolEW = kPoolTileW + 2, kPoolEN = kPoolEW * (kPoolTileH + 2);
constexpr int kPoolMaxSlots = 1024;
static_assert(kPoolTileW * kPoolTileH == kBlock2, "one node per thread in the second step");

struct PoolSim {
    void *buf[2];
    const uint8_t *mask;
    const BodyState *bodies;
    double *partials;        // [ntiles][width] of the final step
    int width;               // its mass and two values for each of its bodies
    Geom g;
    NodeParams p;
    int storage;
    int ntx, ntiles;         // tiles in a row of them; and in all, or a strip's blocks in all
    int kernel;              // PoolKernel
    int spk;                 // steps per launch of the kernel that takes most of a replay
    int tail;                // steps that a strip takes as a replay's last launch, at most; 0: no strips
    long long from;          // steps done when `kernel` was chosen,
    int from_buf;            //   and the buffer that held the state then
    int body, launches;      // of a replay that the simulation does not end in: steps that the main launches
                             //   (spk each) take, and launches in all
    int conv;                // 1: convective outlet at x = nx - 1
    double ou;               // its convection speed (the inlet speed)
    void *outlet[2];         // its recorded values (3 x ny, compute type) per buffer parity
    int active;
    int spl;                 // steps per graph replay (the pool's steps_per_launch)
    long long t0, target;    // pool step at admission; steps to run
    unsigned status;
    double obs[kRingWidth];  // folded final observables
    // early stop (tol > 0): residual checks at done >= next_check, every `every` steps
    double tol, residual;
    long long every, next_check;
    int have_snap;
    double *snap;            // [2][ny*nx] velocity at the last check
    double *rpart;           // [ntiles][2] residual partial sums
};

// A tile or strip of the simulation in a slot: its columns x0 .. x0 + w - 1 (as far as the lattice
// goes) and rows y0 .. y1 - 1, a strip's form, and the index of its partial sums (of the first, for a strip of several blocks).
struct TileRef {
    int slot, tile, kernel;
    int x0, w, y0, y1, form;
};

// Rows of a strip's blocks by form (StripForm).  A strip is one or more whole blocks of a window, as many
// as suit all that is resident; the observables are added up block by block, so they do not depend
// on that.  As short as a strip should ever be, in equal time.
__host__ __device__ constexpr int pool_block_rows(int form) { return form == kPlain ? 8 : form == kMasked ? 4 : 6; }

// The kernels that advance simulations: tiles (FP32 or FP64 arithmetic), the strip sweep of a storage
// format S (kPoolStrips + S) or its patches in LDS (kPoolPatches or kPoolSmall + S).  A graph replay
// launches those that residents need.
enum PoolKernel { kPoolTiles32 = 0, kPoolTiles64 = 1, kPoolStrips = 2, kPoolPatches = 9, kPoolSmall = 16, kPoolKernels = 23 };
__host__ __device__ inline int pool_storage(int kernel) { return (kernel - kPoolStrips) % 7; }

// The arguments of all: the launch's first step in the replay; workgroup w takes entry w of the
// kernel's table, if there are so many.
struct PoolLaunch {
    PoolSim *sims;
    const TileRef *tiles;
    const int *ntiles;
    const long long *t_base;
    int t_off;
};

// The strip sweep over the pool (pool_strip.hpp): steps per launch, columns of a window that are its
// own and the halo on either side, waves per SIMD, the main launches of one replay of so many steps and
// its tail launch.
struct PoolStrips {
    int steps, own, halo, waves;
    hipError_t (*launch)(PoolLaunch a, int steps, int grid, hipStream_t st);
    hipError_t (*tail)(PoolLaunch a, int grid, hipStream_t st);
};
const PoolStrips *pool_strips(int storage);   // nullptr: none
const PoolStrips *pool_strips_f64(int storage);

// Patches over the pool (pool_patch.hip): steps per launch, size, main launches.
struct PoolPatches {
    int steps, w, h;
    hipError_t (*launch)(PoolLaunch a, int steps, int grid, hipStream_t st);
};
const PoolPatches &pool_patches(int kernel);
int pool_least(int storage);       // fewest steps of a replay for which strips are taken
int pool_choose(int storage, long long nodes);   // kernel for a format that has strips, with so many nodes resident

// A replay of spl steps is main launches, spk steps each and what remains last, and a tail launch of
// strips.  The tail takes the last 1 to `tail` steps of a simulation that ends in the replay (its final
// observables are then summed in one way, whichever kernel took the rest), and what strips of `tail`
// steps leave of any other.  Without strips (tail 0) there is no tail.  A launch moves a simulation's
// state to its other buffer, however many steps it takes.

// Steps that the main launches take for a simulation with `left` > 0 steps to go at the replay's start.
__host__ __device__ inline int pool_body(const PoolSim &d, long long left)
{
    if (left > d.spl) return d.body;
    return d.tail ? (int)(left - 1) / d.tail * d.tail : (int)left;
}

// Buffer holding the state at the start of a replay, `done` steps done.
__host__ __device__ inline int pool_buf(const PoolSim &d, long long done)
{
    return (d.launches & 1) ? (int)((d.from_buf + (done - d.from) / d.spl) & 1) : d.from_buf;
}

// Buffer holding the state after `done` steps, at a replay's end or where the simulation ends.
inline int pool_buf_after(const PoolSim &d, long long done)
{
    if (done != d.target || done == d.from) return pool_buf(d, done);
    const int last = (int)((done - d.from - 1) % d.spl) + 1;   // steps of the replay it ends in
    const int body = pool_body(d, last);
    return (pool_buf(d, done - last) + (body + d.spk - 1) / d.spk + (body < last)) & 1;
}

}  // namespace vplbm
