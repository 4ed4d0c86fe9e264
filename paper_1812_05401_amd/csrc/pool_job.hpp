// A pool simulation as a job of the strip sweep or the patches.
#pragma once

#include "pool.hpp"
#include "strip.hpp"

namespace vplbm {

__device__ __forceinline__ StripJob pool_job(const PoolSim *sim, int buf, long long done, int x0, int y0, int y1)
{
    // job.reduce: the density is looked at in every step
    return {sim->buf[buf], sim->buf[buf ^ 1], sim->mask, 0, sim->bodies, 0, sim->g, sim->p, sim->conv ? sim->outlet[buf] : nullptr,
            sim->outlet[buf ^ 1], sim->ou, x0, y0, y1, true, (unsigned)done};
}

}  // namespace vplbm
