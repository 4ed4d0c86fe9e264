// The pool's strip sweep for FP64 arithmetic.
#include "pool_strip.hpp"

namespace vplbm {

// us per step of 14 simulations of 4.9 million nodes, and of the last five, 1.6 million: f64 102 and 26
// on two-step tiles, 57 and 19.5 here, 64 and 19.6 at four steps, 83 and 21.5 at three with three waves per
// SIMD; f32d 80 and 23 on tiles, 45 and 17.6 here, 51 and 18.3 at four steps with two waves.
const PoolStrips *pool_strips_f64(int storage)
{
    static const PoolStrips f64 = pool_strips_form<kF64, 5, 2>(), f32d = pool_strips_form<kF32D, 3, 4>();
    return storage == kF64 ? &f64 : &f32d;
}

}  // namespace vplbm
