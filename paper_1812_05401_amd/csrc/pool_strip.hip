// The pool's strip sweep for FP32 arithmetic.
#include "pool_strip.hpp"

namespace vplbm {

// us per step of 14 simulations of 4.9 million nodes, and of the last five, 1.6 million: f32 42 and 13.8 on
// three-step tiles, 32.6 and 12.4 here; f16s 47 and 17.3 (two-step tiles), 30 and 13.8; bf16s 47 and
// 17.4, 32.6 and 15.3; bf16sr 51 and 18.8, 39 and 18.4.  f16sr 60 and 21.6, 53 and
// 25.6 (one value below 2^-14 sends a whole wave through the second rounding): see pool_choose.
const PoolStrips *pool_strips(int storage)
{
    static const PoolStrips f32 = pool_strips_form<kF32, 4, 4>(), f16s = pool_strips_form<kF16S, 4, 4>(),
                            bf16s = pool_strips_form<kBF16S, 4, 4>(), f16sr = pool_strips_form<kF16SR, 3, 4>(), bf16sr = pool_strips_form<kBF16SR, 3, 4>();
    switch (storage) {
    case kF32: return &f32;
    case kF16S: return &f16s;
    case kBF16S: return &bf16s;
    case kF16SR: return &f16sr;
    case kBF16SR: return &bf16sr;
    case kF64: case kF32D: return pool_strips_f64(storage);
    }
    return nullptr;
}

}  // namespace vplbm
