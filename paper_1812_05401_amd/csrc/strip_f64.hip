// The strip sweep for the formats that compute in FP64.
#include "strip_kernel.hpp"

namespace vplbm {

const StripShape *strip_shape_f64(int storage, long long nodes)
{
    static const StripShape f64 = strip_form<kF64, 1, 5, 2>();
    static const StripShape wide = strip_form<kF32D, 2, 4, 2>(), narrow = strip_form<kF32D, 1, 3, 3>();
    if (nodes < kStripLeast) return nullptr;
    return storage == kF64 ? &f64 : nodes >= kStripWide ? &wide : &narrow;
}

}  // namespace vplbm
