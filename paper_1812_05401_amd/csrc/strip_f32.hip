// The strip sweep for binary32 storage with FP32 arithmetic.
#include "strip_kernel.hpp"

namespace vplbm {

const StripShape *strip_shape_f32(long long nodes)
{
    static const StripShape wide = strip_form<kF32, 2, 6, 2>(), narrow = strip_form<kF32, 1, 4, 4>();
    return nodes >= kStripWide ? &wide : nodes >= kStripLeast ? &narrow : nullptr;
}

}  // namespace vplbm
