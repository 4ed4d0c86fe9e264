// The strip sweep for 2-byte storage.
#include "strip_kernel.hpp"

namespace vplbm {

const StripShape *strip_shape_f16(int storage, long long nodes)
{
    static const StripShape f16 = strip_form<kF16S, 1, 4, 4>(), bf16 = strip_form<kBF16S, 1, 4, 4>();
    static const StripShape f16r = strip_form<kF16SR, 2, 3, 4>(), bf16r = strip_form<kBF16SR, 2, 3, 4>();
    switch (storage) {
    case kF16S: return nodes >= kStripLeast ? &f16 : nullptr;
    case kBF16S: return nodes >= kStripLeast ? &bf16 : nullptr;
    case kF16SR: return nodes >= kStripStochastic ? &f16r : nullptr;
    case kBF16SR: return nodes >= kStripStochastic ? &bf16r : nullptr;
    default: return nullptr;
    }
}

}  // namespace vplbm
