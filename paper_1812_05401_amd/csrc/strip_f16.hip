// The strip sweep for 2-byte storage.
#include "strip_kernel.hpp"

namespace vplbm {

// Stochastic rounding, us per step at 4.2, 8.4 and 16.8 million nodes on tiles, {1, 4, 4} and {2, 3, 4}: bf16 26.1, 48.5,
// 92.2; 24.7, 43.9, 80; 27.0, 44.2, 78.4; f16 on tiles and {2, 3, 4}: 29.7, 56.5, 108; 32.7, 54.6, 90.6 with strips of 18
// rows, 96.1 of 36 (a value below 2^-14 costs a wave a second rounding, which makes strips uneven).
const StripShape *strip_shape_f16(int storage, long long nodes)
{
    static const StripShape f16 = strip_form<kF16S, 1, 4, 4>(), bf16 = strip_form<kBF16S, 1, 4, 4>();
    static const StripShape f16r = strip_form<kF16SR, 2, 3, 4>(18), bf16r = strip_form<kBF16SR, 2, 3, 4>(), bf16n = strip_form<kBF16SR, 1, 4, 4>();
    switch (storage) {
    case kF16S: return nodes >= kStripLeast ? &f16 : nullptr;
    case kBF16S: return nodes >= kStripLeast ? &bf16 : nullptr;
    case kF16SR: return nodes >= kStripStochastic ? &f16r : nullptr;
    case kBF16SR: return nodes >= kStripStochastic ? &bf16r : nodes >= kStripStochasticB ? &bf16n : nullptr;
    default: return nullptr;
    }
}

}  // namespace vplbm
