// optimize_f32_256.hip -- k_optimize with FP32 partials and blocks of 256 threads.
#include "optimize.hpp"

namespace pt {
PT_DEFINE_OPTIMIZE(optimize_f32_256, float, 256)
}  // namespace pt
