// optimize_f32_512.hip -- k_optimize with FP32 partials and blocks of 512 threads.
#include "optimize.hpp"

namespace pt {
PT_DEFINE_OPTIMIZE(optimize_f32_512, float, 512)
}  // namespace pt
