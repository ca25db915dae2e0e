// optimize_f64_256.hip -- k_optimize with FP64 partials and blocks of 256 threads.
#include "optimize.hpp"

namespace pt {
PT_DEFINE_OPTIMIZE(optimize_f64_256, double, 256)
}  // namespace pt
