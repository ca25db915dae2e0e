// optimize_f64_512.hip -- k_optimize with FP64 partials and blocks of 512 threads.
#include "optimize.hpp"

namespace pt {
PT_DEFINE_OPTIMIZE(optimize_f64_512, double, 512)
}  // namespace pt
