// Compile-time plan step and LARS norm kernels for power-of-two group counts,
// binary32 gradients.
#include "lsgd_plan_pow2.hpp"

namespace lsgd {
template PlanKernel pick_plan_pow2<float>(int W, int G, bool cached);
template LarsKernel pick_lars_pow2<float>(int W, int G);
}  // namespace lsgd
