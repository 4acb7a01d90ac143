// Compile-time flat step kernels for power-of-two group counts, bfloat16 gradients.
#include "lsgd_flat_pow2.hpp"

namespace lsgd {
template FlatPick pick_flat<uint16_t>(int W, int G, bool cached);
}  // namespace lsgd
