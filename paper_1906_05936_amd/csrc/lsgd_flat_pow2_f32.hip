// Compile-time flat step kernels for power-of-two group counts, binary32 gradients.
#include "lsgd_flat_pow2.hpp"

namespace lsgd {
template FlatPick pick_flat<float>(int W, int G, bool cached);
}  // namespace lsgd
