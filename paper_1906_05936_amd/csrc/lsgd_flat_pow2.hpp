// Definition of pick_flat (lsgd_pow2.hpp), included by the translation units
// that instantiate it.
#pragma once

#include "lsgd_pow2.hpp"

namespace lsgd {

// Compile-time (W, G) kernels for power-of-two group counts G with N = W*G
// <= 128: groups of up to 16 workers (W a power of two, or 3, 5, 6, 7 or 12), or
// 32 to 128 workers in up to 4 groups, or 32 to 128 groups of up to 4
// workers; every other grouping takes the stream kernel (lsgd_stream.hpp).
// Both give the same bits.
// The compile-time kernel for (W, G), with parameters and momentum through
// the caches when `cached` (instantiated only where cached_state_for holds).
template <typename GT, int W, int G>
FlatKernel flat_ct(bool cached) {
    if constexpr (ct_serves<GT>(W, G)) {
        constexpr int U = tile_units<GT>(W * G);
        if constexpr (cached_state_for(W * G))
            if (cached) return flat_step_kernel<GT, W, G, U, 1>();
        return flat_step_kernel<GT, W, G, U, 0>();
    }
    return nullptr;
}

template <typename GT, int W>
FlatKernel pick_flat_g(int G, bool cached) {
    switch (G) {
        case 1: return flat_ct<GT, W, 1>(cached);
        case 2: return flat_ct<GT, W, 2>(cached);
        case 4: return flat_ct<GT, W, 4>(cached);
        case 8: return flat_ct<GT, W, 8>(cached);
        case 16:
            if constexpr (W * 16 <= kMaxWorkers) return flat_ct<GT, W, 16>(cached);
            else return nullptr;
        case 32:
            if constexpr (W <= 4) return flat_ct<GT, W, 32>(cached);
            else return nullptr;
        case 64:
            if constexpr (W <= 2) return flat_ct<GT, W, 64>(cached);
            else return nullptr;
        case 128:
            if constexpr (W == 1) return flat_ct<GT, W, 128>(cached);
            else return nullptr;
    }
    return nullptr;
}

// Groups of 32 to 128 workers, in up to 4 groups.
template <typename GT, int W>
FlatKernel pick_flat_big_w(int G, bool cached) {
    switch (G) {
        case 1: return flat_ct<GT, W, 1>(cached);
        case 2:
            if constexpr (W * 2 <= kMaxWorkers) return flat_ct<GT, W, 2>(cached);
            else return nullptr;
        case 4:
            if constexpr (W * 4 <= kMaxWorkers) return flat_ct<GT, W, 4>(cached);
            else return nullptr;
    }
    return nullptr;
}

template <typename GT>
FlatPick pick_flat(int W, int G, bool cached) {
    FlatKernel k = nullptr;
    switch (W) {
        case 1: k = pick_flat_g<GT, 1>(G, cached); break;
        case 2: k = pick_flat_g<GT, 2>(G, cached); break;
        case 3: k = pick_flat_g<GT, 3>(G, cached); break;
        case 4: k = pick_flat_g<GT, 4>(G, cached); break;
        case 5: k = pick_flat_g<GT, 5>(G, cached); break;
        case 6: k = pick_flat_g<GT, 6>(G, cached); break;
        case 7: k = pick_flat_g<GT, 7>(G, cached); break;
        case 8: k = pick_flat_g<GT, 8>(G, cached); break;
        case 12: k = pick_flat_g<GT, 12>(G, cached); break;
        case 16: k = pick_flat_g<GT, 16>(G, cached); break;
        case 32: k = pick_flat_big_w<GT, 32>(G, cached); break;
        case 64: k = pick_flat_big_w<GT, 64>(G, cached); break;
        case 128: k = pick_flat_big_w<GT, 128>(G, cached); break;
    }
    if (k) return FlatPick{k, tile_units<GT>(W * G)};
    return FlatPick{nullptr, 1};
}

}  // namespace lsgd
