// Definitions of pick_plan_pow2 and pick_lars_pow2 (lsgd_pow2.hpp), included by
// the translation units that instantiate them.
#pragma once

#include "lsgd_plan_kernels.hpp"
#include "lsgd_pow2.hpp"

namespace lsgd {

template <typename GT, int W, int G>
PlanKernel plan_ct(bool cached) {
    if constexpr (ct_serves<GT>(W, G)) {
        constexpr int U = tile_units<GT>(W * G);
        if constexpr (cached_state_for(W * G))
            if (cached) return plan_step_kernel<GT, W, G, U, 1>();
        return plan_step_kernel<GT, W, G, U, 0>();
    }
    return nullptr;
}

template <typename GT, int W>
PlanKernel pick_plan_g(int G, bool cached) {
    switch (G) {
        case 1: return plan_ct<GT, W, 1>(cached);
        case 2: return plan_ct<GT, W, 2>(cached);
        case 4: return plan_ct<GT, W, 4>(cached);
        case 8: return plan_ct<GT, W, 8>(cached);
        case 16:
            if constexpr (W * 16 <= kMaxWorkers) return plan_ct<GT, W, 16>(cached);
            else return nullptr;
        case 32:
            if constexpr (W <= 4) return plan_ct<GT, W, 32>(cached);
            else return nullptr;
        case 64:
            if constexpr (W <= 2) return plan_ct<GT, W, 64>(cached);
            else return nullptr;
        case 128:
            if constexpr (W == 1) return plan_ct<GT, W, 128>(cached);
            else return nullptr;
    }
    return nullptr;
}

// Groups of 32 to 128 workers, in up to 4 groups.
template <typename GT, int W>
PlanKernel pick_plan_big_w(int G, bool cached) {
    switch (G) {
        case 1: return plan_ct<GT, W, 1>(cached);
        case 2:
            if constexpr (W * 2 <= kMaxWorkers) return plan_ct<GT, W, 2>(cached);
            else return nullptr;
        case 4:
            if constexpr (W * 4 <= kMaxWorkers) return plan_ct<GT, W, 4>(cached);
            else return nullptr;
    }
    return nullptr;
}

// Compile-time kernels for the power-of-two group counts of pick_flat, with
// parameters and momentum through the caches when `cached`.
template <typename GT>
PlanKernel pick_plan_pow2(int W, int G, bool cached) {
    switch (W) {
        case 1: return pick_plan_g<GT, 1>(G, cached);
        case 2: return pick_plan_g<GT, 2>(G, cached);
        case 3: return pick_plan_g<GT, 3>(G, cached);
        case 4: return pick_plan_g<GT, 4>(G, cached);
        case 5: return pick_plan_g<GT, 5>(G, cached);
        case 6: return pick_plan_g<GT, 6>(G, cached);
        case 7: return pick_plan_g<GT, 7>(G, cached);
        case 8: return pick_plan_g<GT, 8>(G, cached);
        case 12: return pick_plan_g<GT, 12>(G, cached);
        case 16: return pick_plan_g<GT, 16>(G, cached);
        case 32: return pick_plan_big_w<GT, 32>(G, cached);
        case 64: return pick_plan_big_w<GT, 64>(G, cached);
        case 128: return pick_plan_big_w<GT, 128>(G, cached);
    }
    return nullptr;
}

// LARS pass-1 kernels: compile-time (W, G) as for the step, null elsewhere.
template <typename GT, int W>
LarsKernel pick_lars_g(int G) {
    switch (G) {
        case 1: return lars_kernel_for<GT, W, 1>();
        case 2: return lars_kernel_for<GT, W, 2>();
        case 4: return lars_kernel_for<GT, W, 4>();
        case 8: return lars_kernel_for<GT, W, 8>();
        case 16:
            if constexpr (W * 16 <= kMaxWorkers) return lars_kernel_for<GT, W, 16>();
            else return nullptr;
        case 32:
            if constexpr (W <= 4) return lars_kernel_for<GT, W, 32>();
            else return nullptr;
        case 64:
            if constexpr (W <= 2) return lars_kernel_for<GT, W, 64>();
            else return nullptr;
        case 128:
            if constexpr (W == 1) return lars_kernel_for<GT, W, 128>();
            else return nullptr;
    }
    return nullptr;
}

template <typename GT, int W>
LarsKernel pick_lars_big_w(int G) {
    switch (G) {
        case 1: return lars_kernel_for<GT, W, 1>();
        case 2:
            if constexpr (W * 2 <= kMaxWorkers) return lars_kernel_for<GT, W, 2>();
            else return nullptr;
        case 4:
            if constexpr (W * 4 <= kMaxWorkers) return lars_kernel_for<GT, W, 4>();
            else return nullptr;
    }
    return nullptr;
}

template <typename GT>
LarsKernel pick_lars_pow2(int W, int G) {
    switch (W) {
        case 1: return pick_lars_g<GT, 1>(G);
        case 2: return pick_lars_g<GT, 2>(G);
        case 3: return pick_lars_g<GT, 3>(G);
        case 4: return pick_lars_g<GT, 4>(G);
        case 5: return pick_lars_g<GT, 5>(G);
        case 6: return pick_lars_g<GT, 6>(G);
        case 7: return pick_lars_g<GT, 7>(G);
        case 8: return pick_lars_g<GT, 8>(G);
        case 12: return pick_lars_g<GT, 12>(G);
        case 16: return pick_lars_g<GT, 16>(G);
        case 32: return pick_lars_big_w<GT, 32>(G);
        case 64: return pick_lars_big_w<GT, 64>(G);
        case 128: return pick_lars_big_w<GT, 128>(G);
    }
    return nullptr;
}

}  // namespace lsgd
