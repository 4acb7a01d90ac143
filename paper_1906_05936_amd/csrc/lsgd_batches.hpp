// Device code shared by the kernels that run a reduction program
// (lsgd_program.hpp): the register batches and the kernel arguments.
#pragma once

#include <stddef.h>

#include "lsgd_kernels.hpp"
#include "lsgd_plan_kernels.hpp"
#include "lsgd_program.hpp"

#pragma clang fp contract(off)

namespace lsgd {

// The steps' arguments with the reduction program, all in the kernel arguments.
// The program's batches, which every wave reads first, start a cache line (the
// padding in StepArgs and PlanArgs sees to it): 8 bytes off it a split step of up
// to 30000 elements took 2 % longer (1x32 bfloat16 n = 2500 3.15 / 3.22 us, 2x24
// binary32 3.61 / 3.70; plans of ten tensors 1.6 %).
struct FlatProgArgs {
    StepArgs a;
    Program pr;
};
struct PlanProgArgs {
    PlanArgs a;
    Program pr;
};
struct LarsProgArgs {
    LarsArgs la;
    Program pr;
};
template <typename A>
constexpr bool batches_on_a_line() {
    return (offsetof(A, pr) + offsetof(Program, batch)) % 64 == 0;
}
static_assert(batches_on_a_line<FlatProgArgs>() && batches_on_a_line<PlanProgArgs>() && batches_on_a_line<LarsProgArgs>(),
              "adjust the padding");

// Calls f(count, sub) with the batch's member count and inner group size as
// compile-time constants.
template <int V>
struct IntC {
    static constexpr int value = V;
};
template <typename F>
__device__ __forceinline__ void with_batch(int count, int sub, const F& f) {
#define LSGD_BATCH(C, S) \
    case (C) | ((S) << 4): f(IntC<C>{}, IntC<S>{}); break;
    switch (count | (sub << 4)) {
        LSGD_BATCH(1, 0) LSGD_BATCH(2, 0) LSGD_BATCH(3, 0) LSGD_BATCH(4, 0)
        LSGD_BATCH(5, 0) LSGD_BATCH(6, 0) LSGD_BATCH(7, 0) LSGD_BATCH(8, 0)
        LSGD_BATCH(1, 1) LSGD_BATCH(2, 1) LSGD_BATCH(3, 1) LSGD_BATCH(4, 1)
        LSGD_BATCH(5, 1) LSGD_BATCH(6, 1) LSGD_BATCH(7, 1) LSGD_BATCH(8, 1)
        LSGD_BATCH(2, 2) LSGD_BATCH(4, 2) LSGD_BATCH(6, 2) LSGD_BATCH(8, 2)
        LSGD_BATCH(3, 3) LSGD_BATCH(6, 3) LSGD_BATCH(4, 4) LSGD_BATCH(8, 4)
    }
#undef LSGD_BATCH
}

// x / group_div: a multiplication where the divisor is a power of two (the
// same rounding of the same exact quotient).
template <int T>
__device__ __forceinline__ void divide_group(float (&x)[T], float scale, float div) {
    if (scale != 0.f) {
#pragma unroll
        for (int v = 0; v < T; ++v) x[v] = x[v] * scale;
    } else {
#pragma unroll
        for (int v = 0; v < T; ++v) x[v] = x[v] / div;
    }
}

// The sum of a batch from leaves leaf(k, x): PW over its members, or over the
// divided sums of its whole groups.
template <int CNT, int SUB, int T, typename Leaf>
__device__ __forceinline__ void batch_sum(const Leaf& leaf, float scale, float div, float (&out)[T]) {
    if constexpr (SUB == 0) {
        pw_tree<0, CNT, T>(leaf, out);
    } else {
        pw_tree<0, CNT / SUB, T>([&](int g, float (&x)[T]) {
            pw_tree<0, SUB, T>([&](int k, float (&y)[T]) { leaf(g * SUB + k, y); }, x);
            divide_group<T>(x, scale, div);
        }, out);
    }
}

}  // namespace lsgd
