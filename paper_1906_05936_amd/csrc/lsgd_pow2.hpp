// Compile-time (W, G) kernels for power-of-two group counts: pickers by
// gradient type. Each type's kernels are instantiated in translation units of
// their own (lsgd_flat_pow2_*.hip, lsgd_plan_pow2_*.hip), so that they compile
// in parallel and a change to the host code does not compile them again.
#pragma once

#include "lsgd_kernels.hpp"

namespace lsgd {

struct PlanArgs;
struct LarsArgs;

using FlatKernel = void (*)(StepArgs);
using PlanKernel = void (*)(PlanArgs);
using LarsKernel = void (*)(LarsArgs);

// A kernel and the number of units per lane tile it processes.
struct FlatPick {
    FlatKernel kernel;
    int tile;
};

// Null kernels for a grouping they do not cover.
template <typename GT>
FlatPick pick_flat(int W, int G, bool cached);
template <typename GT>
PlanKernel pick_plan_pow2(int W, int G, bool cached);
template <typename GT>
LarsKernel pick_lars_pow2(int W, int G);

}  // namespace lsgd
