// Launches of the stream step kernels (lsgd_stream.hpp).
#pragma once

#include "lsgd_host.hpp"
#include "lsgd_kernels.hpp"
#include "lsgd_program.hpp"

namespace lsgd {

struct PlanArgs;
struct LarsArgs;

// Units per lane tile: 16 elements for either gradient type.
constexpr int stream_tile(bool bf16) { return bf16 ? 2 : 4; }

// `cached`: parameters and momentum through the caches.
void launch_flat_stream(const StepArgs& a, const Program& pr, bool bf16, bool cached, unsigned blocks, hipStream_t s);
void launch_plan_stream(const PlanArgs& a, const Program& pr, bool bf16, bool cached, unsigned blocks, hipStream_t s);
void launch_lars_norms_stream(const LarsArgs& a, const Program& pr, bool bf16, unsigned blocks, hipStream_t s);

}  // namespace lsgd
