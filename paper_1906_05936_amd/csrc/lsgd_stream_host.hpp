// Launches of the stream step kernels (lsgd_stream.hpp).
#pragma once

#include "lsgd_host.hpp"
#include "lsgd_kernels.hpp"
#include "lsgd_program.hpp"

namespace lsgd {

struct PlanArgs;
struct LarsArgs;

// Units per lane tile: 16 elements for either gradient type, 8 in binary32's
// form of two units.
constexpr int stream_tile(bool bf16, bool two_units = false) { return bf16 || two_units ? 2 : 4; }

// Units per lane tile of the LARS norms stream kernel, either type.
constexpr int kLarsStreamTile = 2;

// `cached`: parameters and momentum through the caches; `tile`: units per lane
// tile (stream_tile).
void launch_flat_stream(const StepArgs& a, const Program& pr, bool bf16, bool cached, int tile, unsigned blocks,
                        hipStream_t s);
void launch_plan_stream(const PlanArgs& a, const Program& pr, bool bf16, bool cached, int tile, unsigned blocks,
                        hipStream_t s);
void launch_mean_stream(const MeanArgs& a, const Program& pr, bool bf16, dim3 blocks, hipStream_t s);
// Workgroup tiles of a vector of n elements, in units (launch_shape's count):
// the ragged end is a tile of its own.
int64_t stream_units(int64_t n, bool bf16, int tile);
void launch_lars_norms_stream(const LarsArgs& a, const Program& pr, bool bf16, unsigned blocks, hipStream_t s);

}  // namespace lsgd
