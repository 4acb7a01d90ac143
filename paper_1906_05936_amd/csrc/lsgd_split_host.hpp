// Pickers of the split step kernels (lsgd_split.hpp).
#pragma once

#include "lsgd_host.hpp"
#include "lsgd_kernels.hpp"
#include "lsgd_program.hpp"
#include "lsgd_rules.hpp"

namespace lsgd {

struct PlanArgs;
struct LarsArgs;

constexpr int kSplitVec = 4;           // elements per lane of the split kernels
constexpr int kSplitUnits = 64;        // lanes with elements per workgroup
constexpr int kSplitElems = kSplitVec * kSplitUnits;
constexpr int kLarsMergeChunks = 512;  // most pieces of a tensor whose partials every update workgroup sums itself

// Whether a flat step of n elements takes the split kernels; `compile_time`: a
// compile-time kernel serves the layout, `copy_bytes`: of copies per element.
bool use_split_flat(int64_t n, int32_t n_workers, bool bf16, bool compile_time, int64_t copy_bytes, int n_batches);
// Whether a plan may have split pieces (its rules: split_serves_plan, plan_fits_split).
bool split_plan_allowed(int n_batches);
// Whether a split step writes its copies in passes of their own, given what
// the rule for the other kernels says (`apart`).
bool separate_copy_out_small(int64_t n, int64_t copy_bytes, bool apart);

// Launches of the split kernels: `blocks` workgroups of split_waves() waves.
int split_waves(const Program& pr, int copies);
LaunchShape split_launch_shape(int64_t n, size_t gsz);   // flat: one workgroup per slab and one for the ragged end
size_t split_lds_bytes(const Program& pr);
void launch_flat_split(const StepArgs& a, const Program& pr, bool bf16, unsigned blocks, int copies, hipStream_t s);
void launch_plan_split(const PlanArgs& a, const Program& pr, bool bf16, unsigned blocks, int copies, hipStream_t s);
void launch_lars_norms_split(const LarsArgs& a, const Program& pr, bool bf16, unsigned blocks, hipStream_t s);
void launch_lars_update_split(const LarsArgs& a, unsigned blocks, hipStream_t s);

}  // namespace lsgd
