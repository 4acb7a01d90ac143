// Launches of the split step kernels.
#include "lsgd_split.hpp"

#include "lsgd_split_host.hpp"

namespace lsgd {

namespace {

// The program's batches must fit 64 KB of LDS, so that two workgroups of 16
// waves share a compute unit.
constexpr int kSplitMaxBatches = 64;

// A caller that sets more than one pass per workgroup gets the kernels the
// setting is about.
bool split_allowed(int n_batches) { return n_batches <= kSplitMaxBatches && launch_passes_per_block() == 1; }

}  // namespace

bool use_split_flat(int64_t n, int32_t n_workers, bool bf16, bool compile_time, int64_t copy_bytes, int n_batches) {
    return split_serves(n, n_workers, bf16, compile_time, copy_bytes) && split_allowed(n_batches);
}

bool split_plan_allowed(int n_batches) { return split_allowed(n_batches); }

// A copy pass of its own costs a launch (2.5 to 4 us): up to 64 MB of copies
// the split kernel writes them itself. Measured apart / in the kernel, us:
// 4x4 binary32 R = 16, 6 MB 7.6 / 5.2, 38 MB 16.4 / 14.2, 64 MB 25.7 / 25.8;
// 16x8 R = 128, 51 MB 23.3 / 21.0, 102 MB 47.4 / 45.3, 154 MB 57.8 / 62.3;
// 2x2 R = 128, 51 MB 16.4 / 12.6, 102 MB 23.9 / 24.5, 307 MB 54.5 / 62.6.
constexpr int64_t kSplitCopyBytes = int64_t{64} << 20;

bool separate_copy_out_small(int64_t n, int64_t copy_bytes, bool apart) {
    if (lsgd_get_copy_out_mode() != LSGD_COPY_OUT_AUTO) return apart;
    return apart && n * copy_bytes > kSplitCopyBytes;
}

// A wave per batch, and for many copies (replicas, broadcast gradients) a wave
// for every eight of them, up to kSplitWaves.
int split_waves(const Program& pr, int copies) {
    return std::min(kSplitWaves, std::max(pr.n_batches, (copies + 7) / 8));
}

// A slot per batch; the broadcast of the mean gradient uses two.
size_t split_lds_bytes(const Program& pr) {
    return static_cast<size_t>(std::max(2, pr.n_batches)) * 64 * sizeof(f32x4);
}

LaunchShape split_launch_shape(int64_t n, size_t gsz) {
    const int64_t full = n / kSplitVec;
    const int64_t slabs = (full + kSplitUnits - 1) / kSplitUnits + (n % kSplitVec != 0);
    return pad_for_xcd_chunk(std::min(slabs, stride_grid_cap()), static_cast<int64_t>(gsz) * kSplitElems);
}

void launch_flat_split(const StepArgs& a, const Program& pr, bool bf16, unsigned blocks, int copies, hipStream_t s) {
    FlatProgArgs sa;
    sa.a = a;
    sa.pr = pr;
    const dim3 threads(64 * split_waves(pr, copies));
    if (bf16) hipLaunchKernelGGL(step_flat_split<uint16_t>, dim3(blocks), threads, split_lds_bytes(pr), s, sa);
    else hipLaunchKernelGGL(step_flat_split<float>, dim3(blocks), threads, split_lds_bytes(pr), s, sa);
}

void launch_plan_split(const PlanArgs& a, const Program& pr, bool bf16, unsigned blocks, int copies, hipStream_t s) {
    PlanProgArgs sa;
    sa.a = a;
    sa.pr = pr;
    const dim3 threads(64 * split_waves(pr, copies));
    if (bf16) hipLaunchKernelGGL(step_plan_split<uint16_t>, dim3(blocks), threads, split_lds_bytes(pr), s, sa);
    else hipLaunchKernelGGL(step_plan_split<float>, dim3(blocks), threads, split_lds_bytes(pr), s, sa);
}

void launch_lars_norms_split(const LarsArgs& a, const Program& pr, bool bf16, unsigned blocks, hipStream_t s) {
    LarsProgArgs sa;
    sa.la = a;
    sa.pr = pr;
    const dim3 threads(64 * split_waves(pr, 0));
    if (bf16) hipLaunchKernelGGL(lars_norms_split<uint16_t>, dim3(blocks), threads, split_lds_bytes(pr), s, sa);
    else hipLaunchKernelGGL(lars_norms_split<float>, dim3(blocks), threads, split_lds_bytes(pr), s, sa);
}

void launch_lars_update_split(const LarsArgs& a, unsigned blocks, hipStream_t s) {
    hipLaunchKernelGGL(lars_update_split, dim3(blocks), dim3(kBlock), 0, s, a);
}

}  // namespace lsgd
