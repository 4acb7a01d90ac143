// Launches of the stream step kernels.
#include "lsgd_stream.hpp"

namespace lsgd {

namespace {

// LDS of the stack: a lane tile is 16 floats.
size_t stack_bytes(const Program& pr) { return static_cast<size_t>(pr.stack_depth) * 16 * sizeof(float) * kBlock; }
static_assert(StreamTile<float>::U * Unit<float>::VEC == 16 && StreamTile<uint16_t>::U * Unit<uint16_t>::VEC == 16, "");

}  // namespace

void launch_flat_stream(const StepArgs& a, const Program& pr, bool bf16, bool cached, unsigned blocks, hipStream_t s) {
    FlatProgArgs fa;
    fa.a = a;
    fa.pr = pr;
    const auto k = bf16 ? (cached ? step_flat_stream<uint16_t, 1> : step_flat_stream<uint16_t, 0>)
                        : (cached ? step_flat_stream<float, 1> : step_flat_stream<float, 0>);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kBlock), stack_bytes(pr), s, fa);
}

void launch_plan_stream(const PlanArgs& a, const Program& pr, bool bf16, bool cached, unsigned blocks, hipStream_t s) {
    PlanProgArgs pa;
    pa.a = a;
    pa.pr = pr;
    const auto k = bf16 ? (cached ? step_plan_stream<uint16_t, 1> : step_plan_stream<uint16_t, 0>)
                        : (cached ? step_plan_stream<float, 1> : step_plan_stream<float, 0>);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kBlock), stack_bytes(pr), s, pa);
}

void launch_mean_stream(const MeanArgs& a, const Program& pr, bool bf16, dim3 blocks, hipStream_t s) {
    MeanProgArgs ma;
    ma.a = a;
    ma.pr = pr;
    const auto k = bf16 ? mean_stream<uint16_t> : mean_stream<float>;
    hipLaunchKernelGGL(k, blocks, dim3(kBlock), stack_bytes(pr), s, ma);
}

int64_t stream_units(int64_t n, bool bf16) {
    const int64_t vec = bf16 ? Unit<uint16_t>::VEC : Unit<float>::VEC, per_tile = kBlock * stream_tile(bf16);
    return n % vec == 0 ? n / vec : (n / vec + per_tile - 1) / per_tile * per_tile + 1;
}

void launch_lars_norms_stream(const LarsArgs& a, const Program& pr, bool bf16, unsigned blocks, hipStream_t s) {
    LarsProgArgs la;
    la.la = a;
    la.pr = pr;
    const auto k = bf16 ? lars_norms_stream<uint16_t> : lars_norms_stream<float>;
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kBlock), stack_bytes(pr), s, la);
}

}  // namespace lsgd
