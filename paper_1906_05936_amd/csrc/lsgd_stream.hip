// Launches of the stream step kernels.
#include "lsgd_rules.hpp"
#include "lsgd_stream.hpp"

namespace lsgd {

namespace {

// LDS of the stack, whose slots hold a lane tile of `floats`.
size_t stack_bytes(const Program& pr, int floats) {
    return static_cast<size_t>(pr.stack_depth) * floats * sizeof(float) * kBlock;
}

static_assert(kMaxStack * 16 * sizeof(float) * kBlock <= 160 * 1024, "the deepest stack fits a compute unit's LDS");

template <int CACHED>
auto pick_flat_stream(bool bf16, int tile) {
    if (bf16) return step_flat_stream<uint16_t, 2, CACHED>;
    return tile == 2 ? step_flat_stream<float, 2, CACHED> : step_flat_stream<float, 4, CACHED>;
}

template <int CACHED>
auto pick_plan_stream(bool bf16, int tile) {
    if (bf16) return step_plan_stream<uint16_t, 2, CACHED>;
    return tile == 2 ? step_plan_stream<float, 2, CACHED> : step_plan_stream<float, 4, CACHED>;
}

}  // namespace

void launch_flat_stream(const StepArgs& a, const Program& pr, bool bf16, bool cached, int tile, unsigned blocks,
                        hipStream_t s) {
    FlatProgArgs fa;
    fa.a = a;
    fa.pr = pr;
    const auto k = cached ? pick_flat_stream<1>(bf16, tile) : pick_flat_stream<0>(bf16, tile);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kBlock), stack_bytes(pr, tile * (bf16 ? 8 : 4)), s, fa);
}

void launch_plan_stream(const PlanArgs& a, const Program& pr, bool bf16, bool cached, int tile, unsigned blocks,
                        hipStream_t s) {
    PlanProgArgs pa;
    pa.a = a;
    pa.pr = pr;
    const auto k = cached ? pick_plan_stream<1>(bf16, tile) : pick_plan_stream<0>(bf16, tile);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kBlock), stack_bytes(pr, tile * (bf16 ? 8 : 4)), s, pa);
}

void launch_mean_stream(const MeanArgs& a, const Program& pr, bool bf16, dim3 blocks, hipStream_t s) {
    MeanProgArgs ma;
    ma.a = a;
    ma.pr = pr;
    const MeanForm form = mean_stream_form(a.W, a.n);
    const auto k = bf16                           ? mean_stream<uint16_t, 1, false>
                   : form == MeanForm::kOne       ? mean_stream<float, 1, false>
                   : form == MeanForm::kOneAhead ? mean_stream<float, 1, true>
                                                  : mean_stream<float, 4, true>;
    hipLaunchKernelGGL(k, blocks, dim3(kBlock), stack_bytes(pr, mean_stream_tile(a.W, a.n, bf16) * (bf16 ? 8 : 4)), s, ma);
}

int64_t stream_units(int64_t n, bool bf16, int tile) {
    const int64_t vec = bf16 ? Unit<uint16_t>::VEC : Unit<float>::VEC, per_tile = kBlock * tile;
    return n % vec == 0 ? n / vec : (n / vec + per_tile - 1) / per_tile * per_tile + 1;
}

void launch_lars_norms_stream(const LarsArgs& a, const Program& pr, bool bf16, unsigned blocks, hipStream_t s) {
    LarsProgArgs la;
    la.la = a;
    la.pr = pr;
    const auto k = bf16 ? lars_norms_stream<uint16_t> : lars_norms_stream<float>;
    hipLaunchKernelGGL(k, dim3(blocks), dim3(kBlock), stack_bytes(pr, kLarsStreamTile * (bf16 ? 8 : 4)), s, la);
}

}  // namespace lsgd
