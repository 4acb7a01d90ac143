// Multi-tensor plans of liblsgd: the fused step over a list of parameter
// tensors (a model's per-layer tensors) in one kernel launch.
//
// lsgd_plan_create cuts every tensor into pieces of 2048 elements (times the
// launch shape's passes per workgroup at plan creation, 1 by default), starting
// on unit boundaries, and, where the step or LARS norms kernel's lane tile makes
// a workgroup cover 4096, into pieces of that size too. One workgroup runs one
// piece (a large tensor is walked exactly like the flat kernel walks a vector);
// pieces are taken in the XCD-chunked order of the launch shape. The copy-out
// pass always takes the 2048-element pieces, one lane tile of its own: over
// pieces of 4096 a workgroup made two trips one after the other (binary32, n =
// 2.5e7, R = N, us: 8x8 plan 2383 -> 2230, 10x4 LARS 1643 -> 1574). The LARS
// update takes the pieces of the norms: a workgroup then reads the mean gradient
// from the L2 cache of the XCD that wrote it.
#include <string.h>

#include <algorithm>

#include "lsgd_host.hpp"
#include "lsgd_np2.hpp"
#include "lsgd_plan_kernels.hpp"
#include "lsgd_pow2.hpp"
#include "lsgd_rules.hpp"
#include "lsgd_split_host.hpp"
#include "lsgd_stream_host.hpp"

// One way to cut the plan's tensors: n pieces of `piece` elements in device memory.
struct PieceTable {
    int32_t n;
    int64_t piece;
    lsgd::PlanChunk* d;
};

struct lsgd_plan {
    int device;
    int32_t n_tensors, n_workers, n_groups, n_replicas;
    int32_t W;   // group size, 0 where the groups' sizes differ
    lsgd_dtype gdt, rdt;
    int32_t stride;
    int64_t total_elems;  // elements of all tensors
    PieceTable small, large;   // pieces of 2048 and of 4096 elements (large.n == 0: no kernel of the plan takes them)
    int step_tile[2];          // units per lane tile of the step kernel: mean of means, paper-literal
    int lars_tile;             // of the LARS norms kernel
    // the split kernels' pieces of at most kSplitElems elements (n_fine == 0:
    // neither the step nor LARS takes them)
    int32_t n_fine;
    lsgd::PlanChunk* d_fine;
    lsgd::Program mean_program, literal_program;
    bool step_fine[2];    // the step runs in the split kernels: mean of means, paper-literal
    bool lars_fine;       // the LARS norms too
    bool lars_merge;      // and the LARS update, which sums each tensor's partials itself
    void** d_ptrs;
    // LARS: per-tensor scratch offsets and chunk ranges, and every buffer's
    // byte range (for the workspace aliasing check)
    int64_t gbar_floats;
    int64_t* d_gbar_off;
    int32_t* d_tensor_chunks;
    uint8_t* d_lars_exclude;   // [n_tensors], zero until lsgd_plan_set_lars_exclude
    std::vector<lsgd::Range>* ranges;
    lsgd::SortedRanges* sorted;
    bool grads_apart;     // no gradient buffer overlaps any other buffer (the gradient broadcast needs that)
};

namespace lsgd {
namespace {

// LARS scratch: each tensor's slice of the mean-gradient scratch starts on a
// 64-float (256-byte) boundary.
constexpr int64_t kGbarAlign = 64;

// A compile-time kernel (null: the stream kernels serve the layout) and the
// units per lane tile it processes.
struct PlanPick {
    PlanKernel kernel;
    int tile;
};

constexpr int64_t kSmallPiece = 2048, kLargePiece = 4096;

// Whether a workgroup's lane tiles of `tile` units cover a large piece.
constexpr bool large_pieces(int tile, bool bf16) {
    return static_cast<int64_t>(kBlock) * tile * (bf16 ? Unit<uint16_t>::VEC : Unit<float>::VEC) > kSmallPiece;
}
static_assert(kSmallPiece % 8 == 0, "pieces must start on unit boundaries");
static_assert(large_pieces(4, false) && !large_pieces(2, false) && large_pieces(2, true) && !large_pieces(1, true), "");

// The plan kernel for (W, G): compile-time for the power-of-two groupings of
// pick_flat (lsgd_flat.hip), with parameters and momentum through the caches
// when `cached`; else none (and tile 0).
template <typename GT>
PlanPick pick_plan(int W, int G, bool cached = false) {
    const PlanKernel k = pick_plan_pow2<GT>(W, G, cached);
    if (k) return PlanPick{k, tile_units<GT>(W * G)};
    if (np2_group_count(G)) {   // group counts 3, 5, 6 and 7 (lsgd_np2.hpp)
        const Np2PlanPick q = pick_plan_np2(W, G, cached, sizeof(GT) == 2);
        if (q.kernel) return PlanPick{q.kernel, q.tile};
    }
    return PlanPick{nullptr, 0};
}

lsgd_status check_device(const lsgd_plan* plan) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != plan->device)
        return fail(LSGD_ERR_HIP, "plan was created on device %d, current device is %d", plan->device, dev);
    return LSGD_OK;
}

// The pieces a kernel with lane tiles of `tile` units takes.
const PieceTable& pieces_for(const lsgd_plan* plan, int tile) {
    return large_pieces(tile, plan->gdt == LSGD_BF16) ? plan->large : plan->small;
}

// Points the arguments at a table's pieces, with the launch shape over them.
void use_pieces(const lsgd_plan* plan, const PieceTable& t, PlanArgs& a, LaunchShape& ls) {
    a.chunks = t.d;
    a.n_chunks = t.n;
    ls = pad_for_xcd_chunk(t.n, (plan->gdt == LSGD_BF16 ? 2 : 4) * t.piece);
    a.xcd_chunk = ls.xcd_chunk;
}

// Kernel arguments of a plan step and the launch shape over the pieces `t`.
PlanArgs plan_args(const lsgd_plan* plan, const PieceTable& t, Hyper h, const float* lr_device, LaunchShape& ls) {
    PlanArgs a;
    memset(&a, 0, sizeof a);
    a.ptrs = plan->d_ptrs;
    a.stride = plan->stride;
    a.n_workers = plan->n_workers;
    a.cached_state = use_cached_state(plan->n_workers, plan->total_elems) ? 1 : 0;   // read by the LARS update
    a.n_replicas = plan->n_replicas;
    a.rdt = static_cast<int32_t>(plan->rdt);
    a.h = h;
    a.lr_ptr = lr_device;
    a.copy_src = 0;                              // the copy-out: p to the replicas
    a.copy_dst = 2 + plan->n_workers;
    use_pieces(plan, t, a, ls);
    return a;
}

// The same over the plan's fine pieces, for the split kernels.
void use_fine_pieces(const lsgd_plan* plan, PlanArgs& a, LaunchShape& ls) {
    a.chunks = plan->d_fine;
    a.n_chunks = plan->n_fine;
    ls = pad_for_xcd_chunk(plan->n_fine, (plan->gdt == LSGD_BF16 ? 2 : 4) * kSplitElems);
    a.xcd_chunk = ls.xcd_chunk;
}

// Replicas per workgroup of the plan's copy-out pass over full pieces (as for
// flat steps: a lane loads 32 bytes of p and stores 32 bytes per tile).
constexpr int kPlanCopyRKF32 = 1, kPlanCopyRKBF16 = 2;

// The copy-out pass of a plan step: one workgroup per piece and replica
// group; a lane tile covers a 2048-element piece (the usual piece size).
template <int VEC, int RK>
lsgd_status launch_copy_pieces(const lsgd_plan* plan, PlanArgs& a, hipStream_t s) {
    constexpr int U = kSmallPiece / (VEC * kBlock);
    static_assert(U >= 1, "at least one unit per lane");
    const PieceTable& t = plan->small;
    a.chunks = t.d;
    a.n_chunks = t.n;
    const int64_t win = copy_window_blocks(4 * t.piece, t.n);
    const int64_t blocks = (t.n + win - 1) / win * ((a.n_replicas + RK - 1) / RK) * win;
    a.win_blocks = static_cast<int32_t>(win);
    a.copy_blocks = blocks;
    const int64_t grid = std::min<int64_t>(blocks, stride_grid_cap());   // the kernel strides over the rest
    hipLaunchKernelGGL((copy_out_plan_rmajor<VEC, U, RK>), dim3(static_cast<unsigned>(grid)), dim3(kBlock), 0, s, a);
    return check_launch("lsgd_step_plan (copy-out)");
}

// The copy-out pass to the a.n_replicas destinations of type a.rdt.
lsgd_status launch_plan_copy_out(const lsgd_plan* plan, PlanArgs& a, hipStream_t s) {
    const int rk = copy_replicas_per_group(plan->total_elems, plan->small.n);
    if (a.rdt == static_cast<int32_t>(LSGD_BF16))
        return rk == 1   ? launch_copy_pieces<8, kPlanCopyRKBF16>(plan, a, s)
               : rk == 2 ? launch_copy_pieces<8, 2 * kPlanCopyRKBF16>(plan, a, s)
                         : launch_copy_pieces<8, 4 * kPlanCopyRKBF16>(plan, a, s);
    return rk == 1   ? launch_copy_pieces<4, kPlanCopyRKF32>(plan, a, s)
           : rk == 2 ? launch_copy_pieces<4, 2 * kPlanCopyRKF32>(plan, a, s)
                     : launch_copy_pieces<4, 4 * kPlanCopyRKF32>(plan, a, s);
}

// The copy passes after a plan step that wrote the first k_step replicas and,
// with the broadcast, the first member's gradient.
lsgd_status launch_plan_copies(const lsgd_plan* plan, PlanArgs& a, int32_t k_step, int32_t bcast_copies, hipStream_t s) {
    if (plan->n_replicas > k_step) {
        a.copy_dst = 2 + plan->n_workers + k_step;
        a.n_replicas = plan->n_replicas - k_step;
        const lsgd_status st = launch_plan_copy_out(plan, a, s);
        if (st != LSGD_OK) return st;
    }
    if (bcast_copies > 0) {   // the first member's gradient (slot 2) to the others (slots 3 ..)
        a.copy_src = 2;
        a.copy_dst = 3;
        a.n_replicas = bcast_copies;
        a.rdt = static_cast<int32_t>(LSGD_F32);
        return launch_plan_copy_out(plan, a, s);
    }
    return LSGD_OK;
}

// LARS pass 2: one workgroup per tensor.
__global__ __launch_bounds__(kBlock) void lars_trust_kernel(LarsArgs la) {
    __shared__ double lds[kBlock / 64][2];
    const int32_t t = static_cast<int32_t>(blockIdx.x);
    if (t >= la.n_tensors) return;
    const float tr = lars_trust(la, t, la.tensor_chunks[t], la.tensor_chunks[t + 1], lds);
    if (threadIdx.x == 0) {
        la.trust[t] = tr;
        if (la.trust_out) la.trust_out[t] = tr;
    }
}

// LARS pass-1 kernels: compile-time (W, G) as for the step, else none.
template <typename GT>
LarsKernel pick_lars(int W, int G) {
    if (const LarsKernel k = pick_lars_pow2<GT>(W, G)) return k;
    return np2_group_count(G) ? pick_lars_np2(W, G, sizeof(GT) == 2) : nullptr;
}

// Units per lane tile of the LARS norms kernel for equal groups (W, G).
template <typename GT>
int lars_norms_tile(int W, int G) { return pick_lars<GT>(W, G) ? lars_tile_units<GT>(W * G, G) : kLarsStreamTile; }

// LARS workspace layout: [gbar scratch | per-chunk partials | trust ratios],
// each part starting on a 256-byte boundary.
struct LarsLayout {
    size_t gbar, partials, trust, total;
};

size_t round256(size_t x) { return (x + 255) / 256 * 256; }

LarsLayout lars_layout(const lsgd_plan* plan) {
    LarsLayout l;
    l.gbar = 0;
    l.partials = round256(static_cast<size_t>(plan->gbar_floats) * sizeof(float));
    l.trust = l.partials + round256(static_cast<size_t>(plan->lars_fine ? plan->n_fine : pieces_for(plan, plan->lars_tile).n) * 2 * sizeof(double));
    l.total = l.trust + round256(static_cast<size_t>(plan->n_tensors) * sizeof(float));
    return l;
}

void free_plan(lsgd_plan* p) {
    if (!p) return;
    if (p->small.d) (void)hipFree(p->small.d);
    if (p->large.d) (void)hipFree(p->large.d);
    if (p->d_fine) (void)hipFree(p->d_fine);
    if (p->d_ptrs) (void)hipFree(p->d_ptrs);
    if (p->d_gbar_off) (void)hipFree(p->d_gbar_off);
    if (p->d_tensor_chunks) (void)hipFree(p->d_tensor_chunks);
    if (p->d_lars_exclude) (void)hipFree(p->d_lars_exclude);
    delete p->ranges;
    delete p->sorted;
    delete p;
}

}  // namespace

// The LARS step of a plan with its scratch at `workspace`. A caller-owned
// workspace is checked for size, alignment and overlap with every buffer of
// the call; a library-owned one (`library_workspace`, the per-device array of
// lsgd_lars_step_plan_noalloc) cannot overlap caller memory, and then the
// call also allocates nothing on the host: trust_out and lr_device are
// checked against the plan's ranges one by one.
lsgd_status lars_step(const lsgd_plan* plan, float lr, float momentum_coef, float weight_decay, float trust_coef,
                      void* workspace, size_t workspace_bytes, bool library_workspace, float* trust_out,
                      const float* lr_device, void* stream) {
    if (!plan) return fail(LSGD_ERR_NULL, "plan is NULL");
    if (!workspace) return fail(LSGD_ERR_NULL, "workspace is NULL");
    const LarsLayout l = lars_layout(plan);
    if (workspace_bytes < l.total)
        return fail(LSGD_ERR_SIZE, "workspace_bytes=%zu < %zu (lsgd_lars_workspace_size)", workspace_bytes, l.total);
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0)
        return fail(LSGD_ERR_ALIGN, "workspace is not 256-byte aligned");
    if (trust_out && (reinterpret_cast<uintptr_t>(trust_out) & 3u) != 0)
        return fail(LSGD_ERR_ALIGN, "trust_out is not 4-byte aligned");
    if (lr_device && (reinterpret_cast<uintptr_t>(lr_device) & 3u) != 0)
        return fail(LSGD_ERR_ALIGN, "lr_device is not 4-byte aligned");
    const uintptr_t tb = reinterpret_cast<uintptr_t>(trust_out);
    const uintptr_t te = tb + static_cast<uintptr_t>(plan->n_tensors) * sizeof(float);
    const uintptr_t lb = reinterpret_cast<uintptr_t>(lr_device);
    const uintptr_t le = lb + sizeof(float);
    lsgd_status st = LSGD_OK;
    auto overlaps = [](uintptr_t b0, uintptr_t e0, uintptr_t b1, uintptr_t e1) { return b0 < e1 && b1 < e0; };
    if (trust_out && lr_device && overlaps(tb, te, lb, le))
        return fail(LSGD_ERR_ALIAS, "written buffer trust_out overlaps lr_device");
    const uintptr_t wb = reinterpret_cast<uintptr_t>(workspace);
    const uintptr_t we = library_workspace ? wb : wb + l.total;   // the library's own overlaps no caller buffer
    const SortedRanges& known = *plan->sorted;
    if (known.overlap(wb, we) || (trust_out && known.overlap(tb, te)) || (lr_device && known.overlap_written(lb, le)) ||
        (trust_out && overlaps(wb, we, tb, te)) || (lr_device && overlaps(wb, we, lb, le))) {
        // some pair does overlap: find and name it
        std::vector<Range> ranges(*plan->ranges);
        ranges.push_back(Range{wb, we, true, "workspace"});
        if (trust_out) ranges.push_back(Range{tb, te, true, "trust_out"});
        if (lr_device) ranges.push_back(Range{lb, le, false, "lr_device"});
        if ((st = check_overlap(ranges)) != LSGD_OK) return st;
    }
    if (plan->W == 0) return fail(LSGD_ERR_GROUPS, "the LARS step needs equal group sizes; this plan's differ");
    if ((st = check_device(plan)) != LSGD_OK) return st;

    LarsArgs la;
    memset(&la, 0, sizeof la);
    LaunchShape ls;
    la.pa = plan_args(plan, pieces_for(plan, plan->lars_tile), Hyper{lr, momentum_coef, weight_decay}, lr_device, ls);
    la.gbar_off = plan->d_gbar_off;
    la.tensor_chunks = plan->d_tensor_chunks;
    char* ws = static_cast<char*>(workspace);
    la.gbar = reinterpret_cast<float*>(ws + l.gbar);
    la.partials = reinterpret_cast<double*>(ws + l.partials);
    la.trust = reinterpret_cast<float*>(ws + l.trust);
    la.trust_out = trust_out;
    la.exclude = plan->d_lars_exclude;
    la.n_tensors = plan->n_tensors;
    la.trust_coef = trust_coef;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const int rsz = plan->rdt == LSGD_BF16 ? 2 : 4;
    if (plan->lars_fine) {
        LarsArgs fa = la;
        LaunchShape fs;
        use_fine_pieces(plan, fa.pa, fs);
        launch_lars_norms_split(fa, plan->mean_program, plan->gdt == LSGD_BF16, fs.blocks, s);
        if ((st = check_launch("lsgd_lars_step_plan (norms)")) != LSGD_OK) return st;
        if (plan->lars_merge) {
            const bool apart = separate_copy_out_small(plan->total_elems, static_cast<int64_t>(plan->n_replicas) * rsz,
                                                       separate_copy_out_update(plan->n_replicas, rsz, true));
            if (apart) fa.pa.n_replicas = 0;
            launch_lars_update_split(fa, fs.blocks, s);
            if ((st = check_launch("lsgd_lars_step_plan (update)")) != LSGD_OK || !apart) return st;
            return launch_plan_copy_out(plan, la.pa, s);
        }
    } else if (plan->small.n > 0) {
        int32_t W = plan->W, G = plan->n_groups;
        if (one_group_form(W, G, false)) {
            W = plan->n_workers;
            G = 1;
        }
        const LarsKernel k1 = plan->gdt == LSGD_BF16 ? pick_lars<uint16_t>(W, G) : pick_lars<float>(W, G);
        if (k1) hipLaunchKernelGGL(k1, dim3(ls.blocks), dim3(kBlock), 0, s, la);
        else launch_lars_norms_stream(la, plan->mean_program, plan->gdt == LSGD_BF16, ls.blocks, s);
        if ((st = check_launch("lsgd_lars_step_plan (norms)")) != LSGD_OK) return st;
    }
    hipLaunchKernelGGL(lars_trust_kernel, dim3(plan->n_tensors), dim3(kBlock), 0, s, la);
    if ((st = check_launch("lsgd_lars_step_plan (trust)")) != LSGD_OK) return st;
    if (plan->small.n == 0) return LSGD_OK;
    // the update reads and writes as lsgd_sgd_step does: the same copy-out rule
    const bool split = separate_copy_out_update(plan->n_replicas, rsz,
                                                use_cached_state(plan->n_workers, plan->total_elems));
    if (split) la.pa.n_replicas = 0;
    hipLaunchKernelGGL(lars_update_kernel<2>, dim3(ls.blocks), dim3(kBlock), 0, s, la);
    if ((st = check_launch("lsgd_lars_step_plan (update)")) != LSGD_OK || !split) return st;
    la.pa.n_replicas = plan->n_replicas;
    return launch_plan_copy_out(plan, la.pa, s);
}

}  // namespace lsgd

using namespace lsgd;

extern "C" {

LSGD_API lsgd_status lsgd_plan_create(lsgd_plan** out, int32_t n_tensors, const int64_t* numel,
                                      float* const* params, float* const* momentum,
                                      const void* const* grads, lsgd_dtype gdt, int32_t n_workers,
                                      const int32_t* group_of_worker, int32_t n_groups,
                                      void* const* replicas, int32_t n_replicas, lsgd_dtype rdt) {
    if (!out) return fail(LSGD_ERR_NULL, "out is NULL");
    *out = nullptr;
    if (n_tensors < 1) return fail(LSGD_ERR_SIZE, "n_tensors=%d < 1", n_tensors);
    if (!numel) return fail(LSGD_ERR_NULL, "numel is NULL");
    std::vector<int32_t> order, gstart;
    lsgd_status st = partition_order(n_workers, group_of_worker, n_groups, order, gstart);
    if (st != LSGD_OK) return st;
    // equal group sizes (the mean-of-means step needs them) give W > 0
    bool equal = true;
    for (int32_t j = 0; j < n_groups; ++j) equal = equal && gstart[j + 1] - gstart[j] == gstart[1] - gstart[0];
    if (gdt != LSGD_F32 && gdt != LSGD_BF16) return fail(LSGD_ERR_DTYPE, "gradient dtype %d", (int)gdt);
    if (rdt != LSGD_F32 && rdt != LSGD_BF16) return fail(LSGD_ERR_DTYPE, "replica dtype %d", (int)rdt);
    if (n_replicas < 0 || n_replicas > kMaxReplicas)
        return fail(LSGD_ERR_SIZE, "n_replicas=%d outside [0, %d]", n_replicas, kMaxReplicas);
    if (!params || !momentum || !grads) return fail(LSGD_ERR_NULL, "params, momentum or grads is NULL");
    if (n_replicas > 0 && !replicas) return fail(LSGD_ERR_NULL, "replicas is NULL with n_replicas=%d", n_replicas);

    const size_t gsz = gdt == LSGD_BF16 ? 2 : 4, rsz = rdt == LSGD_BF16 ? 2 : 4;
    const int32_t stride = 2 + n_workers + n_replicas;
    std::vector<void*> table(static_cast<size_t>(n_tensors) * stride, nullptr);
    std::vector<Range> ranges;
    std::vector<PlanChunk> chunks, large_chunks;
    // the kernels' lane tiles, and with them which pieces they take
    const bool bf16 = gdt == LSGD_BF16;
    const int32_t W = equal ? n_workers / n_groups : 0;
    const bool as_one = one_group_form(W, n_groups, false);
    const int32_t tW = as_one ? n_workers : W, tG = as_one ? 1 : n_groups;
    int64_t total_elems = 0, with_elems = 0, small_pieces = 0, four_unit_pieces = 0, ragged = 0;
    for (int32_t t = 0; t < n_tensors; ++t) {
        if (numel[t] < 0) return fail(LSGD_ERR_SIZE, "numel[%d]=%lld < 0", t, static_cast<long long>(numel[t]));
        total_elems += numel[t];
        with_elems += numel[t] > 0;
        ragged += numel[t] % (bf16 ? Unit<uint16_t>::VEC : Unit<float>::VEC) != 0;
        small_pieces += (numel[t] + kSmallPiece - 1) / kSmallPiece;
        four_unit_pieces += (numel[t] + kLargePiece - 1) / kLargePiece;
    }
    auto plan_shape = [&](int32_t w, int32_t g) {
        return PlanShape{total_elems, with_elems, small_pieces, ragged, n_workers, bf16,
                         (bf16 ? pick_plan<uint16_t>(w, g).kernel : pick_plan<float>(w, g).kernel) != nullptr,
                         (g & (g - 1)) == 0, static_cast<int64_t>(n_replicas * rsz)};
    };
    const PlanShape shape = plan_shape(tW, tG);
    auto step_tile = [&](int32_t w, int32_t g) {
        const PlanPick k = bf16 ? pick_plan<uint16_t>(w, g) : pick_plan<float>(w, g);
        return k.kernel ? k.tile : stream_tile(bf16, !bf16 && plan_two_units(shape, four_unit_pieces, device_cus()));
    };
    const int mean_tile = step_tile(tW, tG), literal_tile = as_one ? step_tile(W, n_groups) : mean_tile;
    const int lars_tile = W == 0 ? mean_tile : bf16 ? lars_norms_tile<uint16_t>(tW, tG) : lars_norms_tile<float>(tW, tG);
    const bool need_large = large_pieces(mean_tile, bf16) || large_pieces(literal_tile, bf16) || large_pieces(lars_tile, bf16);
    const int64_t kSmall = kSmallPiece * launch_passes_per_block(), kLarge = kLargePiece * launch_passes_per_block();
    std::vector<int64_t> gbar_off(n_tensors, 0);
    std::vector<int32_t> tensor_chunks(n_tensors + 1, 0);
    int64_t gbar_floats = 0;
    for (int32_t t = 0; t < n_tensors; ++t) {
        const int64_t ne = numel[t];
        tensor_chunks[t] = static_cast<int32_t>(
            std::min<size_t>(large_pieces(lars_tile, bf16) ? large_chunks.size() : chunks.size(), 0x7fffffff));
        gbar_off[t] = gbar_floats;
        gbar_floats += (ne + kGbarAlign - 1) / kGbarAlign * kGbarAlign;
        if (ne == 0) continue;
        void** row = &table[static_cast<size_t>(t) * stride];
        auto add = [&](void* p, size_t esz, bool written, const char* what, int idx) -> lsgd_status {
            if (!p) return fail(LSGD_ERR_NULL, "%s[%d] of tensor %d is NULL", what, idx, t);
            if (!aligned16(p)) return fail(LSGD_ERR_ALIGN, "%s[%d] of tensor %d is not 16-byte aligned", what, idx, t);
            const uintptr_t b = reinterpret_cast<uintptr_t>(p);
            ranges.push_back(Range{b, b + static_cast<uintptr_t>(ne) * esz, written, what});
            return LSGD_OK;
        };
        if ((st = add(params[t], 4, true, "params", t)) != LSGD_OK) return st;
        if ((st = add(momentum[t], 4, true, "momentum", t)) != LSGD_OK) return st;
        row[0] = params[t];
        row[1] = momentum[t];
        for (int32_t k = 0; k < n_workers; ++k) {
            const int32_t w = order[k];
            void* g = const_cast<void*>(grads[static_cast<size_t>(w) * n_tensors + t]);
            if ((st = add(g, gsz, false, "grads", w)) != LSGD_OK) return st;
            row[2 + k] = g;
        }
        for (int32_t r = 0; r < n_replicas; ++r) {
            void* rp = replicas[static_cast<size_t>(r) * n_tensors + t];
            if ((st = add(rp, rsz, true, "replicas", r)) != LSGD_OK) return st;
            row[2 + n_workers + r] = rp;
        }
        // every piece but a tensor's last has the full length (a multiple of the unit)
        for (int64_t s0 = 0; s0 < ne; s0 += kSmall)
            chunks.push_back(PlanChunk{params[t], t, 0, s0, std::min(kSmall, ne - s0)});
        if (need_large)
            for (int64_t s0 = 0; s0 < ne; s0 += kLarge)
                large_chunks.push_back(PlanChunk{params[t], t, 0, s0, std::min(kLarge, ne - s0)});
    }
    if ((st = check_overlap(ranges)) != LSGD_OK) return st;
    Program mean_program, literal_program;
    memset(&mean_program, 0, sizeof mean_program);
    if (equal) build_program(n_groups, gstart.data(), false, mean_program);
    build_program(n_groups, gstart.data(), true, literal_program);
    std::vector<PlanChunk> fine;
    bool step_fine[2] = {false, false}, lars_fine = false, lars_merge = true;
    // An empty tensor's trust ratio has no update workgroup that could write it.
    for (int32_t t = 0; t < n_tensors; ++t)
        if (numel[t] == 0 ||
            (numel[t] / kSplitVec + kSplitUnits - 1) / kSplitUnits + (numel[t] % kSplitVec != 0) > kLarsMergeChunks)
            lars_merge = false;
    if (split_plan_allowed(std::max(mean_program.n_batches, literal_program.n_batches))) {
        step_fine[0] = split_serves_plan(shape);
        step_fine[1] = as_one ? split_serves_plan(plan_shape(W, n_groups)) : step_fine[0];
        lars_fine = split_serves_lars(shape, lars_merge);
    }
    if (step_fine[0] || step_fine[1] || lars_fine) {
        for (int32_t t = 0; t < n_tensors; ++t) {
            if (lars_fine) tensor_chunks[t] = static_cast<int32_t>(fine.size());
            const int64_t whole = numel[t] / kSplitVec * kSplitVec;
            for (int64_t s0 = 0; s0 < whole; s0 += kSplitElems)
                fine.push_back(PlanChunk{params[t], t, 0, s0, std::min<int64_t>(kSplitElems, whole - s0)});
            if (whole < numel[t]) fine.push_back(PlanChunk{params[t], t, 0, whole, numel[t] - whole});
        }
        if (fine.empty()) step_fine[0] = step_fine[1] = lars_fine = false;
    }
    if (chunks.size() > 0x7fffffff || fine.size() > 0x7fffffff) return fail(LSGD_ERR_SIZE, "too many pieces");
    // one workgroup per tensor in the LARS trust kernel, in one launch
    if (n_tensors > kMaxGridBlocks)
        return fail(LSGD_ERR_SIZE, "more than %lld tensors", static_cast<long long>(kMaxGridBlocks));
    tensor_chunks[n_tensors] = static_cast<int32_t>(lars_fine                       ? fine.size()
                                                    : large_pieces(lars_tile, bf16) ? large_chunks.size()
                                                                                    : chunks.size());

    lsgd_plan* p = new lsgd_plan;
    memset(p, 0, sizeof *p);
    if (hipGetDevice(&p->device) != hipSuccess) {
        delete p;
        return fail(LSGD_ERR_HIP, "hipGetDevice failed");
    }
    p->n_tensors = n_tensors;
    p->n_workers = n_workers;
    p->n_groups = n_groups;
    p->W = W;
    p->n_replicas = n_replicas;
    p->gdt = gdt;
    p->rdt = rdt;
    p->small = PieceTable{static_cast<int32_t>(chunks.size()), kSmall, nullptr};
    p->large = PieceTable{static_cast<int32_t>(large_chunks.size()), kLarge, nullptr};
    p->step_tile[0] = mean_tile;
    p->step_tile[1] = literal_tile;
    p->lars_tile = lars_tile;
    p->stride = stride;
    p->total_elems = total_elems;
    p->n_fine = static_cast<int32_t>(fine.size());
    p->mean_program = mean_program;
    p->literal_program = literal_program;
    p->step_fine[0] = step_fine[0];
    p->step_fine[1] = step_fine[1];
    p->lars_fine = lars_fine;
    p->lars_merge = lars_merge;
    p->gbar_floats = gbar_floats;
    p->ranges = new std::vector<Range>(ranges);
    p->sorted = new SortedRanges(ranges);
    for (Range& r : ranges)   // sorted already: with every buffer written, any overlap counts
        if (strcmp(r.what, "grads") == 0) r.written = true;
    p->grads_apart = !any_written_overlap(ranges);
    hipError_t e = hipSuccess;
    const size_t table_bytes = table.size() * sizeof(void*);
    auto upload = [&](const std::vector<PlanChunk>& from, PlanChunk** to) {
        if (e != hipSuccess || from.empty()) return;
        e = hipMalloc(to, from.size() * sizeof(PlanChunk));
        if (e == hipSuccess) e = hipMemcpy(*to, from.data(), from.size() * sizeof(PlanChunk), hipMemcpyHostToDevice);
    };
    upload(chunks, &p->small.d);
    upload(large_chunks, &p->large.d);
    upload(fine, &p->d_fine);
    if (e == hipSuccess) e = hipMalloc(&p->d_ptrs, table_bytes);
    if (e == hipSuccess) e = hipMemcpy(p->d_ptrs, table.data(), table_bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMalloc(&p->d_gbar_off, gbar_off.size() * sizeof(int64_t));
    if (e == hipSuccess) e = hipMalloc(&p->d_lars_exclude, static_cast<size_t>(n_tensors));
    if (e == hipSuccess) {
        const std::vector<uint8_t> none(static_cast<size_t>(n_tensors), 0);
        e = hipMemcpy(p->d_lars_exclude, none.data(), none.size(), hipMemcpyHostToDevice);
    }
    if (e == hipSuccess) e = hipMalloc(&p->d_tensor_chunks, tensor_chunks.size() * sizeof(int32_t));
    if (e == hipSuccess)
        e = hipMemcpy(p->d_gbar_off, gbar_off.data(), gbar_off.size() * sizeof(int64_t), hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(p->d_tensor_chunks, tensor_chunks.data(), tensor_chunks.size() * sizeof(int32_t),
                      hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        free_plan(p);
        return fail(LSGD_ERR_HIP, "lsgd_plan_create: %s", hipGetErrorString(e));
    }
    *out = p;
    return LSGD_OK;
}

LSGD_API lsgd_status lsgd_step_plan_ex(const lsgd_plan* plan, float lr, float momentum_coef,
                                       float weight_decay, const lsgd_step_options* options,
                                       void* stream) {
    if (!plan) return fail(LSGD_ERR_NULL, "plan is NULL");
    const lsgd_step_options none = {LSGD_REDUCE_MEAN_OF_MEANS, 0, nullptr};
    const lsgd_step_options& o = options ? *options : none;
    if (o.reduction != LSGD_REDUCE_MEAN_OF_MEANS && o.reduction != LSGD_REDUCE_LITERAL)
        return fail(LSGD_ERR_UNSUPPORTED, "reduction %d", o.reduction);
    const bool literal = o.reduction == LSGD_REDUCE_LITERAL;
    const bool bcast = o.broadcast_grad != 0;
    const float* lr_device = o.lr_device;
    if (!literal && plan->W == 0)
        return fail(LSGD_ERR_GROUPS, "the mean-of-means step needs equal group sizes; this plan's differ");
    if (bcast && plan->gdt != LSGD_F32)
        return fail(LSGD_ERR_DTYPE, "broadcast_grad needs binary32 gradients");
    if (lr_device && (reinterpret_cast<uintptr_t>(lr_device) & 3u) != 0)
        return fail(LSGD_ERR_ALIGN, "lr_device is not 4-byte aligned");
    const uintptr_t lb = reinterpret_cast<uintptr_t>(lr_device);
    const uintptr_t le = lb + sizeof(float);
    if ((bcast && (!plan->grads_apart || (lr_device && plan->sorted->overlap(lb, le)))) ||
        (lr_device && plan->sorted->overlap_written(lb, le))) {   // some pair does overlap: find and name it
        std::vector<Range> ranges(*plan->ranges);
        if (bcast)   // the gradient buffers are written too
            for (Range& r : ranges)
                if (strcmp(r.what, "grads") == 0) r.written = true;
        if (lr_device) ranges.push_back(Range{lb, le, false, "lr_device"});
        lsgd_status st = check_overlap(ranges);
        if (st != LSGD_OK) return st;
    }
    if (plan->small.n == 0) return LSGD_OK;
    lsgd_status st = check_device(plan);
    if (st != LSGD_OK) return st;
    const int tile = plan->step_tile[literal];
    LaunchShape ls;
    PlanArgs a = plan_args(plan, pieces_for(plan, tile), Hyper{lr, momentum_coef, weight_decay}, lr_device, ls);
    a.literal = literal ? 1 : 0;
    if (plan->step_fine[literal]) {
        const Program& pr = literal ? plan->literal_program : plan->mean_program;
        const int rsz = plan->rdt == LSGD_BF16 ? 2 : 4, gsz = plan->gdt == LSGD_BF16 ? 2 : 4;
        const int32_t bcast_copies = bcast ? plan->n_workers - 1 : 0;
        const int64_t copy_bytes = static_cast<int64_t>(plan->n_replicas) * rsz + 4 * bcast_copies;
        const bool apart = separate_copy_out_small(
            plan->total_elems, copy_bytes,
            separate_copy_out_bytes(plan->n_workers, gsz, rsz, copy_bytes, bcast, plan->total_elems, false));
        const int32_t k_step =
            apart ? replicas_in_step(plan->n_workers, plan->n_replicas, gsz, rsz, plan->total_elems, false) : plan->n_replicas;
        PlanArgs fa = a;
        LaunchShape fs;
        use_fine_pieces(plan, fa, fs);
        fa.bcast_grad = bcast ? (apart ? 1 : plan->n_workers) : 0;
        fa.n_replicas = k_step;
        const hipStream_t s = static_cast<hipStream_t>(stream);
        launch_plan_split(fa, pr, gsz == 2, fs.blocks, k_step + fa.bcast_grad, s);
        if ((st = check_launch("lsgd_step_plan")) != LSGD_OK || !apart) return st;
        return launch_plan_copies(plan, a, k_step, bcast_copies, s);
    }
    const bool cached = use_cached_state(plan->n_workers, plan->total_elems);
    // equal groups (W > 0): the compile-time kernels where there is one, for
    // either reduction; the stream kernel otherwise
    PlanKernel k = nullptr;
    int32_t W = plan->W, G = plan->n_groups;
    if (one_group_form(W, G, literal)) {
        W = plan->n_workers;
        G = 1;
    }
    if (W > 0)
        k = plan->gdt == LSGD_BF16 ? pick_plan<uint16_t>(W, G, cached).kernel : pick_plan<float>(W, G, cached).kernel;
    // as for flat steps: the replicas and the broadcast's copies of the mean
    // gradient to the other N - 1 members go to copy passes of their own
    // where the rule takes the separate form
    const int32_t bcast_copies = bcast ? plan->n_workers - 1 : 0;
    const int rsz = plan->rdt == LSGD_BF16 ? 2 : 4, gsz = plan->gdt == LSGD_BF16 ? 2 : 4;
    const bool split = separate_copy_out_bytes(plan->n_workers, gsz, rsz,
                                               static_cast<int64_t>(plan->n_replicas) * rsz + 4 * bcast_copies, bcast,
                                               plan->total_elems, !k);
    a.bcast_grad = bcast ? (split ? 1 : plan->n_workers) : 0;
    // split: the step kernel writes the first k replicas, the copy-out pass the rest
    const int32_t k_step =
        split ? replicas_in_step(plan->n_workers, plan->n_replicas, gsz, rsz, plan->total_elems, !k) : plan->n_replicas;
    a.n_replicas = k_step;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    if (k) hipLaunchKernelGGL(k, dim3(ls.blocks), dim3(kBlock), 0, s, a);
    else launch_plan_stream(a, literal ? plan->literal_program : plan->mean_program, plan->gdt == LSGD_BF16, cached, tile, ls.blocks, s);
    if ((st = check_launch("lsgd_step_plan")) != LSGD_OK || !split) return st;
    return launch_plan_copies(plan, a, k_step, bcast_copies, s);
}

LSGD_API lsgd_status lsgd_plan_copy_out(const lsgd_plan* plan, void* stream) {
    if (!plan) return fail(LSGD_ERR_NULL, "plan is NULL");
    if (plan->small.n == 0 || plan->n_replicas == 0) return LSGD_OK;
    lsgd_status st = check_device(plan);
    if (st != LSGD_OK) return st;
    LaunchShape ls;
    PlanArgs a = plan_args(plan, plan->small, Hyper{0.f, 0.f, 0.f}, nullptr, ls);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    return launch_plan_copy_out(plan, a, s);
}

LSGD_API lsgd_status lsgd_step_plan(const lsgd_plan* plan, float lr, float momentum_coef,
                                    float weight_decay, void* stream) {
    return lsgd_step_plan_ex(plan, lr, momentum_coef, weight_decay, nullptr, stream);
}

LSGD_API lsgd_status lsgd_lars_workspace_size(const lsgd_plan* plan, size_t* bytes) {
    if (!plan) return fail(LSGD_ERR_NULL, "plan is NULL");
    if (!bytes) return fail(LSGD_ERR_NULL, "bytes is NULL");
    *bytes = lars_layout(plan).total;
    return LSGD_OK;
}

LSGD_API lsgd_status lsgd_lars_step_plan(const lsgd_plan* plan, float lr, float momentum_coef,
                                         float weight_decay, float trust_coef, void* workspace,
                                         size_t workspace_bytes, float* trust_out,
                                         const float* lr_device, void* stream) {
    return lsgd::lars_step(plan, lr, momentum_coef, weight_decay, trust_coef, workspace, workspace_bytes, false,
                           trust_out, lr_device, stream);
}

LSGD_API lsgd_status lsgd_plan_set_lars_exclude(lsgd_plan* plan, const uint8_t* exclude) {
    if (!plan) return fail(LSGD_ERR_NULL, "plan is NULL");
    std::vector<uint8_t> flags(static_cast<size_t>(plan->n_tensors), 0);
    if (exclude)
        for (int32_t t = 0; t < plan->n_tensors; ++t) flags[t] = exclude[t] ? 1 : 0;
    lsgd_status st = check_device(plan);
    if (st != LSGD_OK) return st;
    const hipError_t e = hipMemcpy(plan->d_lars_exclude, flags.data(), flags.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return fail(LSGD_ERR_HIP, "lsgd_plan_set_lars_exclude: %s", hipGetErrorString(e));
    return LSGD_OK;
}

LSGD_API void lsgd_plan_destroy(lsgd_plan* plan) { free_plan(plan); }

}  // extern "C"
