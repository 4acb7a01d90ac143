// Host-side helpers shared by the translation units of liblsgd: error text,
// argument validation, the membership-to-member-order map and launch sizing.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <string>
#include <vector>

#include "lsgd.h"

namespace lsgd {

// Records the detail of a failing call for lsgd_last_error() and returns `st`.
lsgd_status fail(lsgd_status st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// hipGetLastError() after a launch, mapped to LSGD_ERR_HIP with its text.
lsgd_status check_launch(const char* what);

// Subgroup indexing: validates the worker->group map (every id in [0, G), G | N,
// every group of exactly W = N/G members) and returns the member order, G rows
// of W worker ids, each row ascending. Returns LSGD_OK or LSGD_ERR_GROUPS/SIZE.
lsgd_status member_order(int32_t n_workers, const int32_t* group_of_worker, int32_t n_groups,
                         std::vector<int32_t>& order);

// Any partition into non-empty groups (the paper-literal reduction): member
// order grouped by group id, ascending worker id inside a group, and the
// G + 1 group offsets into it. LSGD_ERR_GROUPS for an id out of range or an
// empty group.
lsgd_status partition_order(int32_t n_workers, const int32_t* group_of_worker, int32_t n_groups,
                            std::vector<int32_t>& order, std::vector<int32_t>& group_start);

bool aligned16(const void* p);

// A byte range [begin, end) of one buffer argument; `written` for outputs.
struct Range {
    uintptr_t begin, end;
    bool written;
    const char* what;
};

// LSGD_ERR_ALIAS if a written range overlaps any other range (empty ranges
// never overlap). Sort-and-sweep, O(k log k).
lsgd_status check_overlap(std::vector<Range>& ranges);

// Whether a written range overlaps another, for ranges check_overlap has sorted.
bool any_written_overlap(const std::vector<Range>& sorted);

// Ranges sorted by check_overlap (the plan's, checked at creation), so that a
// step checks the one or two more buffers it is given against all of them
// without sorting them again: the 5474 ranges of a ResNet-50 plan with 16
// workers and replicas took longer to copy and sort than the step to launch.
class SortedRanges {
public:
    SortedRanges() = default;
    explicit SortedRanges(const std::vector<Range>& sorted);
    // Whether [b, e) overlaps any range (any written one).
    bool overlap(uintptr_t b, uintptr_t e) const { return e > b && reaches(max_end_, b, e); }
    bool overlap_written(uintptr_t b, uintptr_t e) const { return e > b && reaches(max_written_end_, b, e); }

private:
    bool reaches(const std::vector<uintptr_t>& max_end, uintptr_t b, uintptr_t e) const;
    std::vector<uintptr_t> begin_, max_end_, max_written_end_;   // prefix maxima over the ranges before
};

// Default launch shape of the planless kernels: automatic XCD chunk (each XCD
// walks kAutoChunkBytes of every buffer per turn), one-shot grids, one pass per
// workgroup. Changed process-wide by lsgd_set_launch_shape.
constexpr int32_t kXcdChunkAuto = -1;
constexpr int64_t kAutoChunkBytes = 512 * 1024;
constexpr int32_t kDefaultXcdChunk = kXcdChunkAuto;
constexpr int32_t kDefaultBlocksPerCu = 0;
constexpr int32_t kDefaultUnitsPerLane = 1;

struct LaunchShape {
    unsigned blocks;     // grid size (padded to a multiple of 8 * xcd_chunk)
    uint32_t xcd_chunk;  // 0 when the grid is too small to renumber
    uint32_t upl;        // consecutive passes of kBlock units per logical block
};

// Grid for `units` 16-byte units processed in lane tiles of `tile` units:
// ceil(units / (kBlock * tile * upl)) workgroups, capped at compute units *
// blocks-per-CU when that is set (the kernels then grid-stride), then padded
// for the XCD chunking.
LaunchShape launch_shape(int64_t units, int tile = 1);

// The launch shape's passes per workgroup (units_per_lane).
int32_t launch_passes_per_block();

// Whether a step with N gradients of gsz bytes, n elements and `copy_bytes`
// bytes per element of copies (replicas of rsz bytes, and the gradient
// broadcast's copies of the mean gradient to the other members) writes them in
// copy passes of their own (lsgd_set_copy_out_mode); `stream`: the step runs in
// a stream kernel.
bool separate_copy_out_bytes(int32_t n_workers, size_t gsz, size_t rsz, int64_t copy_bytes, bool broadcast, int64_t n,
                             bool stream);
// Group counts other than powers of two that have compile-time kernels too
// (lsgd_np2.hpp; 12: the LARS norms only).
inline bool np2_group_count(int G) { return G == 3 || G == 5 || G == 6 || G == 7 || G == 12; }

// One worker per group in a count that is no power of two, under the mean of
// means: the result equals that of one group of all N workers in the same
// member order (the same pairwise sum over the same sequence of values, then
// one division by N = G; the group means are the members themselves), and the
// compile-time kernels take that form (W = N, G = 1): 1e7 elements without
// replicas, as G groups / as one group, us: binary32 5x1 57 / 55, 6x1 64 / 60,
// bfloat16 3x1 38.5 / 37.4, 12x1 81 / 63.
inline bool one_group_form(int32_t W, int32_t G, bool literal) {
    return !literal && W == 1 && G > 1 && (G & (G - 1)) != 0;
}
// With the separate copy-out: how many of the n_replicas replicas (rsz bytes
// each) the step kernel still writes itself; the copy-out pass writes the
// rest (lsgd_set_step_replicas).
int32_t replicas_in_step(int32_t n_workers, int32_t n_replicas, size_t gsz, size_t rsz, int64_t n, bool stream);
// The same for lsgd_sgd_step and the LARS update; `cached`: their parameter
// and momentum accesses go through the caches.
bool separate_copy_out_update(int32_t n_replicas, size_t rsz, bool cached);

// Largest grid of a grid-stride kernel whose XCD assignment must not change
// between strides: kMaxGridBlocks, or the blocks_per_cu cap of
// lsgd_set_launch_shape rounded down to a multiple of 8.
int64_t stride_grid_cap();

// Workgroups per window of the replica-major copy-out pass over `blocks`
// workgroups that each read `block_p_bytes` of p: about 8 MB of p per window,
// windows of equal size, a multiple of 8 workgroups (so that each XCD reads
// the same part of the window for every replica).
int64_t copy_window_blocks(int64_t block_p_bytes, int64_t blocks);

// Grid of exactly `blocks` logical workgroups, each covering `block_bytes` of
// every buffer, padded for the XCD chunking (kernels skip logical blocks
// >= `blocks`).
LaunchShape pad_for_xcd_chunk(int64_t blocks, int64_t block_bytes);

// Compute units of the current device (cached per device).
int device_cus();

// lsgd_lars_step_plan with its scratch at `workspace` (workspace_bytes long);
// `library_workspace`: the scratch is the library's own per-device array
// (lsgd_lars_step_plan_noalloc), which no caller buffer can overlap, and the
// call then makes no host allocation either.
lsgd_status lars_step(const lsgd_plan* plan, float lr, float momentum_coef, float weight_decay, float trust_coef,
                      void* workspace, size_t workspace_bytes, bool library_workspace, float* trust_out,
                      const float* lr_device, void* stream);

}  // namespace lsgd
