// Reduction programs: the two-level pairwise mean of a group layout known only
// at run time, written out by the host as a list of register batches and a
// list of additions between their sums. Plain C++, no HIP.
//
// A batch is a run of at most kBatchMembers consecutive entries of the member
// order, summed by one lane in registers with a compile-time tree:
//   - a run of one group that starts at a multiple of kBatchMembers inside the
//     group (sub == 0), or
//   - where every group has the same 1 to 4 members, a power-of-two number of
//     whole groups (sub == the group size): each group's sum is divided, then
//     the quotients are summed.
// PW (the pairwise sum with the largest-power-of-two split) over k terms is PW
// over the sums of its aligned runs of b terms, for every power of two b, so
// the batches' sums are the leaves of the same tree: inside a group that
// starts a batch every kBatchMembers members, and over groups that are packed
// in powers of two.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace lsgd {

constexpr int kBatchMembers = 8;
constexpr int kMaxBatches = 128;   // every batch holds at least one of the kMaxWorkers members
constexpr int kMaxLevels = 16;
// Most partial sums the stack form ever holds: 63 single workers leave six, and
// a group of 57 to 65 members after them three more.
constexpr int kMaxStack = 9;

// One batch, and what the stack form of the program does with its sum:
// `pre` additions of a popped partial sum (earlier partial + sum), a division
// by the group divisor if `div`, `post` more additions, then a push.
struct Batch {
    uint8_t first;        // first member
    uint8_t count : 4;    // members, 1 .. kBatchMembers
    uint8_t sub : 4;      // 0, or the members of each whole group in the batch
    uint8_t pre : 4;
    uint8_t post : 4;
    uint8_t div;          // the batch ends its group (sub == 0)
};

// One addition of the tree form: slot[dst] += slot[src], then a division by
// the group divisor if `div` (the root of a group of several batches). Batches
// that are a whole group are divided when they are summed.
struct TreeOp {
    uint8_t dst, src, div, pad;
};

struct Program {
    int32_t n_batches;
    int32_t n_levels;      // of the tree form; the additions of a level are independent of one another
    int32_t stack_depth;   // most partial sums the stack form holds besides the running one
    float group_div;       // W, or N in the paper-literal reduction
    float group_scale;     // 1 / group_div where that is exact (a power of two), else 0
    float total_div;       // G, or 1 (paper-literal, or one group)
    Batch batch[kMaxBatches];
    TreeOp op[kMaxBatches];
    uint8_t level_end[kMaxLevels];   // level l: ops [level_end[l-1], level_end[l])
};

namespace program_detail {

inline int split_point(int k) {   // largest power of two below k (k >= 2)
    int h = 1;
    while (h * 2 < k) h *= 2;
    return h;
}

struct Builder {
    Program& p;
    int level_of[kMaxBatches];

    // The pairwise tree over `k` nodes whose sums stand in slots slot[0..k);
    // returns the level of its root. `div`: the root is a group's sum.
    int tree(const int* slot, const int* level, int k, bool div) {
        if (k == 1) return level[0];
        const int h = split_point(k);
        const int l = 1 + std::max(tree(slot, level, h, false), tree(slot + h, level + h, k - h, false));
        p.op[n_ops] = TreeOp{static_cast<uint8_t>(slot[0]), static_cast<uint8_t>(slot[h]), static_cast<uint8_t>(div), 0};
        level_of[n_ops++] = l;
        return l;
    }
    int n_ops = 0;
};

inline int trailing_ones(int x) {
    int c = 0;
    while (x & 1) { ++c; x >>= 1; }
    return c;
}

}  // namespace program_detail

// The program of n_groups groups, group j the members [start[j], start[j+1])
// of the member order. `literal`: the paper-literal reduction (each group's
// sum / N, no further division); else the mean of the group means, which needs
// equal group sizes.
inline void build_program(int n_groups, const int32_t* start, bool literal, Program& p) {
    using namespace program_detail;
    const int N = start[n_groups];
    const int W = start[1] - start[0];
    bool equal = true;
    for (int j = 0; j < n_groups; ++j) equal = equal && start[j + 1] - start[j] == W;
    // One member per group under the mean of means: x / 1 = x, so the groups
    // are the terms of one sum, divided by G = N once.
    const int32_t one[2] = {0, N};
    const bool flat = !literal && equal && W == 1;
    const int32_t* gs = flat ? one : start;
    const int G = flat ? 1 : n_groups;
    const int w = flat ? N : W;
    const int div = literal ? N : w;
    p.group_div = static_cast<float>(div);
    p.group_scale = (div & (div - 1)) == 0 ? 1.0f / static_cast<float>(div) : 0.0f;
    p.total_div = literal ? 1.0f : static_cast<float>(G);
    p.n_batches = 0;
    p.stack_depth = 0;
    int root_slot[kMaxBatches], root_level[kMaxBatches];
    Builder b{p, {}};
    int roots = 0, depth = 0;
    // whole groups per batch: the largest power of two that fits
    int pack = 1;
    if (equal && G > 1)
        while (2 * pack * w <= kBatchMembers) pack *= 2;
    auto put = [&](int first, int count, int sub, int pre, bool divide, int post) {
        p.batch[p.n_batches++] = Batch{static_cast<uint8_t>(first), static_cast<uint8_t>(count),
                                       static_cast<uint8_t>(sub), static_cast<uint8_t>(pre),
                                       static_cast<uint8_t>(post), static_cast<uint8_t>(divide)};
        depth -= pre + post;
        ++depth;
        p.stack_depth = std::max(p.stack_depth, depth);
    };
    const int leaves = pack > 1 ? (G + pack - 1) / pack : G;   // of the tree over groups
    for (int j = 0; j < leaves; ++j) {
        const bool last = j + 1 == leaves;
        const int post = last ? __builtin_popcount(static_cast<unsigned>(j)) : trailing_ones(j);
        root_slot[roots] = p.n_batches;
        if (pack > 1) {
            const int g0 = j * pack, g1 = std::min(G, g0 + pack);
            put(g0 * w, (g1 - g0) * w, w, 0, false, post);
            root_level[roots] = 0;
        } else {
            const int m0 = gs[j], m1 = gs[j + 1];
            const int nb = (m1 - m0 + kBatchMembers - 1) / kBatchMembers;
            int slot[kMaxBatches], level[kMaxBatches];
            for (int i = 0; i < nb; ++i) {
                slot[i] = p.n_batches;
                level[i] = 0;
                const bool end = i + 1 == nb;
                put(m0 + i * kBatchMembers, std::min(kBatchMembers, m1 - m0 - i * kBatchMembers), 0,
                    end ? __builtin_popcount(static_cast<unsigned>(i)) : trailing_ones(i), end, end ? post : 0);
            }
            root_level[roots] = b.tree(slot, level, nb, true);
        }
        ++roots;
    }
    b.tree(root_slot, root_level, roots, false);
    // the additions by level, in the order they were made
    p.n_levels = 0;
    for (int i = 0; i < b.n_ops; ++i) p.n_levels = std::max(p.n_levels, b.level_of[i]);
    TreeOp sorted[kMaxBatches];
    int at = 0;
    for (int l = 1; l <= p.n_levels; ++l) {
        for (int i = 0; i < b.n_ops; ++i)
            if (b.level_of[i] == l) sorted[at++] = p.op[i];
        p.level_end[l - 1] = static_cast<uint8_t>(at);
    }
    for (int i = 0; i < at; ++i) p.op[i] = sorted[i];
}

}  // namespace lsgd
