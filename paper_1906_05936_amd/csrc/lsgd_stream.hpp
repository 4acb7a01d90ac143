// Device code of the stream step: group layouts without a compile-time kernel
// (counts of 9 to 11, 13 to 15, 17 and more, larger groups, unequal groups)
// over vectors and plans of any size.
//
// A lane sums the members of its units batch by batch of the reduction program:
// at most 8 members per batch, whose loads are all in flight at once and whose
// sum is a compile-time tree, so that a member costs one addition per element
// (and, with bfloat16, one operation to widen it). The partial sums of batches
// and groups wait on a stack in LDS, private to the lane. At 8 TB/s a bfloat16
// element leaves about 12 vector operations; the accumulator in registers that
// this replaced, whose every push visited every level with selects, took more.
// Step of 1.2e7 elements without replicas, that accumulator / now, GB/s:
// bfloat16 10x4 3346 / 5859, 9x8 3699 / 5868, 20x3 3048 / 5885, unequal 2, 3,
// 5, 6 4796 / 5714; binary32 10x4 5394 / 6353, 9x8 6104 / 6405, 20x3 5251 /
// 6309. Bound by memory since: a large copy runs at 6443 GB/s.
//
// binary32 has two forms. Four units per lane (consecutive instructions of a
// wave stay on a buffer's pages), the next batch's loads issued before the
// additions in LDS (without that 9x8 ran at 6022 GB/s, with two units at 6019):
// one workgroup per compute unit, so a step takes as long as its fullest unit.
// Two units, nothing issued ahead: two workgroups per unit, which is better for
// few workers and where the last round of four-unit tiles leaves most units
// idle (stream_two_units, lsgd_rules.hpp). bfloat16: two units (one: 10x4 5775,
// 20x3 5675); issuing ahead took 256 registers and cost it 7 to 17%.
//
// A lane whose units lie beyond the end loads the last whole unit again and
// stores nothing; the ragged end is a tile of its own, one element per lane.
#pragma once

#include "lsgd_batches.hpp"
#include "lsgd_stream_host.hpp"

#pragma clang fp contract(off)

namespace lsgd {

// Whether a lane tile of U units issues the next batch's loads ahead.
template <typename GT, int U>
constexpr bool stream_ahead() { return sizeof(GT) == 4 && U == 4; }

// A lane tile: its units' (or, tail, its element's) first elements, clamped
// into the buffer, and whether each is the lane's to store.
template <int U>
struct Tile {
    int64_t e[U];
    bool own[U];
    bool tail;
};

// Tile `t` (kBlock * U units) of the elements [start, start + len); whole
// units first, then, where len is not a multiple of VEC, the ragged end.
template <int U, int VEC>
__device__ __forceinline__ Tile<U> tile_at(int64_t start, int64_t len, int64_t t) {
    const int64_t full = len / VEC;
    const int rem = static_cast<int>(len - full * VEC);
    const int64_t tiles = (full + kBlock * U - 1) / (kBlock * U);
    Tile<U> r;
    r.tail = t >= tiles;
#pragma unroll
    for (int q = 0; q < U; ++q) {
        if (r.tail) {
            const int lane = static_cast<int>(threadIdx.x);
            r.own[q] = q == 0 && lane < rem;
            r.e[q] = start + full * VEC + min(lane, rem - 1);
        } else {
            const int64_t u = t * (kBlock * U) + q * kBlock + threadIdx.x;
            r.own[q] = u < full;
            r.e[q] = start + (u < full ? u : full - 1) * VEC;
        }
    }
    return r;
}

__device__ __forceinline__ constexpr int64_t tile_count(int64_t len, int vec, int tile) {
    const int64_t full = len / vec;
    return (full + kBlock * tile - 1) / (kBlock * tile) + (len != full * vec);
}

template <typename GT>
__device__ __forceinline__ u32x4 load_element(const void* g, int64_t e) {
    const GT* p = static_cast<const GT*>(g) + e;
    if constexpr (sizeof(GT) == 4) return u32x4{*gload_ptr<uint32_t>(p), 0, 0, 0};
    else return u32x4{*gload_ptr<uint16_t>(p), 0, 0, 0};
}

// The mean gradient of a lane tile. stk: this workgroup's LDS, slot s of a
// lane at (s * T/4 + part) * kBlock + thread (conflict-free 128-bit accesses).
// kAhead: the next batch's loads are issued before the additions in LDS.
template <typename GT, int U, bool kAhead, typename Src>
__device__ __forceinline__ void stream_mean(const Src& s, const Program& pr, const Tile<U>& t, f32x4* stk,
                                            float (&x)[U * Unit<GT>::VEC]) {
    constexpr int VEC = Unit<GT>::VEC;
    constexpr int T = U * VEC;
    const float scale = pr.group_scale, div = pr.group_div;
    int sp = static_cast<int>(threadIdx.x);   // the stack's top, as an index of stk
    auto add_top = [&] {
        sp -= (T / 4) * kBlock;
#pragma unroll
        for (int h = 0; h < T / 4; ++h) {
            const f32x4 y = stk[sp + h * kBlock];
            x[4 * h] = y.x + x[4 * h];
            x[4 * h + 1] = y.y + x[4 * h + 1];
            x[4 * h + 2] = y.z + x[4 * h + 2];
            x[4 * h + 3] = y.w + x[4 * h + 3];
        }
    };
    // the first `count` (at most the array's length) members from `first`
    auto load = [&](int first, int count, auto& r) {
        constexpr int K = sizeof(r) / sizeof(r[0]);
        if (!t.tail) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (k < count) {
                    const void* g = s.grad(first + k);
#pragma unroll
                    for (int q = 0; q < U; ++q) r[k][q] = load_raw<GT>(g, t.e[q]);
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (k < count) {
                    r[k][0] = load_element<GT>(s.grad(first + k), t.e[0]);
#pragma unroll
                    for (int q = 1; q < U; ++q) r[k][q] = r[k][0];
                }
            }
        }
    };
    u32x4 ahead[kAhead ? kBatchMembers : 1][U];
    const int nb = pr.n_batches;
    Batch w = pr.batch[0];
    if constexpr (kAhead) load(w.first, w.count, ahead);
    for (int b = 0; b < nb; ++b) {
        with_batch(w.count, w.sub, [&](auto cnt, auto sub) {
            constexpr int CNT = decltype(cnt)::value, SUB = decltype(sub)::value;
            auto sum = [&](const auto& r) {
                batch_sum<CNT, SUB, T>([&](int k, float (&y)[T]) {
#pragma unroll
                    for (int q = 0; q < U; ++q) widen<GT>(r[k][q], slice<VEC, T>(y, q));
                }, scale, div, x);
            };
            if constexpr (kAhead) {
                sum(ahead);
            } else {
                u32x4 r[CNT][U];
                load(w.first, CNT, r);
                sum(r);
            }
        });
        const Batch v = w;
        if (b + 1 < nb) {
            w = pr.batch[b + 1];
            if constexpr (kAhead) load(w.first, w.count, ahead);
        }
        for (int i = 0; i < v.pre; ++i) add_top();
        if (v.div) divide_group<T>(x, scale, div);
        for (int i = 0; i < v.post; ++i) add_top();
        if (b + 1 < nb) {
#pragma unroll
            for (int h = 0; h < T / 4; ++h) stk[sp + h * kBlock] = f32x4{x[4 * h], x[4 * h + 1], x[4 * h + 2], x[4 * h + 3]};
            sp += (T / 4) * kBlock;
        }
    }
    if (pr.total_div != 1.f) {
#pragma unroll
        for (int v = 0; v < T; ++v) x[v] = x[v] / pr.total_div;
    }
}

// The mean of a run of inputs whose count has no compile-time kernel: `pr` is
// the program of one group of that many members, `first` the run's first input.
struct MeanProgArgs {
    MeanArgs a;
    Program pr;
};

struct MeanSrc {
    const MeanArgs& a;
    int first;
    __device__ const void* grad(int k) const { return a.in[first + k]; }
};

// U units per lane, kAhead as for stream_mean: mean_stream_form's choice for
// binary32; one unit and nothing ahead for bfloat16 (9 inputs, n = 1e5, two units
// / one 7.5 / 5.4 us, 1e7 57.9 / 53.7; 64 inputs 1e5 16.8 / 11.2).
template <typename GT, int U, bool kAhead>
__global__ __launch_bounds__(kBlock) void mean_stream(MeanProgArgs ma) {
    extern __shared__ f32x4 stream_lds[];
    constexpr int VEC = Unit<GT>::VEC;
    constexpr int T = U * VEC;
    const MeanArgs& a = ma.a;
    const MeanSrc s{a, static_cast<int>(blockIdx.y) * a.W};
    float* out = a.out[blockIdx.y];
    const int64_t tiles = tile_count(a.n, VEC, U);
    for (int64_t base = static_cast<int64_t>(logical_block(blockIdx.x, a.xcd_chunk)) * a.upl; base < tiles;
         base += static_cast<int64_t>(gridDim.x) * a.upl) {
        for (uint32_t i = 0; i < a.upl && base + i < tiles; ++i) {
            const Tile<U> t = tile_at<U, VEC>(0, a.n, base + i);
            float g[T];
            stream_mean<GT, U, kAhead>(s, ma.pr, t, stream_lds, g);
            if (t.tail) {
                if (t.own[0]) gstore_ptr<float>(out)[t.e[0]] = g[0];
                continue;
            }
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (t.own[q]) store_f32<VEC, false>(out, t.e[q], VEC, slice<VEC, T>(g, q));
        }
    }
}

// One lane tile of the fused step.
template <typename GT, int U, typename Src>
__device__ __forceinline__ void stream_step_tile(const Src& s, const Program& pr, const Tile<U>& t, f32x4* stk) {
    constexpr int VEC = Unit<GT>::VEC;
    constexpr int T = U * VEC;
    if (t.tail) {   // one element per lane
        float g[T];
        stream_mean<GT, U, stream_ahead<GT, U>()>(s, pr, t, stk, g);
        if (!t.own[0]) return;
        const int64_t e = t.e[0];
        float g1[1] = {g[0]}, p[1] = {gload_ptr<float>(s.p())[e]}, m[1] = {gload_ptr<float>(s.m())[e]};
        if constexpr (sizeof(GT) == 4)
            for (int k = 0; k < s.bcast_grad(); ++k) gstore_ptr<float>(const_cast<void*>(s.grad(k)))[e] = g1[0];
        sgd_update<1>(s.hyper(), g1, p, m);
        gstore_ptr<float>(s.p())[e] = p[0];
        gstore_ptr<float>(s.m())[e] = m[0];
        const int rdt = s.rdt();
        for (int r = 0; r < s.n_replicas(); ++r) {
            if (rdt == kF32) gstore_ptr<float>(s.replica(r))[e] = p[0];
            else gstore_ptr<uint16_t>(s.replica(r))[e] = static_cast<uint16_t>(f32_to_bf16_bits(p[0]));
        }
        return;
    }
    float p[T], m[T], g[T];
    load_state<VEC, U, false>(s, t.e, VEC, p, m);   // their latency overlaps the gradient stream
    stream_mean<GT, U, stream_ahead<GT, U>()>(s, pr, t, stk, g);
    sgd_update<T>(s.hyper(), g, p, m);
    // a lane's units past the end are its last ones: q units are its own
#pragma unroll
    for (int q = 0; q < U; ++q) {
        if (!t.own[q]) break;
        const int64_t e[1] = {t.e[q]};
        broadcast_mean<GT, 1, false>(s, e, VEC, slice<VEC, T>(g, q));
    }
    if (t.own[U - 1]) {
        store_state<VEC, U, false>(s, t.e, VEC, p, m);
    } else {
#pragma unroll
        for (int q = 0; q + 1 < U; ++q) {
            const int64_t e[1] = {t.e[q]};
            if (t.own[q]) store_state<VEC, 1, false>(s, e, VEC, slice<VEC, T>(p, q), slice<VEC, T>(m, q));
        }
    }
}

template <typename GT, int U, int CACHED>
__global__ __launch_bounds__(kBlock) void step_flat_stream(FlatProgArgs fa) {
    extern __shared__ f32x4 stream_lds[];
    constexpr int VEC = Unit<GT>::VEC;
    const StepArgs& a = fa.a;
    const FlatSrcT<CACHED> s{a, resolve_hyper(a.h, a.lr_ptr)};
    const int64_t tiles = tile_count(a.n, VEC, U);
    for (int64_t base = static_cast<int64_t>(logical_block(blockIdx.x, a.xcd_chunk)) * a.upl; base < tiles;
         base += static_cast<int64_t>(gridDim.x) * a.upl)
        for (uint32_t q = 0; q < a.upl && base + q < tiles; ++q)
            stream_step_tile<GT, U>(s, fa.pr, tile_at<U, VEC>(0, a.n, base + q), stream_lds);
}

template <typename GT, int U, int CACHED>
__global__ __launch_bounds__(kBlock) void step_plan_stream(PlanProgArgs pa) {
    extern __shared__ f32x4 stream_lds[];
    constexpr int VEC = Unit<GT>::VEC;
    for_plan_chunks<CACHED>(pa.a, [&](const PlanSrcT<CACHED>& s, const PlanChunk& ch, int32_t) {
        const int64_t tiles = tile_count(ch.len, VEC, U);
        for (int64_t t = 0; t < tiles; ++t)
            stream_step_tile<GT, U>(s, pa.pr, tile_at<U, VEC>(ch.start, ch.len, t), stream_lds);
    });
}

// LARS pass 1: the mean gradient to the scratch and the piece's sums of
// squares. Two units per lane and no loads ahead for either type, so that
// several waves per SIMD cover one another's reductions (binary32 with the
// step's form, one wave per SIMD: 8x4 409 us for the whole LARS step, now 361).
template <typename GT>
__global__ __launch_bounds__(kBlock) void lars_norms_stream(LarsProgArgs sa) {
    extern __shared__ f32x4 stream_lds[];
    __shared__ double sums[kBlock / 64][2];
    constexpr int U = kLarsStreamTile;
    constexpr int VEC = Unit<GT>::VEC;
    constexpr int T = U * VEC;
    const LarsArgs& la = sa.la;
    for_plan_chunks(la.pa, [&](const PlanSrc& s, const PlanChunk& ch, int32_t c) {
        float* gb = la.gbar + read_table(&la.gbar_off[ch.tensor]);
        double sp = 0.0, sg = 0.0;
        const int64_t tiles = tile_count(ch.len, VEC, U);
        for (int64_t i = 0; i < tiles; ++i) {
            const Tile<U> t = tile_at<U, VEC>(ch.start, ch.len, i);
            float g[T];
            stream_mean<GT, U, false>(s, sa.pr, t, stream_lds, g);
            if (t.tail) {
                if (t.own[0]) {
                    const float p1[1] = {gload_ptr<float>(s.p())[t.e[0]]}, g1[1] = {g[0]};
                    gstore_ptr<float>(gb)[t.e[0]] = g1[0];
                    lars_accumulate<1>(p1, g1, 1, sp, sg);
                }
                continue;
            }
            // all units' parameters in one go (addresses past the end are
            // clamped): one after the other they cost a memory latency each
            float p[T];
#pragma unroll
            for (int q = 0; q < U; ++q) load_f32_cached<VEC, false>(s.p(), t.e[q], VEC, slice<VEC, T>(p, q));
#pragma unroll
            for (int q = 0; q < U; ++q) {
                if (!t.own[q]) continue;
                store_f32_cached<VEC, false>(gb, t.e[q], VEC, slice<VEC, T>(g, q));
                lars_accumulate<VEC>(slice<VEC, T>(p, q), slice<VEC, T>(g, q), VEC, sp, sg);
            }
        }
        block_sum2(sp, sg, sums);
        if (threadIdx.x == 0) {
            la.partials[2 * static_cast<int64_t>(c)] = sp;
            la.partials[2 * static_cast<int64_t>(c) + 1] = sg;
        }
    });
}

}  // namespace lsgd
