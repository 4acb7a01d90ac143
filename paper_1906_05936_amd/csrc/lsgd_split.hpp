// Device code of the split step: for vectors (and plans of tensors) too small
// to fill the chip with one lane tile per workgroup, the members of a lane's
// unit are divided over the waves of its workgroup.
//
// A lane that sums all N members itself takes one memory latency after the
// other (64 bfloat16 gradients of 30,000 elements: 21 us; 128 binary32: 69 us;
// 40 in 10 groups through the accumulator: 43 us), and a small vector has no
// other waves to fill them. Here a workgroup covers 64 units (1 KB of every
// gradient) with up to 16 waves; each wave sums one register batch of the
// reduction program (at most 8 members, all loads in flight at once), parks the
// sum in LDS, and the remaining additions run level by level of the pairwise
// tree, spread over the waves. One wave then holds the mean, updates
// parameters and momentum and all waves write
// the replicas. The ragged end of a vector is a workgroup of its own, one
// element per lane, so that no lane runs a second pass for it.
#pragma once

#include "lsgd_batches.hpp"
#include "lsgd_split_host.hpp"

#pragma clang fp contract(off)

namespace lsgd {

constexpr int kSplitWaves = 16;   // most waves per workgroup

// A lane's four gradient elements as raw bits: 16 or 8 bytes. (Eight bfloat16
// elements per lane took 102 registers, too many for 16 waves per workgroup.)
template <typename GT> struct Raw4;
template <> struct Raw4<float> { using type = u32x4; };
template <> struct Raw4<uint16_t> { using type = u32x2; };

template <typename GT>
__device__ __forceinline__ typename Raw4<GT>::type load_raw4(const void* g, int64_t e, bool tail) {
    const GT* p = static_cast<const GT*>(g) + e;
    typename Raw4<GT>::type r;
    if (!tail) return __builtin_nontemporal_load(gload_ptr<typename Raw4<GT>::type>(p));
    r = 0;
    if constexpr (sizeof(GT) == 4) r.x = *gload_ptr<uint32_t>(p);
    else r.x = *gload_ptr<uint16_t>(p);
    return r;
}

template <typename GT>
__device__ __forceinline__ void widen4(const typename Raw4<GT>::type& r, float (&x)[kSplitVec]) {
    if constexpr (sizeof(GT) == 4) {
        x[0] = __uint_as_float(r.x); x[1] = __uint_as_float(r.y);
        x[2] = __uint_as_float(r.z); x[3] = __uint_as_float(r.w);
    } else {
        x[0] = __uint_as_float(r.x << 16); x[1] = __uint_as_float(r.x & 0xffff0000u);
        x[2] = __uint_as_float(r.y << 16); x[3] = __uint_as_float(r.y & 0xffff0000u);
    }
}

// Where a slab's elements are: 64 units from `start`, of which `live` lanes
// hold one, or (tail) the ragged end, one element per lane.
struct Slab {
    int64_t e;    // this lane's first element
    int live;     // lanes with elements
    bool tail;
};

__device__ __forceinline__ Slab slab_at(int64_t start, int64_t len, int lane) {
    constexpr int VEC = kSplitVec;
    if (len < VEC) return Slab{start + lane, static_cast<int>(len), true};
    const int64_t units = len / VEC;
    return Slab{start + static_cast<int64_t>(lane) * VEC, static_cast<int>(units < kSplitUnits ? units : kSplitUnits), false};
}

// Slot `slot` of the workgroup's LDS: four floats per lane (conflict-free
// 128-bit accesses).
__device__ __forceinline__ void lds_put(f32x4* lds, int slot, int lane, const float (&x)[kSplitVec]) {
    lds[slot * 64 + lane] = f32x4{x[0], x[1], x[2], x[3]};
}
__device__ __forceinline__ void lds_get(const f32x4* lds, int slot, int lane, float (&x)[kSplitVec]) {
    const f32x4 t = lds[slot * 64 + lane];
    x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
}

// The mean gradient of a slab, in LDS slot 0 before the total division. `pr`
// is read with uniform indices. Every wave of the workgroup calls it; it ends
// with a barrier. before_tree() runs once the wave's batches are summed.
template <typename GT, typename Src, typename Before>
__device__ __forceinline__ void split_sum(const Src& s, const Program& pr, const Slab& sl, f32x4* lds, int wave,
                                          int waves, int lane, const Before& before_tree) {
    constexpr int VEC = kSplitVec;
    const float scale = pr.group_scale, div = pr.group_div;
    const bool live = lane < sl.live;
    for (int b = wave; b < pr.n_batches; b += waves) {
        const Batch w = pr.batch[b];
        if (live) {
            float x[VEC];
            with_batch(w.count, w.sub, [&](auto cnt, auto sub) {
                constexpr int CNT = decltype(cnt)::value, SUB = decltype(sub)::value;
                typename Raw4<GT>::type r[CNT];
                if (!sl.tail) {
#pragma unroll
                    for (int q = 0; q < CNT; ++q) r[q] = load_raw4<GT>(s.grad(w.first + q), sl.e, false);
                } else {
#pragma unroll
                    for (int q = 0; q < CNT; ++q) r[q] = load_raw4<GT>(s.grad(w.first + q), sl.e, true);
                }
                batch_sum<CNT, SUB, VEC>([&](int k, float (&y)[VEC]) { widen4<GT>(r[k], y); }, scale, div, x);
            });
            if (w.div && w.pre == 0) divide_group<VEC>(x, scale, div);
            lds_put(lds, b, lane, x);
        }
    }
    before_tree();
    __syncthreads();
    int i0 = 0;
    for (int l = 0; l < pr.n_levels; ++l) {
        const int i1 = pr.level_end[l];
        for (int i = i0 + wave; i < i1; i += waves) {
            const TreeOp o = pr.op[i];
            float x[VEC], y[VEC];
            lds_get(lds, o.dst, lane, x);
            lds_get(lds, o.src, lane, y);
#pragma unroll
            for (int v = 0; v < VEC; ++v) x[v] = x[v] + y[v];
            if (o.div) divide_group<VEC>(x, scale, div);
            lds_put(lds, o.dst, lane, x);
        }
        i0 = i1;
        __syncthreads();
    }
}

// The new parameters in LDS slot 0 to the replicas, spread over the waves.
template <typename Src>
__device__ __forceinline__ void write_replicas(const Src& s, const Slab& sl, bool live, const f32x4* lds, int wave,
                                               int waves, int lane) {
    const int R = s.n_replicas(), rdt = s.rdt();
    if (!live || wave >= R) return;
    float x[kSplitVec];
    lds_get(lds, 0, lane, x);
    for (int r = wave; r < R; r += waves) {
        if (!sl.tail) store_replica<kSplitVec, false>(s.replica(r), rdt, sl.e, kSplitVec, x);
        else if (rdt == kF32) gstore_ptr<float>(s.replica(r))[sl.e] = x[0];
        else gstore_ptr<uint16_t>(s.replica(r))[sl.e] = static_cast<uint16_t>(f32_to_bf16_bits(x[0]));
    }
}

// One slab of the fused step. `first`: the slab's first element, `len` its
// elements (a multiple of VEC, or fewer than VEC at the ragged end).
template <typename GT, typename Src>
__device__ __forceinline__ void split_step_slab(const Src& s, const Program& pr, int64_t first, int64_t len, f32x4* lds) {
    constexpr int VEC = kSplitVec;
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int waves = static_cast<int>(blockDim.x) >> 6;
    const Slab sl = slab_at(first, len, lane);
    const bool live = lane < sl.live;
    float p[VEC], m[VEC];
    split_sum<GT>(s, pr, sl, lds, wave, waves, lane, [&] {
        if (wave == 0 && live) {   // in flight during the additions in LDS
            if (sl.tail) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) p[v] = m[v] = 0.f;
                p[0] = gload_ptr<float>(s.p())[sl.e];
                m[0] = gload_ptr<float>(s.m())[sl.e];
            } else {
                load_f32_cached<VEC, false>(s.p(), sl.e, VEC, p);
                load_f32_cached<VEC, false>(s.m(), sl.e, VEC, m);
            }
        }
    });
    const int R = s.n_replicas(), nb = s.bcast_grad();
    if (wave == 0 && live) {
        float g[VEC];
        lds_get(lds, 0, lane, g);
        if (pr.total_div != 1.f) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) g[v] = g[v] / pr.total_div;
        }
        sgd_update<VEC>(s.hyper(), g, p, m);
        if (sl.tail) {
            gstore_ptr<float>(s.p())[sl.e] = p[0];
            gstore_ptr<float>(s.m())[sl.e] = m[0];
        } else {
            store_f32_cached<VEC, false>(s.p(), sl.e, VEC, p);
            store_f32_cached<VEC, false>(s.m(), sl.e, VEC, m);
        }
        if (R > 0) lds_put(lds, 0, lane, p);
        if (nb > 0) lds_put(lds, 1, lane, g);
    }
    if (R + nb == 0) return;
    __syncthreads();
    write_replicas(s, sl, live, lds, wave, waves, lane);
    if constexpr (sizeof(GT) == 4) {
        if (nb > 0 && live) {
            float x[VEC];
            lds_get(lds, 1, lane, x);
            for (int k = wave; k < nb; k += waves) {
                float* g = static_cast<float*>(const_cast<void*>(s.grad(k)));
                if (!sl.tail) store_f32<VEC, false>(g, sl.e, VEC, x);
                else gstore_ptr<float>(g)[sl.e] = x[0];
            }
        }
    }
}

template <typename GT>
__global__ __launch_bounds__(64 * kSplitWaves) void step_flat_split(FlatProgArgs sa) {
    extern __shared__ f32x4 split_lds[];
    constexpr int VEC = kSplitVec;
    const StepArgs& a = sa.a;
    const FlatSrcT<1> s{a, resolve_hyper(a.h, a.lr_ptr)};
    const int64_t full = a.n / VEC;
    const int64_t slabs = (full + kSplitUnits - 1) / kSplitUnits, rem = a.n - full * VEC;
    for (int64_t i = logical_block(blockIdx.x, a.xcd_chunk); i < slabs + (rem != 0); i += gridDim.x) {
        if (i >= gridDim.x) __syncthreads();   // the slab before is read out of LDS
        const int64_t first = i < slabs ? i * kSplitUnits * VEC : full * VEC;
        split_step_slab<GT>(s, sa.pr, first, i < slabs ? (full * VEC - first) : rem, split_lds);
    }
}

// a.chunks are the plan's fine pieces (at most kSplitElems elements each).
template <typename GT>
__global__ __launch_bounds__(64 * kSplitWaves) void step_plan_split(PlanProgArgs sa) {
    extern __shared__ f32x4 split_lds[];
    bool again = false;
    for_plan_chunks<1>(sa.a, [&](const PlanSrcT<1>& s, const PlanChunk& ch, int32_t) {
        if (again) __syncthreads();   // the piece before is read out of LDS
        again = true;
        split_step_slab<GT>(s, sa.pr, ch.start, ch.len, split_lds);
    });
}

// LARS pass 1 on the fine pieces: the mean gradient to the scratch, and the
// piece's binary64 sums of p^2 and gbar^2 (wave 0; xor butterfly, so in a
// fixed order).
template <typename GT>
__global__ __launch_bounds__(64 * kSplitWaves) void lars_norms_split(LarsProgArgs sa) {
    extern __shared__ f32x4 split_lds[];
    const LarsArgs& la = sa.la;
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int waves = static_cast<int>(blockDim.x) >> 6;
    bool again = false;
    for_plan_chunks<1>(la.pa, [&](const PlanSrcT<1>& s, const PlanChunk& ch, int32_t c) {
        if (again) __syncthreads();
        again = true;
        const Slab sl = slab_at(ch.start, ch.len, lane);
        const bool live = lane < sl.live;
        float p[kSplitVec] = {0.f, 0.f, 0.f, 0.f};
        split_sum<GT>(s, sa.pr, sl, split_lds, wave, waves, lane, [&] {
            if (wave == 0 && live) {
                if (sl.tail) p[0] = gload_ptr<float>(s.p())[sl.e];
                else load_f32_cached<kSplitVec, false>(s.p(), sl.e, kSplitVec, p);
            }
        });
        if (wave != 0) return;
        double sp = 0.0, sg = 0.0;
        if (live) {
            float* gb = la.gbar + read_table(&la.gbar_off[ch.tensor]);
            float g[kSplitVec];
            lds_get(split_lds, 0, lane, g);
            if (sa.pr.total_div != 1.f) {
#pragma unroll
                for (int v = 0; v < kSplitVec; ++v) g[v] = g[v] / sa.pr.total_div;
            }
            if (sl.tail) gstore_ptr<float>(gb)[sl.e] = g[0];
            else store_f32_cached<kSplitVec, false>(gb, sl.e, kSplitVec, g);
            lars_accumulate<kSplitVec>(p, g, sl.tail ? 1 : kSplitVec, sp, sg);
        }
        wave_sum2(sp, sg);
        if (lane == 0) {
            la.partials[2 * static_cast<int64_t>(c)] = sp;
            la.partials[2 * static_cast<int64_t>(c) + 1] = sg;
        }
    });
}

// LARS passes 2 and 3 in one, on the fine pieces: every workgroup sums its
// tensor's partials itself (at most kLarsMergeChunks of them, read through the
// L2; a launch of its own for the trust ratios took 3 to 5 us), then updates
// its piece and writes its replicas.
static __global__ __launch_bounds__(kBlock) void lars_update_split(LarsArgs la) {
    __shared__ double sums[kBlock / 64][2];
    __shared__ float trust_of_tensor;
    __shared__ f32x4 moved[64];
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    for_plan_chunks<1>(la.pa, [&](const PlanSrcT<1>& s, const PlanChunk& ch, int32_t c) {
        const Slab sl = slab_at(ch.start, ch.len, lane);
        const bool live = lane < sl.live;
        float g[kSplitVec] = {}, p[kSplitVec] = {}, m[kSplitVec] = {};
        if (wave == 0 && live) {
            const float* gb = la.gbar + read_table(&la.gbar_off[ch.tensor]);
            if (sl.tail) {
                g[0] = gload_ptr<float>(gb)[sl.e];
                p[0] = gload_ptr<float>(s.p())[sl.e];
                m[0] = gload_ptr<float>(s.m())[sl.e];
            } else {
                load_f32_cached<kSplitVec, false>(gb, sl.e, kSplitVec, g);
                load_f32_cached<kSplitVec, false>(s.p(), sl.e, kSplitVec, p);
                load_f32_cached<kSplitVec, false>(s.m(), sl.e, kSplitVec, m);
            }
        }
        const int32_t c0 = read_table(&la.tensor_chunks[ch.tensor]);
        const int32_t c1 = read_table(&la.tensor_chunks[ch.tensor + 1]);
        const float trust = lars_trust(la, ch.tensor, c0, c1, sums);
        if (threadIdx.x == 0) {
            trust_of_tensor = trust;
            if (c == c0) {
                la.trust[ch.tensor] = trust;
                if (la.trust_out) la.trust_out[ch.tensor] = trust;
            }
        }
        __syncthreads();
        if (wave == 0 && live) {
            lars_update<kSplitVec>(s.hyper(), trust_of_tensor, g, p, m);
            if (sl.tail) {
                gstore_ptr<float>(s.p())[sl.e] = p[0];
                gstore_ptr<float>(s.m())[sl.e] = m[0];
            } else {
                store_f32_cached<kSplitVec, false>(s.p(), sl.e, kSplitVec, p);
                store_f32_cached<kSplitVec, false>(s.m(), sl.e, kSplitVec, m);
            }
            lds_put(moved, 0, lane, p);
        }
        __syncthreads();
        write_replicas(s, sl, live, moved, wave, kBlock / 64, lane);
        __syncthreads();   // `moved` and `sums` are free for the next piece
    });
}

}  // namespace lsgd
