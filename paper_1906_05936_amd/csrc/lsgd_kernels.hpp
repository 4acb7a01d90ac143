// Device code of liblsgd: the Layered SGD aggregation and update for gfx950.
//
// Every step is elementwise along the parameter vector, so the kernels stream
// HBM: in the kernels here a lane owns one or more 16-byte "units" of the
// gradient layout (4 binary32 or 8 bfloat16 elements), loads all N worker units
// of each with 128-bit nontemporal loads, reduces them in registers in the fixed
// pairwise order, applies the update and writes parameters, momentum and replicas
// with 128-bit stores. No element is touched by two lanes, so they need no
// atomics, no LDS and no cross-lane reductions. (The stream kernels,
// lsgd_stream.hpp, keep a lane's partial sums in LDS; the split kernels,
// lsgd_split.hpp, divide a unit's members over waves; the LARS norms, in
// lsgd_plan_kernels.hpp, sum squares over a workgroup.)
//
// Rounding contract (matches the header): binary32, one rounding per written
// operation, no contraction into fused multiply-add.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#pragma clang fp contract(off)

namespace lsgd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kMaxWorkers = 128;   // == LSGD_MAX_WORKERS
constexpr int kMaxReplicas = 128;  // == LSGD_MAX_REPLICAS
constexpr int kBlock = 256;        // threads per workgroup (4 wave64)
// A dispatch holds at most 2^32 - 1 work-items; grids stay at or below this
// many workgroups (a multiple of 8, the XCD count).
constexpr int64_t kMaxGridBlocks = (0xffffffffLL / kBlock) / 8 * 8;

enum : int { kF32 = 0, kBF16 = 1 };

// Elements per 16-byte gradient unit. bf16 is carried as its uint16 bits.
template <typename GT> struct Unit;
template <> struct Unit<float> { static constexpr int VEC = 4; };
template <> struct Unit<uint16_t> { static constexpr int VEC = 8; };

// Largest power of two strictly below k (k >= 2): the split point of the
// pairwise sum PW(x[0..k)) = PW(x[0..h)) + PW(x[h..k)).
__host__ __device__ constexpr int pw_split(int k) {
    int h = 1;
    while (h * 2 < k) h *= 2;
    return h;
}

// Workgroups are dispatched to the eight XCDs round-robin by block index (block
// b runs on XCD b % 8). With xcd_chunk = C > 0 the kernels renumber blocks so
// that each XCD runs C consecutive logical blocks per turn: the chip-wide set of
// active addresses stays one contiguous window per buffer, while each XCD walks
// C * 4 KB runs of every buffer, which keeps fewer distinct pages live in that
// XCD's address-translation caches. The host pads the grid to a multiple of
// 8*C so that the renumbering is a bijection on [0, gridDim.x).
__device__ __forceinline__ uint32_t logical_block(uint32_t b, uint32_t chunk) {
    if (chunk == 0) return b;
    const uint32_t x = b & 7u, i = b >> 3;
    return ((i / chunk) * 8u + x) * chunk + (i % chunk);
}

// Runs body(u) for every unit u in [0, units). A logical block owns `upl`
// consecutive passes of kBlock units (one unit per lane per pass), so each
// workgroup walks upl * 4 KB of every buffer in address order; logical blocks
// are taken in XCD-chunked order, grid-stride when the grid is smaller than
// the work.
template <typename Body>
__device__ __forceinline__ void for_units(int64_t units, uint32_t chunk, uint32_t upl,
                                          const Body& body) {
    const int64_t span = static_cast<int64_t>(kBlock) * upl;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * span;
    for (int64_t base = static_cast<int64_t>(logical_block(blockIdx.x, chunk)) * span; base < units;
         base += stride) {
        for (uint32_t q = 0; q < upl; ++q) {
            const int64_t u = base + static_cast<int64_t>(q) * kBlock + threadIdx.x;
            if (u < units) body(u);
        }
    }
}

// Tiled variant of for_units: a lane's tile is U units kBlock apart (so every
// wave instruction still covers 1 KB of one buffer), and a kernel visits each
// buffer once per tile for all U units (stream-major), which keeps consecutive
// instructions of a wave on the same pages and DRAM rows. tile(e0) gets the U
// element offsets of a tile whose units are all complete; unit(u) handles the
// units of the last, partial tile one by one (u < units_all).
template <int U, int VEC, typename TileFn, typename UnitFn>
__device__ __forceinline__ void for_tiles(int64_t units_full, int64_t units_all, uint32_t chunk,
                                          uint32_t upl, const TileFn& tile, const UnitFn& unit) {
    const int64_t tspan = static_cast<int64_t>(kBlock) * U;
    const int64_t span = tspan * upl;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * span;
    for (int64_t base = static_cast<int64_t>(logical_block(blockIdx.x, chunk)) * span; base < units_all;
         base += stride) {
        for (uint32_t pass = 0; pass < upl; ++pass) {
            const int64_t t0 = base + static_cast<int64_t>(pass) * tspan + threadIdx.x;
            if (t0 + static_cast<int64_t>(U - 1) * kBlock < units_full) {
                int64_t e0[U];
#pragma unroll
                for (int q = 0; q < U; ++q) e0[q] = (t0 + static_cast<int64_t>(q) * kBlock) * VEC;
                tile(e0);
            } else {
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const int64_t u = t0 + static_cast<int64_t>(q) * kBlock;
                    if (u < units_all) unit(u);
                }
            }
        }
    }
}

// The q-th VEC-float slice of a tile array.
template <int VEC, int T>
__device__ __forceinline__ float (&slice(float (&x)[T], int q))[VEC] {
    return *reinterpret_cast<float(*)[VEC]>(&x[q * VEC]);
}
template <int VEC, int T>
__device__ __forceinline__ const float (&slice(const float (&x)[T], int q))[VEC] {
    return *reinterpret_cast<const float(*)[VEC]>(&x[q * VEC]);
}

// ---------------------------------------------------------------- loads/stores

// Address-space views. Every buffer the kernels read or write is device
// global memory: accessing it through a global-space pointer gives the
// global_load / global_store forms, also for pointers the kernel itself read
// from a table (for those the compiler would otherwise use the generic flat
// forms). Tables that no kernel writes (the plans' chunk and pointer tables)
// are read through the constant space, so that they become scalar loads
// instead of vector loads the compiler must order after every store.
#define LSGD_GLOBAL __attribute__((address_space(1)))
#define LSGD_CONST __attribute__((address_space(4)))

template <typename T>
__device__ __forceinline__ const LSGD_GLOBAL T* gload_ptr(const void* p) {
    return (const LSGD_GLOBAL T*)(p);
}
template <typename T>
__device__ __forceinline__ LSGD_GLOBAL T* gstore_ptr(void* p) {
    return (LSGD_GLOBAL T*)(p);
}
template <typename T>
__device__ __forceinline__ T read_table(const T* p) {
    return *(const LSGD_CONST T*)(p);
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// binary32 -> bfloat16 bits, nearest-even via the carry of a 0x7fff(+1 if odd)
// bias; NaN is returned as a quiet NaN of the same sign.
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// One gradient unit of a worker, widened to binary32. TAIL units (the ragged end
// of a tensor, cnt < VEC) read element by element and zero-fill the rest.
template <typename GT, bool TAIL>
__device__ __forceinline__ void load_grad(const void* g, int64_t e0, int cnt,
                                          float (&x)[Unit<GT>::VEC]) {
    constexpr int VEC = Unit<GT>::VEC;
    const GT* p = static_cast<const GT*>(g) + e0;
    if constexpr (TAIL) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            if constexpr (sizeof(GT) == 4) x[v] = v < cnt ? gload_ptr<float>(p)[v] : 0.f;
            else x[v] = v < cnt ? bf16_bits_to_f32(gload_ptr<uint16_t>(p)[v]) : 0.f;
        }
    } else if constexpr (sizeof(GT) == 4) {
        f32x4 t = __builtin_nontemporal_load(gload_ptr<f32x4>(p));
        x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
    } else {
        u32x4 t = __builtin_nontemporal_load(gload_ptr<u32x4>(p));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            x[2 * q] = __uint_as_float(t[q] << 16);
            x[2 * q + 1] = __uint_as_float(t[q] & 0xffff0000u);
        }
    }
}

// VEC binary32 values at p + e0 (VEC is 4 or 8: one or two 128-bit accesses).
template <int VEC, bool TAIL>
__device__ __forceinline__ void load_f32(const float* p, int64_t e0, int cnt, float (&x)[VEC]) {
    if constexpr (TAIL) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) x[v] = v < cnt ? gload_ptr<float>(p + e0)[v] : 0.f;
    } else {
#pragma unroll
        for (int q = 0; q < VEC / 4; ++q) {
            f32x4 t = __builtin_nontemporal_load(gload_ptr<f32x4>(p + e0) + q);
            x[4 * q] = t.x; x[4 * q + 1] = t.y; x[4 * q + 2] = t.z; x[4 * q + 3] = t.w;
        }
    }
}

template <int VEC, bool TAIL>
__device__ __forceinline__ void store_f32(float* p, int64_t e0, int cnt, const float (&x)[VEC]) {
    if constexpr (TAIL) {
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            if (v < cnt) gstore_ptr<float>(p + e0)[v] = x[v];
    } else {
#pragma unroll
        for (int q = 0; q < VEC / 4; ++q) {
            f32x4 t = {x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
            __builtin_nontemporal_store(t, gstore_ptr<f32x4>(p + e0) + q);
        }
    }
}

// Plain (cache-allocating) variants, for data that is read again soon: the
// LARS mean-gradient scratch (written by one kernel, read by the next).
template <int VEC, bool TAIL>
__device__ __forceinline__ void load_f32_cached(const float* p, int64_t e0, int cnt, float (&x)[VEC]) {
    if constexpr (TAIL) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) x[v] = v < cnt ? gload_ptr<float>(p + e0)[v] : 0.f;
    } else {
#pragma unroll
        for (int q = 0; q < VEC / 4; ++q) {
            const f32x4 t = *(gload_ptr<f32x4>(p + e0) + q);
            x[4 * q] = t.x; x[4 * q + 1] = t.y; x[4 * q + 2] = t.z; x[4 * q + 3] = t.w;
        }
    }
}

template <int VEC, bool TAIL>
__device__ __forceinline__ void store_f32_cached(float* p, int64_t e0, int cnt, const float (&x)[VEC]) {
    if constexpr (TAIL) {
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            if (v < cnt) gstore_ptr<float>(p + e0)[v] = x[v];
    } else {
#pragma unroll
        for (int q = 0; q < VEC / 4; ++q)
            *(gstore_ptr<f32x4>(p + e0) + q) = f32x4{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
    }
}

// A replica unit: binary32 copy, or nearest-even bfloat16 (VEC*2 bytes: 8 or 16).
template <int VEC, bool TAIL>
__device__ __forceinline__ void store_replica(void* r, int rdt, int64_t e0, int cnt,
                                              const float (&x)[VEC]) {
    if (rdt == kF32) {
        store_f32<VEC, TAIL>(static_cast<float*>(r), e0, cnt, x);
        return;
    }
    uint16_t* h = static_cast<uint16_t*>(r) + e0;
    if constexpr (TAIL) {
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            if (v < cnt) gstore_ptr<uint16_t>(h)[v] = static_cast<uint16_t>(f32_to_bf16_bits(x[v]));
    } else if constexpr (VEC == 4) {
        u32x2 t = {f32_to_bf16_bits(x[0]) | (f32_to_bf16_bits(x[1]) << 16),
                   f32_to_bf16_bits(x[2]) | (f32_to_bf16_bits(x[3]) << 16)};
        __builtin_nontemporal_store(t, gstore_ptr<u32x2>(h));
    } else {
        u32x4 t;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            t[q] = f32_to_bf16_bits(x[2 * q]) | (f32_to_bf16_bits(x[2 * q + 1]) << 16);
        __builtin_nontemporal_store(t, gstore_ptr<u32x4>(h));
    }
}

// One whole 16-byte gradient unit as raw bits (4 binary32 or 8 bfloat16
// values), so that a batch of loads in flight costs four registers each whatever
// the dtype.
template <typename GT>
__device__ __forceinline__ u32x4 load_raw(const void* g, int64_t e0) {
    return __builtin_nontemporal_load(gload_ptr<u32x4>(static_cast<const GT*>(g) + e0));
}

// Raw unit bits -> binary32 values (bfloat16 widening is exact).
template <typename GT>
__device__ __forceinline__ void widen(const u32x4& r, float (&x)[Unit<GT>::VEC]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if constexpr (sizeof(GT) == 4) {
            x[q] = __uint_as_float(r[q]);
        } else {
            x[2 * q] = __uint_as_float(r[q] << 16);
            x[2 * q + 1] = __uint_as_float(r[q] & 0xffff0000u);
        }
    }
}

// ------------------------------------------------------------- pairwise sums

// Compile-time pairwise tree over leaves LO .. LO+CNT-1: leaf(k, x) produces the
// k-th term; the tree is PW with the largest-power-of-two split.
template <int LO, int CNT, int VEC, typename Leaf>
__device__ __forceinline__ void pw_tree(const Leaf& leaf, float (&out)[VEC]) {
    if constexpr (CNT == 1) {
        leaf(LO, out);
    } else {
        constexpr int H = pw_split(CNT);
        float a[VEC], b[VEC];
        pw_tree<LO, H, VEC>(leaf, a);
        pw_tree<LO + H, CNT - H, VEC>(leaf, b);
#pragma unroll
        for (int v = 0; v < VEC; ++v) out[v] = a[v] + b[v];
    }
}

// Runtime-count pairwise accumulator (a binary counter of partial sums). After
// k pushes, slot[l] holds the sum of an aligned block of 2^l terms for every set
// bit l of k; the largest block holds the earliest terms. result() folds the
// blocks from the smallest up, each time adding the earlier (larger) block on
// the left: exactly PW(x[0..k)) with the largest-power-of-two split.
// Every slot is updated by a select, never by a conditional store, so that the
// compiler cannot merge the per-level stores into one variable-index store
// (which would move the slots to scratch memory). At most 2^LEVELS - 1 pushes.
template <int VEC, int LEVELS>
struct PwAcc {
    float slot[LEVELS][VEC];
    uint32_t count = 0;

    __device__ __forceinline__ void push(float (&x)[VEC]) {
        bool carrying = true;
#pragma unroll
        for (int l = 0; l < LEVELS; ++l) {
            const bool full = (count >> l) & 1u;
            const bool merge = carrying && full;
            const bool park = carrying && !full;
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const float merged = slot[l][v] + x[v];
                slot[l][v] = park ? x[v] : slot[l][v];
                x[v] = merge ? merged : x[v];
            }
            carrying = merge;
        }
        ++count;
    }

    __device__ __forceinline__ void result(float (&out)[VEC]) const {
        bool have = false;
#pragma unroll
        for (int l = 0; l < LEVELS; ++l) {
            if ((count >> l) & 1u) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) out[v] = have ? slot[l][v] + out[v] : slot[l][v];
                have = true;
            }
        }
    }
};

__host__ __device__ constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// Largest divisor of k that is <= b (k, b >= 1); for a power of two k, the
// largest power of two <= b.
__host__ __device__ constexpr int largest_divisor_le(int k, int b) {
    return b <= 1 ? 1 : (k % b == 0 ? b : largest_divisor_le(k, b - 1));
}

// ------------------------------------------------------------- the update

struct Hyper {
    float lr, mu, wd;
};

// Alg. 3 update with heavy-ball momentum and L2 weight decay, each operation
// rounded separately: d = gbar + wd*p; m = mu*m + d; p = p - lr*m.
template <int VEC>
__device__ __forceinline__ void sgd_update(const Hyper& h, const float (&gbar)[VEC],
                                           float (&p)[VEC], float (&m)[VEC]) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        float d = gbar[v] + h.wd * p[v];
        m[v] = h.mu * m[v] + d;
        p[v] = p[v] - h.lr * m[v];
    }
}

// ------------------------------------------------------------- pointer sources

// Kernel arguments of the planless calls. Pointer tables travel by value
// (kernarg segment, read with scalar loads). grads[] is in member order:
// entry j*W + k is the k-th member (ascending worker id) of group j.
struct StepArgs {
    float* p;
    float* m;
    const float* gbar;  // lsgd_sgd_step only
    int64_t n;
    Hyper h;
    int32_t n_workers;
    int32_t pad[2];        // lsgd_batches.hpp: the reduction program behind starts a cache line
    int32_t n_replicas, rdt;
    uint32_t xcd_chunk, upl;
    const float* lr_ptr;   // non-null: the learning rate is read here when the kernel runs
    int32_t bcast_grad;    // write the mean gradient into the first bcast_grad (binary32) member buffers
    int32_t literal;       // paper-literal reduction (else mean of means)
    int32_t win_blocks;    // replica-major copy-out: workgroups per window and replica group (a multiple of 8)
    int64_t copy_blocks;   // replica-major copy-out: logical workgroups (the grid strides over them)
    const void* grads[kMaxWorkers];
    void* replicas[kMaxReplicas];
};

// The hyperparameters a kernel uses: lr from device memory when given.
__device__ __forceinline__ Hyper resolve_hyper(const Hyper& h, const float* lr_ptr) {
    Hyper r = h;
    if (lr_ptr) r.lr = *lr_ptr;
    return r;
}

// Group-mean outputs of lsgd_group_mean / inputs of lsgd_global_mean.
struct MeanArgs {
    int64_t n;
    int32_t W;   // inputs per mean: mean j is over in[j*W .. j*W + W)
    uint32_t xcd_chunk, upl;
    const void* in[kMaxWorkers];
    float* out[kMaxWorkers];
};

// ------------------------------------------------------------- per-unit bodies


// Widened gradient values one lane may hold at once: up to kUnrollFloats the
// whole two-level tree is unrolled with every load issued up front (32 fp32
// units = a 4x4 grouping with two-unit tiles); above it groups stream through
// in batches of about kStreamFloats, which bounds registers for the 32- to
// 128-worker groupings. Batches of 128 floats beat 64 by 2% on 8x8 bfloat16
// (177 VGPRs, two waves per SIMD) and tied elsewhere; 32 tied.
constexpr int kUnrollFloats = 128;
constexpr int kStreamFloats = 128;

// The groupings that compile-time kernels serve (among those the pickers
// list); every other one takes the stream kernels (lsgd_stream.hpp). Step of
// 1e7 elements without replicas, two states in turn, compile-time / stream, us:
//   binary32, N <= 16: 4x4 127 / 135, 8x1 72 / 82, 1x5 55 / 70;
//   binary32, N > 16: 8x4 256 / 229, 8x8 480 / 428, 1x64 477 / 429, 16x8 904 /
//     822, 5x5 195 / 186, 4x6 187 / 180, 32x2 434 / 431, but groups of 16: 2x16
//     225 / 231, 4x16 425 / 431, 8x16 807 / 822 (3x16 347 / 331);
//   bfloat16: 3x5 72 / 81, 4x6 107 / 109, 8x8 242 / 241, 16x8 457 / 450, but 12
//     groups: 12x2 120 / 108, 12x5 230 / 219, 12x3 148 / 149.
// One worker per group in a count that is no power of two runs as one group
// (one_group_form) or, in the paper-literal reduction, in the stream kernels.
template <typename GT>
constexpr bool ct_serves(int W, int G) {
    if (W == 1 && (G & (G - 1)) != 0) return false;
    return sizeof(GT) == 4 ? W * G <= 16 || (W == 16 && (G & (G - 1)) == 0) : G != 12;
}

// Units per lane tile in the compile-time fused kernels for N gradients.
// Binary32: two units (visited stream-major; measured +6-8% over one) while the
// whole tree fits the unrolled form (N <= 16), four once the groups stream
// through the accumulator (+3-8% over two; at N <= 16 three or four units lose
// 1-3%, since they leave the unrolled form). bfloat16 tiles stay at one unit:
// two units measured -1% at 4x4, +0.6% / -0.2% on the 3.5e8-element 8x8
// workload (step kernel alone / whole step), +1.6% at 8x8 and +4% at 16x8 on
// 2.6e7 elements.
template <typename GT>
constexpr int tile_units(int n_workers) {
    return sizeof(GT) == 4 ? (n_workers * 2 * Unit<GT>::VEC <= kUnrollFloats ? 2 : 4) : 1;
}

// Pairwise sum of K leaves (compile-time K) of T floats each: unrolled while
// K * LW floats (LW = floats a leaf loads) stay within kUnrollFloats, so that
// every load is issued up front; otherwise streamed in batches of about
// kStreamFloats through a compile-time-sized pairwise accumulator. Both give
// PW over the K leaves in order.
template <int K, int T, int LW, typename Leaf>
__device__ __forceinline__ void pw_leaves(const Leaf& leaf, float (&out)[T]) {
    if constexpr (K * LW <= kUnrollFloats) {
        pw_tree<0, K, T>(leaf, out);
    } else {
        // batches of a divisor of K leaves (a power of two where K is one), so
        // that they cover the K leaves exactly: a batch of kStreamFloats / LW
        // leaves that does not divide K would call leaf() past K
        constexpr int B0 = kStreamFloats / LW;
        constexpr int B = largest_divisor_le(K, B0 < 1 ? 1 : (B0 > K ? K : B0));
        static_assert(K % B == 0, "leaf batches cover the K leaves exactly");
        PwAcc<T, ilog2(K) + 1> acc;
#pragma unroll 1
        for (int j0 = 0; j0 < K; j0 += B) {
            float x[B][T];
#pragma unroll
            for (int q = 0; q < B; ++q) leaf(j0 + q, x[q]);
#pragma unroll
            for (int q = 0; q < B; ++q) acc.push(x[q]);
        }
        acc.result(out);
    }
}

// Optional broadcast of the mean gradient into the (binary32) gradient
// buffers of the first s.bcast_grad() members: all N when the step kernel
// writes the whole broadcast, only the first member when a copy pass of its
// own then copies that buffer to the others.
template <typename GT, int U, bool TAIL, typename Src>
__device__ __forceinline__ void broadcast_mean(const Src& s, const int64_t (&e0)[U], int cnt,
                                               float (&gbar)[U * Unit<GT>::VEC]) {
    constexpr int VEC = Unit<GT>::VEC;
    constexpr int T = U * VEC;
    if constexpr (sizeof(GT) == 4) {
        const int nw = s.bcast_grad();
        if (nw > 0) {
            for (int k = 0; k < nw; ++k) {
                float* g = static_cast<float*>(const_cast<void*>(s.grad(k)));
#pragma unroll
                for (int q = 0; q < U; ++q) store_f32<VEC, TAIL>(g, e0[q], cnt, slice<VEC, T>(gbar, q));
            }
        }
    }
}

// Parameters and momentum loaded, through the caches where they will be
// stored through them (s.cached_state(); see store_state), else
// nontemporally.
template <int VEC, int U, bool TAIL, typename Src>
__device__ __forceinline__ void load_state(const Src& s, const int64_t (&e0)[U], int cnt,
                                           float (&p)[U * VEC], float (&m)[U * VEC]) {
    constexpr int T = U * VEC;
    if (s.cached_state()) {
#pragma unroll
        for (int q = 0; q < U; ++q) load_f32_cached<VEC, TAIL>(s.p(), e0[q], cnt, slice<VEC, T>(p, q));
#pragma unroll
        for (int q = 0; q < U; ++q) load_f32_cached<VEC, TAIL>(s.m(), e0[q], cnt, slice<VEC, T>(m, q));
    } else {
#pragma unroll
        for (int q = 0; q < U; ++q) load_f32<VEC, TAIL>(s.p(), e0[q], cnt, slice<VEC, T>(p, q));
#pragma unroll
        for (int q = 0; q < U; ++q) load_f32<VEC, TAIL>(s.m(), e0[q], cnt, slice<VEC, T>(m, q));
    }
}

// Parameters and momentum of the compile-time fused kernels and of the
// update kernel go through the caches (write-back) when there are at most 16
// gradient buffers and parameters plus momentum fit the Infinity Cache
// (kCachedStateBytes), nontemporally otherwise. Measured in the same process
// with the Infinity Cache flushed before every step (so that no step reads
// what the previous one left there), cached loads and stores against
// nontemporal ones: 4x4 +4% at n = 1.2e7, +7% at 2.6e7, +5% at 3e7, +3% at
// 3.5e7, +0.6% at 4e7, -1% at 5e7, -4% at 1e8 and 2e8; 2x2 +12-14% up to
// 3.5e7, even at 2e8; the update alone +8% at 2.6e7, -4% at 3.5e8. With 32
// and more buffers cached stores lost 1-5% at every size. The kernels are
// instantiated both ways where the first condition holds and the host picks
// one at launch (a runtime branch between the forms inside one kernel cost
// the 64- and 128-buffer kernels 2-3%).
constexpr int64_t kCachedStateBytes = int64_t{288} << 20;
__host__ __device__ constexpr bool cached_state_for(int n_workers) { return n_workers <= 16; }
// The whole rule, for n elements of parameters (and of momentum).
__host__ __device__ constexpr bool use_cached_state(int n_workers, int64_t n) {
    return cached_state_for(n_workers) && n <= kCachedStateBytes / 8;
}

// Parameters, momentum and replicas stored. Parameters and momentum go
// through the caches (write-back) when s.cached_state() is set, else with
// nontemporal stores.
template <int VEC, int U, bool TAIL, typename Src>
__device__ __forceinline__ void store_state(const Src& s, const int64_t (&e0)[U], int cnt,
                                            const float (&p)[U * VEC], const float (&m)[U * VEC]) {
    constexpr int T = U * VEC;
    if (s.cached_state()) {
#pragma unroll
        for (int q = 0; q < U; ++q) store_f32_cached<VEC, TAIL>(s.p(), e0[q], cnt, slice<VEC, T>(p, q));
#pragma unroll
        for (int q = 0; q < U; ++q) store_f32_cached<VEC, TAIL>(s.m(), e0[q], cnt, slice<VEC, T>(m, q));
    } else {
#pragma unroll
        for (int q = 0; q < U; ++q) store_f32<VEC, TAIL>(s.p(), e0[q], cnt, slice<VEC, T>(p, q));
#pragma unroll
        for (int q = 0; q < U; ++q) store_f32<VEC, TAIL>(s.m(), e0[q], cnt, slice<VEC, T>(m, q));
    }
    const int R = s.n_replicas();
    const int rdt = s.rdt();
    for (int r = 0; r < R; ++r) {
        void* rp = s.replica(r);
#pragma unroll
        for (int q = 0; q < U; ++q) store_replica<VEC, TAIL>(rp, rdt, e0[q], cnt, slice<VEC, T>(p, q));
    }
}

// The update on loaded state, then parameters, momentum and replicas stored.
template <int VEC, int U, bool TAIL, typename Src>
__device__ __forceinline__ void update_and_store(const Src& s, const int64_t (&e0)[U], int cnt,
                                                 const float (&gbar)[U * VEC], float (&p)[U * VEC],
                                                 float (&m)[U * VEC]) {
    sgd_update<U * VEC>(s.hyper(), gbar, p, m);
    store_state<VEC, U, TAIL>(s, e0, cnt, p, m);
}

// Everything after the mean gradient, for a tile of U units: optional
// broadcast, the update, and the copy-out.
template <typename GT, int U, bool TAIL, typename Src>
__device__ __forceinline__ void finish_tile(const Src& s, const int64_t (&e0)[U], int cnt,
                                            float (&gbar)[U * Unit<GT>::VEC]) {
    constexpr int VEC = Unit<GT>::VEC;
    constexpr int T = U * VEC;
    broadcast_mean<GT, U, TAIL>(s, e0, cnt, gbar);
    float p[T], m[T];
    load_state<VEC, U, TAIL>(s, e0, cnt, p, m);
    update_and_store<VEC, U, TAIL>(s, e0, cnt, gbar, p, m);
}

// Fused step on one tile of U units, compile-time W and G (powers of two).
// Every array holds T = U*VEC floats: the tree is the same PW for each of them.
// Small N*T: the whole two-level tree is unrolled and every load issued up
// front. Large: groups are streamed GU at a time and folded into a pairwise
// accumulator over groups, which yields the same PW order. TAIL (the ragged
// end of a tensor, cnt < VEC elements) only with U = 1.
// Mean of means: each group's sum / W, then the sum over groups / G. With
// s.literal() (uniform) the paper-literal form: each group's sum / N = W*G,
// summed over the groups with no further division. Every divisor is a power
// of two, so each division is a multiplication by the exact reciprocal (the
// same rounding of the same exact quotient).
template <typename GT, int W, int G, int U, bool TAIL, typename Src>
__device__ __forceinline__ void mean_tile_ct(const Src& s, const int64_t (&e0)[U], int cnt,
                                             float (&gbar)[U * Unit<GT>::VEC]) {
    static_assert(!TAIL || U == 1, "ragged units are processed one at a time");
    constexpr int VEC = Unit<GT>::VEC;
    constexpr int T = U * VEC;
    const bool lit = s.literal() != 0;
    // Divisions by powers of two are the exact multiplications by 1/W, 1/N or
    // 1/G; the others (W = 3, 5, 6 or 7; G = 3, 5, 6, 7 or (LARS norms) 12; N of either)
    // are divisions. The mean of means divides each group's sum by W and the
    // total by G; the literal reduction each group's sum by N, the total by 1.
    constexpr bool kPow2W = (W & (W - 1)) == 0;
    constexpr bool kPow2G = (G & (G - 1)) == 0;
    const float group_div = lit ? static_cast<float>(W * G) : static_cast<float>(W);
    const float group_scale = 1.0f / group_div;
    const float total_scale = lit ? 1.0f : 1.0f / static_cast<float>(G);
    auto group_leaf = [&](int j, float (&gm)[T]) {
        auto member_leaf = [&](int k, float (&x)[T]) {
            const void* g = s.grad(j * W + k);
#pragma unroll
            for (int q = 0; q < U; ++q) load_grad<GT, TAIL>(g, e0[q], cnt, slice<VEC, T>(x, q));
        };
        float sum[T];
        if constexpr (W <= 16) pw_tree<0, W, T>(member_leaf, sum);
        else pw_leaves<W, T, T>(member_leaf, sum);   // larger groups: members streamed through an accumulator
        if constexpr (kPow2W && kPow2G) {
#pragma unroll
            for (int v = 0; v < T; ++v) gm[v] = sum[v] * group_scale;
        } else if constexpr (!kPow2W) {
#pragma unroll
            for (int v = 0; v < T; ++v) gm[v] = sum[v] / group_div;
        } else if (lit) {   // W a power of two, N not
#pragma unroll
            for (int v = 0; v < T; ++v) gm[v] = sum[v] / group_div;
        } else {
#pragma unroll
            for (int v = 0; v < T; ++v) gm[v] = sum[v] * group_scale;
        }
    };
    float tot[T];
    pw_leaves<G, T, W * T>(group_leaf, tot);
    if constexpr (kPow2G) {
#pragma unroll
        for (int v = 0; v < T; ++v) gbar[v] = tot[v] * total_scale;
    } else if (lit) {
#pragma unroll
        for (int v = 0; v < T; ++v) gbar[v] = tot[v];
    } else {
#pragma unroll
        for (int v = 0; v < T; ++v) gbar[v] = tot[v] / static_cast<float>(G);
    }
}

template <typename GT, int W, int G, int U, bool TAIL, typename Src>
__device__ __forceinline__ void fused_tile_ct(const Src& s, const int64_t (&e0)[U], int cnt) {
    float gbar[U * Unit<GT>::VEC];
    mean_tile_ct<GT, W, G, U, TAIL>(s, e0, cnt, gbar);
    finish_tile<GT, U, TAIL>(s, e0, cnt, gbar);
}

template <typename GT, int W, int G, bool TAIL, typename Src>
__device__ __forceinline__ void fused_unit_ct(const Src& s, int64_t e0, int cnt) {
    const int64_t e[1] = {e0};
    fused_tile_ct<GT, W, G, 1, TAIL>(s, e, cnt);
}

// Pointer source for the planless fused step: everything from StepArgs.
// CACHED: store parameters and momentum through the caches (1) or
// nontemporally (0).
template <int CACHED>
struct FlatSrcT {
    const StepArgs& a;
    Hyper h;
    __device__ const void* grad(int k) const { return a.grads[k]; }
    __device__ float* p() const { return a.p; }
    __device__ float* m() const { return a.m; }
    __device__ void* replica(int r) const { return a.replicas[r]; }
    __device__ int n_replicas() const { return a.n_replicas; }
    __device__ int rdt() const { return a.rdt; }
    __device__ Hyper hyper() const { return h; }
    __device__ int bcast_grad() const { return a.bcast_grad; }
    __device__ int literal() const { return a.literal; }
    __device__ int cached_state() const { return CACHED; }
};

// ------------------------------------------------------------- flat kernels

// Lane tiles over the units of a flat vector (for_tiles). The unit index space
// is [0, full] with unit `full` the ragged tail (n % VEC elements, present
// only when that is nonzero): the lane whose partial tile holds it runs it
// through the TAIL form of the unit body.
template <typename GT, int W, int G, int U, int CACHED>
__device__ __forceinline__ void step_flat_ct_body(const StepArgs& a) {
    constexpr int VEC = Unit<GT>::VEC;
    const FlatSrcT<CACHED> s{a, resolve_hyper(a.h, a.lr_ptr)};
    const int64_t full = a.n / VEC;
    const int rem = static_cast<int>(a.n - full * VEC);
    for_tiles<U, VEC>(
        full, full + (rem != 0), a.xcd_chunk, a.upl,
        [&](const int64_t (&e0)[U]) { fused_tile_ct<GT, W, G, U, false>(s, e0, VEC); },
        [&](int64_t u) {
            if (u < full) fused_unit_ct<GT, W, G, false>(s, u * VEC, VEC);
            else fused_unit_ct<GT, W, G, true>(s, u * VEC, rem);
        });
}

template <typename GT, int W, int G, int U, int CACHED>
__global__ __launch_bounds__(kBlock) void step_flat_ct(StepArgs a) {
    step_flat_ct_body<GT, W, G, U, CACHED>(a);
}

// The same kernel with at most CAP waves per SIMD. Left to itself, the
// compiler schedules for the highest occupancy the registers allow, and
// for some groupings it gets there by holding fewer loads in flight: the
// bfloat16 kernels for groups of 3 in 8 or more groups sink each gradient
// load to its use and wait for it (one 16-byte load in flight per wave), and
// the small binary32 groupings run four or more waves with short load
// batches. Under a cap of 2 or 3 the scheduler keeps a batch of loads in
// flight instead.
template <typename GT, int W, int G, int U, int CACHED, int CAP>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, CAP))) void step_flat_ct_cap(StepArgs a) {
    step_flat_ct_body<GT, W, G, U, CACHED>(a);
}

// The wave cap of the compile-time flat step kernel for G groups of W
// workers, 0 for none: measured, each grouping against the uncapped kernel
// at the ResNet-50 size (25.6M elements, same process, replicas R = N and
// R = 0). A grouping is listed where a cap gains at least one point of the
// 8 TB/s peak on the mean of the two and loses at most one in either.
struct WaveCapEntry {
    short W, G, cap;
};
constexpr WaveCapEntry kWaveCapF32[] = {
    {1, 8, 2}, {1, 16, 2}, {2, 4, 2}, {2, 8, 2}, {3, 3, 2}, {3, 4, 2}, {3, 5, 2}, {4, 2, 2}, {4, 4, 2},
    {5, 2, 2}, {5, 3, 2}, {6, 2, 2}, {8, 1, 2}, {12, 1, 2}, {16, 1, 2}, {16, 2, 2}, {16, 4, 2}, {16, 8, 2},
    {1, 2, 3}, {1, 4, 3}, {2, 1, 3}, {2, 2, 3}, {3, 1, 3}, {3, 2, 3}, {4, 1, 3}, {4, 3, 3}, {5, 1, 3},
    {6, 1, 3},
};
constexpr WaveCapEntry kWaveCapBF16[] = {
    {1, 2, 2}, {1, 4, 2}, {2, 1, 2}, {2, 2, 2}, {3, 1, 2}, {3, 8, 2}, {3, 16, 2}, {3, 32, 2}, {4, 1, 2},
    {5, 16, 2}, {8, 1, 2}, {8, 6, 2}, {1, 8, 3}, {1, 16, 3}, {2, 4, 3}, {4, 2, 3}, {5, 1, 3}, {6, 1, 3},
};
template <typename GT>
constexpr int flat_wave_cap(int W, int G) {
    constexpr bool kBF16 = sizeof(GT) == 2;
    const WaveCapEntry* t = kBF16 ? kWaveCapBF16 : kWaveCapF32;
    const int n = kBF16 ? sizeof(kWaveCapBF16) / sizeof(WaveCapEntry) : sizeof(kWaveCapF32) / sizeof(WaveCapEntry);
    for (int i = 0; i < n; ++i)
        if (t[i].W == W && t[i].G == G) return t[i].cap;
    return 0;
}

// The flat step kernel for (W, G): capped where the table says so.
template <typename GT, int W, int G, int U, int CACHED>
constexpr auto flat_step_kernel() {
    constexpr int cap = flat_wave_cap<GT>(W, G);
    if constexpr (cap != 0) return step_flat_ct_cap<GT, W, G, U, CACHED, cap>;
    else return step_flat_ct<GT, W, G, U, CACHED>;
}

// The mean of a run of K of the call's inputs (PW, / K), compile-time K:
// lsgd_group_mean takes group blockIdx.y's members, lsgd_global_mean the group
// means. A workgroup reads one group's K + 1 streams; walking all groups per
// lane kept K loads in flight at a time and switched streams for each.
template <typename GT, int K, int U, bool TAIL>
__device__ __forceinline__ void mean_tile(const MeanArgs& a, const int64_t (&e0)[U], int cnt) {
    constexpr int VEC = Unit<GT>::VEC;
    constexpr int T = U * VEC;
    const int j = static_cast<int>(blockIdx.y);
    float sum[T];
    pw_leaves<K, T, T>([&](int k, float (&x)[T]) {
        const void* g = a.in[j * K + k];
#pragma unroll
        for (int q = 0; q < U; ++q) load_grad<GT, TAIL>(g, e0[q], cnt, slice<VEC, T>(x, q));
    }, sum);
#pragma unroll
    for (int v = 0; v < T; ++v) sum[v] = sum[v] / static_cast<float>(K);
#pragma unroll
    for (int q = 0; q < U; ++q) store_f32<VEC, TAIL>(a.out[j], e0[q], cnt, slice<VEC, T>(sum, q));
}

template <typename GT, int K, int U>
__global__ __launch_bounds__(kBlock) void mean_kernel_ct(MeanArgs a) {
    constexpr int VEC = Unit<GT>::VEC;
    const int64_t full = a.n / VEC;
    const int rem = static_cast<int>(a.n - full * VEC);
    for_tiles<U, VEC>(
        full, full + (rem != 0), a.xcd_chunk, a.upl,
        [&](const int64_t (&e0)[U]) { mean_tile<GT, K, U, false>(a, e0, VEC); },
        [&](int64_t u) {
            const int64_t e[1] = {u * VEC};
            if (u < full) mean_tile<GT, K, 1, false>(a, e, VEC);
            else mean_tile<GT, K, 1, true>(a, e, rem);
        });
}

// lsgd_sgd_step: update and copy-out from a precomputed mean gradient, one
// tile of U 4-element units, stream-major.
template <int U, bool TAIL, int CACHED>
__device__ __forceinline__ void sgd_tile(const StepArgs& a, const Hyper& h, const int64_t (&e0)[U],
                                         int cnt) {
    constexpr int T = U * 4;
    float g[T], p[T], m[T];
#pragma unroll
    for (int q = 0; q < U; ++q) load_f32<4, TAIL>(a.gbar, e0[q], cnt, slice<4, T>(g, q));
    if constexpr (CACHED != 0) {
#pragma unroll
        for (int q = 0; q < U; ++q) load_f32_cached<4, TAIL>(a.p, e0[q], cnt, slice<4, T>(p, q));
#pragma unroll
        for (int q = 0; q < U; ++q) load_f32_cached<4, TAIL>(a.m, e0[q], cnt, slice<4, T>(m, q));
    } else {
#pragma unroll
        for (int q = 0; q < U; ++q) load_f32<4, TAIL>(a.p, e0[q], cnt, slice<4, T>(p, q));
#pragma unroll
        for (int q = 0; q < U; ++q) load_f32<4, TAIL>(a.m, e0[q], cnt, slice<4, T>(m, q));
    }
    sgd_update<T>(h, g, p, m);
    if constexpr (CACHED != 0) {
#pragma unroll
        for (int q = 0; q < U; ++q) store_f32_cached<4, TAIL>(a.p, e0[q], cnt, slice<4, T>(p, q));
#pragma unroll
        for (int q = 0; q < U; ++q) store_f32_cached<4, TAIL>(a.m, e0[q], cnt, slice<4, T>(m, q));
    } else {
#pragma unroll
        for (int q = 0; q < U; ++q) store_f32<4, TAIL>(a.p, e0[q], cnt, slice<4, T>(p, q));
#pragma unroll
        for (int q = 0; q < U; ++q) store_f32<4, TAIL>(a.m, e0[q], cnt, slice<4, T>(m, q));
    }
    for (int r = 0; r < a.n_replicas; ++r) {
        void* rp = a.replicas[r];
#pragma unroll
        for (int q = 0; q < U; ++q) store_replica<4, TAIL>(rp, a.rdt, e0[q], cnt, slice<4, T>(p, q));
    }
}

template <int U, int CACHED>
__global__ __launch_bounds__(kBlock) void sgd_kernel(StepArgs a) {
    const Hyper h = resolve_hyper(a.h, a.lr_ptr);
    const int64_t full = a.n / 4;
    const int rem = static_cast<int>(a.n - full * 4);
    for_tiles<U, 4>(
        full, full + (rem != 0), a.xcd_chunk, a.upl,
        [&](const int64_t (&e0)[U]) { sgd_tile<U, false, CACHED>(a, h, e0, 4); },
        [&](int64_t u) {
            const int64_t e[1] = {u * 4};
            if (u < full) sgd_tile<1, false, CACHED>(a, h, e, 4);
            else sgd_tile<1, true, CACHED>(a, h, e, rem);
        });
}

// ------------------------------------------------------------- copy-out pass
//
// With several replicas the copy-out runs as a pass of its own after the step
// kernel (which then writes no replica). It runs replica-major over windows of
// the parameter vector: workgroup b writes block s of window w to replica
// group q (RK consecutive replicas), b = (w*ceil(R/RK) + q)*win_blocks + s, so
// at any time the chip writes a few replica streams instead of all R. With
// win_blocks a multiple of 8 each XCD (workgroups go to XCD b % 8) reads the
// same eighth of the window for every replica group: after the first group the
// window comes from that XCD's L2 (p is read with cache-allocating loads; a
// window is 8 MB, 1 MB per XCD). A lane loads U units of p and stores them to
// each of its group's replicas: several loads in flight and several stores per
// load keep the pass at the write bandwidth (one unit and one replica per lane
// left the bfloat16 pass at about half of it). Binary32 replicas take
// 4-element units, bfloat16 replicas 8-element units, so every store is 16
// bytes. Grids above kMaxGridBlocks stride over the logical workgroups.
template <int VEC, int U, int RK>
__device__ __forceinline__ void copy_out_rmajor_block(const StepArgs& a, int64_t b) {
    const int64_t full = a.n / VEC;
    const int rem = static_cast<int>(a.n - full * VEC);
    const int n_rg = (a.n_replicas + RK - 1) / RK;
    const int64_t per_win = static_cast<int64_t>(a.win_blocks) * n_rg;
    const int64_t w = b / per_win;
    const int64_t rb = b - w * per_win;
    const int q = static_cast<int>(rb / a.win_blocks);
    const int64_t sblk = rb - static_cast<int64_t>(q) * a.win_blocks;
    const int64_t u0 = (w * a.win_blocks + sblk) * kBlock * U + threadIdx.x;
    const int r0 = q * RK;
    float x[U][VEC];
#pragma unroll
    for (int t = 0; t < U; ++t) {
        const int64_t u = u0 + static_cast<int64_t>(t) * kBlock;
        if (u < full) load_f32_cached<VEC, false>(a.p, u * VEC, VEC, x[t]);
        else if (u == full && rem != 0) load_f32_cached<VEC, true>(a.p, u * VEC, rem, x[t]);
    }
#pragma unroll
    for (int k = 0; k < RK; ++k) {
        if (r0 + k >= a.n_replicas) break;
        void* dst = a.replicas[r0 + k];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int64_t u = u0 + static_cast<int64_t>(t) * kBlock;
            if (u < full) store_replica<VEC, false>(dst, a.rdt, u * VEC, VEC, x[t]);
            else if (u == full && rem != 0) store_replica<VEC, true>(dst, a.rdt, u * VEC, rem, x[t]);
        }
    }
}

// The grid (a multiple of 8 workgroups, or all of them) strides over the
// logical workgroups, so each keeps its XCD.
template <int VEC, int U, int RK>
__global__ __launch_bounds__(kBlock) void copy_out_rmajor_kernel(StepArgs a) {
    for (int64_t b = blockIdx.x; b < a.copy_blocks; b += gridDim.x) copy_out_rmajor_block<VEC, U, RK>(a, b);
}

}  // namespace lsgd
