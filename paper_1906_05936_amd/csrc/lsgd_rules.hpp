// Which kernels a call takes: rules on sizes, counts and types, each with the
// measurements that put its line where it is. Plain C++, no HIP.
//
// Unless a rule says otherwise its figures are microseconds of one step on the
// GPU (graph replays, two states in turn), and "n is whole" means a multiple
// of a gradient unit (16 bytes: 4 binary32 or 8 bfloat16 elements).
#pragma once

#include <stdint.h>

namespace lsgd {

// ------------------------------------------------------ split kernels, flat
//
// The split kernels divide the members over the waves of a workgroup and give
// the ragged end a workgroup of its own; the others sum all members in a lane,
// and a ragged end is a second pass of one lane. `compile_time`: a
// compile-time kernel serves the layout.
//
// `copy_bytes`: bytes of copies per element (replicas, broadcast gradients),
// which the split kernels divide over their waves too.
//
// Up to 16 workers with a compile-time kernel, time of split over compile-time
// (ranges are means over random layouts of one range of sizes):
//   more than 32 bytes of copies: split, binary32 0.34 to 0.98, ragged bfloat16
//   0.30 to 0.73, whole bfloat16 of more than 4 workers 0.79 to 1.03 (1x8 n =
//   3825, 23 copies 3.7 / 9.1 us);
//   whole bfloat16 with fewer never (1x4 n = 65536 2.6 / 2.4 us, 4x4 131072 3.6 /
//   3.1, 1 to 8 workers 1.02 to 1.32), ragged always (1x4 0.85, 4x4 0.56, 9 to 16
//   workers 0.39 to 0.50);
//   whole binary32 from 8 workers (8 0.82 to 1.02, 9 to 16 0.72 to 0.91), with
//   copies from 5 (0.71 to 1.05, 4 0.90 to 1.11; 1x4 65536 without 2.9 / 2.4 us),
//   beyond 1024 elements (n = 1000: 1.2);
//   ragged binary32 from 2 workers (0.66 to 1.04), with copies from 4 (0.60 to
//   1.02, 2 and 3 0.96 to 1.13; 1x8 n = 11 2.4 / 2.8 us, 3x4 205, 4 copies 3.2 / 4.4).
// More workers or no compile-time kernel, split / the other one:
//   bfloat16: 8x8 n = 262144 10.8 / 10.8 us; but more than 64 whole ones only up
//   to 3 * 2^16 (16x8 185360 0.85 of it, 262144 21.0 / 18.2; ragged 262141
//   22.1 / 76.5);
//   binary32 of more than 16 workers: up to 2^18 + 2^23 / workers (17 to 24 workers
//   0.75 around 3e5 elements, 0.96 around 6.5e5, 1.09 beyond; 25 to 32 0.80, 1.04,
//   1.15; 33 to 48 0.84 and, around 4.5e5, 1.04; 49 to 64 0.96 around 3.3e5, 1.2
//   beyond; 65 to 128 0.86 around 2.3e5, 1.05 around 3.3e5).
inline bool split_serves(int64_t n, int n_workers, bool bf16, bool compile_time, int64_t copy_bytes) {
    const bool whole = n % (bf16 ? 8 : 4) == 0;
    const bool many_copies = copy_bytes > 32;
    if (compile_time && n_workers <= 16) {
        if (n > int64_t{1} << 18) return false;
        if (bf16) return !whole || (many_copies && n_workers > 4);
        if (many_copies) return true;
        if (whole) return n > 1024 && n_workers >= (copy_bytes ? 5 : 8);
        return n_workers >= (copy_bytes ? 4 : 2);
    }
    if (bf16) return n <= (compile_time && whole && n_workers > 64 ? int64_t{3} << 16 : int64_t{1} << 18);
    return n <= (int64_t{1} << 18) + (n_workers > 16 ? (int64_t{1} << 23) / n_workers : 0);
}

// ------------------------------------------------------ split kernels, plans
//
struct PlanShape {
    int64_t elems, tensors;    // elements of all tensors, tensors that have any
    int64_t pieces;            // pieces of 2048 elements
    int64_t ragged;            // tensors that end in part of a gradient unit
    int n_workers;
    bool bf16, compile_time;   // a compile-time kernel serves the step
    bool pow2_groups;          // its group count is a power of two
    int64_t copy_bytes;        // bytes of replicas per element
};

// Plans too small to fill the chip. Time of split over the others around the
// line (means over random layouts and tensor counts):
//   up to 16 workers bfloat16 to 2^20 (4x4 10.2 / 16.1 us), binary32 to 2^19 (30
//   tensors, 1x4 4.1 / 5.2 us, 4x4 8.2 / 10.1), to 2^20 where the tensors hold 2^15
//   elements or fewer on average (1e6, 60 tensors 0.92, 3 to 30 tensors 1.03 to 1.12);
//   more workers, without compile-time kernel: bfloat16 to 2^20 (17 to 48 workers
//   0.70 to 1.0 around 9e5), of more than 48 to 5 * 2^17 (0.80 to 0.98 around 6.5e5,
//   1.15 to 1.5 beyond); binary32 with ragged tensors to 2^20 (17 to 32 workers
//   0.95 to 0.99 around 9e5), of more than 32 to 3 * 2^18 (0.89 to 0.94, 1.0
//   beyond), whole ones to 2^18 + 10 * 2^20 / workers (17 to 24 0.89 around 6.5e5,
//   33 to 48 0.92 and 1.05, 49 to 64 1.02 around 4.5e5, 65 to 128 0.91 around 2.3e5,
//   1.05 around 3.3e5);
//   with one, ragged tensors (bfloat16 17 to 64 workers 0.68 to 0.77, 65 to 128
//   0.92) and binary32 (4x16 639360 41.4 / 58.3 us, 1.04e6 0.91) to 2^20.
inline bool plan_fits_split(const PlanShape& s) {
    const int64_t n = s.elems;
    if (n > int64_t{1} << 20) return false;
    if (s.n_workers <= 16) return s.bf16 || n <= int64_t{1} << 19 || n <= s.tensors << 15;
    if (s.compile_time && (s.ragged || !s.bf16)) return true;
    if (s.bf16) return n <= (s.n_workers <= 48 ? int64_t{1} << 20 : int64_t{5} << 17);
    if (s.ragged) return s.n_workers <= 32 || n <= int64_t{3} << 18;
    return n <= (int64_t{1} << 18) + (int64_t{10} << 20) / s.n_workers;
}

// Plans of any size whose tensors leave most of a workgroup's piece empty. One
// piece of 2048 elements costs the other kernels the same however short it is
// (4096-element tiles twice that), a split piece holds 256. R = 0, split / the
// others: binary32 without compile-time kernel 10x4 20000 tensors of 200 204 /
// 2196, 3000 of 700 80 / 306, 8x8 3000 of 700 122 / 141 with two-unit tiles;
// 1x4 20000 of 200 28 / 74, 5000 of 1000 29 / 43, but 2x4 2000 of 900 20.0 /
// 16.4, 4x4 66 / 61 and 70 / 70;
// bfloat16 4x4 20000 of 200 52 / 204, 8x8 2000 of 900 110 / 123.
inline bool plan_of_small_tensors(const PlanShape& s) {
    if (!s.bf16 && s.compile_time && s.n_workers > 4) return false;
    const int64_t held = s.pieces * 2048;
    return s.bf16 || s.compile_time ? 2 * s.elems < held : 5 * s.elems < 2 * held;
}

// Whether a plan's step takes the split kernels. Where a tensor is ragged, or
// there is no compile-time kernel, always. Where all are whole (time of split
// over compile-time, means over random layouts and tensor counts):
//   bfloat16 up to 16 workers: not (1 to 8 workers 1.02 to 1.2, 9 to 16 0.95 to
//   1.13), but from 5 with more than 32 bytes of copies (0.74 to 1.03) or another
//   group count than a power of two (0.66 to 1.14, 9 to 16 0.81 to 0.97), to 3 * 2^18
//   (0.92 around 6.5e5);
//   bfloat16 of more workers: 17 to 24 to 2^19 (0.64 to 0.67 around 3e5; 5x4 464512
//   elements 9.0 / 19.3 us), up to 48 to 2^18 (0.33 to 0.81, 1.0 beyond), more to 3
//   * 2^16 (0.65 to 0.87, 1.0 beyond); with many copies a quarter further (1x32
//   300032, R = 32 8.6 / 11.9 us);
//   binary32 with many copies or such a group count to 2^19 (0.51 to 0.98), else
//   from 8 workers beyond 4096 elements (0.66 to 0.91, below 0.96 to 1.19), from 4
//   beyond 8192 (0.75 to 0.96, below 0.94 to 1.05), fewer only small tensors of more
//   than 2^19 elements (1x2, 1e6, 160 tensors 0.93 / 1.24 of the time before either;
//   2^19, 10 tensors 1.06 / 0.97).
inline bool split_serves_plan(const PlanShape& s) {
    if (!plan_fits_split(s)) return plan_of_small_tensors(s);
    if (!s.compile_time || s.ragged) return true;
    const bool many_copies = s.copy_bytes > 32;
    const int64_t n = s.elems;
    if (s.n_workers > 16) {
        const int64_t line = s.n_workers <= 24 ? int64_t{1} << 19 : s.n_workers <= 48 ? int64_t{1} << 18 : int64_t{3} << 16;
        return !s.bf16 || n <= (many_copies ? line + line / 4 : line);
    }
    if (s.bf16) return n <= int64_t{3} << 18 && s.n_workers > 4 && (many_copies || !s.pow2_groups);
    if (many_copies || !s.pow2_groups) return n <= int64_t{1} << 19;
    if (s.n_workers < 4) return n > int64_t{1} << 19 && n <= s.tensors << 13;
    return n > (s.n_workers < 8 ? 8192 : 4096);
}

// Whether LARS steps take the split kernels; `merged`: every workgroup of the
// update can sum its tensor's partials (else they need a launch of their own).
// Split / the others, us, or of the time before either where noted:
//   merged, binary32 of up to 16 workers to 2^19 elements, or 2^20 where the
//   tensors are small (1x4 2^19, 60 tensors 0.81 of the others, 1e6 16.4 / 13.5,
//   160 tensors 1.03 / 1.14 of the time before);
//   bfloat16 with a compile-time kernel and no ragged tensor, of the time before:
//   merged to 9 * 2^16 (4x4 2^18 0.79 / 0.85, 60 tensors 2^19 0.87 / 0.87 and,
//   R = 16, 14.1 / 18.1 us, 1e6 1.11 / 1.00), of up to 24 workers in groups whose
//   count is no power of two to 3 * 2^18 (5x4 698304 16.2 / 21.3 us, 9 to 16 workers
//   0.64 to 0.87 of the others, 25 and more 1.2 from 2^19); not merged, more than
//   16 workers to 3 * 2^16 (8x8 131072 0.50 to 0.75 / 0.68 to 0.98, 3 tensors
//   262144 1.27 / 0.99);
//   not merged, bfloat16 of 9 to 16 workers to 2^19 (1x4 3 tensors 2^19 12.0 /
//   11.1, 4x4 14.6 / 17.1, 1x9 13.5 / 14.1, 1e6 21.5 / 18.0) and more than 16
//   workers (8x8 2^19 26.5 / 44.8; binary32 35.2 / 51.3, but 1x4, one tensor, 16.8
//   / 12.4, 4x4 26.5 / 19.8);
//   binary32 of more than 16 workers beyond 2^19 not where the tensors are few and
//   large (8x8, n = 1e6, 3 tensors 63.6 / 58.7, 16 tensors 63.8 / 76.5), and not
//   of more than 64 (1.04 to 1.48 of the others).
inline bool split_serves_lars(const PlanShape& s, bool merged) {
    const int64_t n = s.elems;
    const bool many = s.n_workers > 16;
    if (n > int64_t{1} << 20) return false;
    if (s.bf16 && s.compile_time && s.ragged == 0)
        return merged ? n <= (s.pow2_groups || s.n_workers > 24 ? int64_t{9} << 16 : int64_t{3} << 18)
                      : many && n <= int64_t{3} << 16;
    if (!merged && !many && !(s.bf16 && s.n_workers > 8 && n <= int64_t{1} << 19)) return false;
    return s.bf16 || n <= int64_t{1} << 19 || (s.n_workers <= 64 && n <= s.tensors << (many ? 18 : 13));
}

// ------------------------------------------------------ copy pass of a plan
//
// Replicas that a workgroup of the copy pass writes per piece of 2048 elements
// (times 2 for bfloat16 replicas): 1, or more where the pieces are mostly empty
// (`elems` in `pieces` pieces), so that fewer workgroups each read their tables.
// Binary32, whole step, 1 / 2 / 4, us: 4x4 LARS, 3000 tensors of 700, R = 16 113
// / 88 / 75; 1x4 LARS, 20000 of 200, R = 4 194 / 152 / 129; 8x8, 300 of 2500, R =
// 64 98 / 76 / 78; 8x8, 60 tensors, 1.2e7 elements 1049 / 1095 / 1110.
inline int copy_replicas_per_group(int64_t elems, int64_t pieces) {
    return elems < pieces * 1024 ? 4 : elems < pieces * 1600 ? 2 : 1;
}

// ------------------------------------------- binary32 stream kernels, units
//
// Whether a binary32 step in a stream kernel takes lane tiles of two units and
// nothing issued ahead instead of four: `pieces` workgroup tiles of 4096
// elements on `cus` compute units, one at a time each, in at most `rounds`
// rounds where the choice matters. Four / two units, us:
//   up to 11 workers always (1x9: n = 1e6 10.0 / 9.9, 3e6 32.6 / 28.2, 1e7 95.2
//   / 82.4, 2.5e7 245.9 / 233.3), up to 16 to 2^24 elements (1x14 1e7 122.0 /
//   117.2, 2.5e7 329.0 / 336.0; unequal 2, 3, 5, 6 1e7 134.6 / 130.8, 2.5e7
//   356.6 / 367.4), but not where four-unit tiles make one round that is more
//   than half full (1x9, n = 1e6, R = 4 11.6 / 13.4, R = 8 13.8 / 14.4);
//   more workers, where the last round fills at most half of the units (8x8:
//   n = 2^19 26.7 / 23.2, 6e5 30 / 33.8, 2^20 44.5 / 47.7, 2^20 + 1 57.7 / 48.6,
//   1.1e6 63.2 / 54.6, 1.3e6 70.9 / 71.6, 1.6e6 73.3 / 78.0, 2.4e6 114.7 / 120.7;
//   16x8: 2^19 48.9 / 43.1, 1.1e6 117.8 / 104.9), in the first two rounds.
inline bool stream_two_units(int64_t pieces, int rounds, int n_workers, int64_t n, int cus) {
    if (pieces <= cus && pieces > cus / 2) return false;
    if (n_workers <= 16) return n_workers < 12 || n <= int64_t{1} << 24;
    return pieces <= int64_t{rounds} * cus && (pieces - 1) % cus < cus / 2;
}

// The same for a plan of `pieces` pieces of 4096 elements: two units also where
// the pieces of 2048 (s.pieces) are at most half as many again, so that four-unit
// tiles would be half empty (10x4, 1000 tensors of 5000 204 / 174, 3000 of 1500
// 325 / 156), and where more than a fifth of the pieces end in a ragged element,
// a tile of its own after the other (8x8: 1000 ragged tensors of 3000 217 / 154,
// whole ones 133 / 152, 300 of 10000 161 / 146, 1000 of 9000 486 / 438).
inline bool plan_two_units(const PlanShape& s, int64_t pieces, int cus) {
    return 2 * s.pieces <= 3 * pieces || 5 * s.ragged > pieces || stream_two_units(pieces, 4, s.n_workers, s.elems, cus);
}

// ------------------------------------------------ copies in a pass of their own
//
// Parameters and momentum beyond this do not survive in the Infinity Cache
// from one step to the next, whatever runs in between.
constexpr int64_t kWarmStateBytes = int64_t{128} << 20;

// Whether a step of n elements writes `copy_bytes` bytes of copies per element
// (replicas of rsz bytes, the broadcast's copies of the mean gradient) after the
// step kernel (apart) or in it. gsz: bytes of a gradient element. `cached`:
// parameters and momentum go through the caches (at most 16 workers); `stream`:
// the step runs in a stream kernel.
//  - gradients of 256 bytes and more: apart;
//  - nontemporal parameters and momentum: from 32 bytes (in the kernel / apart:
//    8x4 binary32 R = 8 364 / 342, bfloat16 R = 16 241 / 234);
//  - beyond kWarmStateBytes: from 32 bytes (unequal 2, 3, 5, 6, n = 2.5e7:
//    binary32 32 B 486 / 472, 48 B 569 / 512, 1x9 bfloat16 32 B 304 / 280),
//    16 for bfloat16 gradients with binary32 replicas (unequal, 297 / 275);
//  - else the pass has a launch (2 to 3 us) and a second reading of the
//    parameters to make good. bfloat16 gradients with binary32 replicas: from
//    24 bytes and 26 MB of copies (apart / in the kernel, 1x4 to 4x4: n = 6e5
//    32 B 1.04 to 1.07, 48 B 0.87 to 0.93, 1e6 24 B 1.05 to 1.14, 32 B 0.89 to
//    0.97, 3e6 24 B 0.83 to 0.88);
//  - the others: from 48 bytes (up to 4 workers 56, stream kernels 64) and 128
//    MB of copies (4x4 binary32: n = 3e5 48 B 1.34, 1e6 48 B 1.15, 56 B 1.13, 2e6
//    56 B 1.00, 3e6 48 B 0.98, 40 B 0.97 to 1.00 from 2e6; 1x4 48 B 1.01 to 1.11,
//    56 B 0.96 to 0.99 from 3e6; 2x4 48 B 0.98 to 1.03; 1x9, a stream kernel, 48
//    B 1.05 to 1.08, 56 B 1.03 to 1.07);
//  - with the broadcast, whose copies the step kernel already has at hand: from
//    64 bytes, 52 from 12 workers (n = 3e6: 2x4 60 B 1.09, 3x3 48 B 1.07, 3x4 52
//    B 1.02, 4x4 60 B 0.97; 1.2e7: 2x4 60 B 1.04, 3x4 60 B 0.98).
inline bool copies_apart(int n_workers, int gsz, int rsz, int64_t copy_bytes, bool broadcast, int64_t n, bool stream,
                         bool cached) {
    if (copy_bytes <= 0) return false;
    if (static_cast<int64_t>(n_workers) * gsz >= 256) return true;
    if (!cached) return copy_bytes >= 32;
    const bool widened = gsz == 2 && rsz == 4;
    if (n > kWarmStateBytes / 8) return copy_bytes >= (widened ? 16 : 32);
    const int64_t mb = n * copy_bytes >> 20;
    if (widened) return copy_bytes >= 24 && mb >= 26;
    const int crossing = broadcast ? (n_workers >= 12 ? 52 : 64) : stream ? 64 : n_workers <= 4 ? 56 : 48;
    return copy_bytes >= crossing && mb >= 128;
}

// ---------------------------------------------------- means, any input count
//
// The form of the binary32 stream kernel for means of `inputs` inputs of n
// elements. One unit per lane, nothing issued ahead, up to 2^19 elements (n =
// 1e5, four units / one, us: 9 inputs 9.1 / 5.3, 64 24.8 / 11.2, 128 43.1 /
// 20.8; 3e5, 128: 46.3 / 27.6); one unit, the next batch issued ahead, beyond
// (9 inputs 1e6 11.7 / 11.0, 1e7 95 / 81, 20 inputs 2.5e7 386 / 379, 64 1057 /
// 992); but four units for 32 inputs or more up to 2^22 (32 inputs 1e6 22.4 /
// 23.7, 3e6 64.9 / 71.4; 64 1e6 41.9 / 44.5).
enum class MeanForm { kOne, kOneAhead, kFourAhead };
inline MeanForm mean_stream_form(int inputs, int64_t n) {
    if (n <= int64_t{1} << 19) return MeanForm::kOne;
    return inputs >= 32 && n <= int64_t{1} << 22 ? MeanForm::kFourAhead : MeanForm::kOneAhead;
}
inline int mean_stream_tile(int inputs, int64_t n, bool bf16) {
    return !bf16 && mean_stream_form(inputs, n) == MeanForm::kFourAhead ? 4 : 1;
}

}  // namespace lsgd
