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
// Up to 16 workers with a compile-time kernel, split / compile-time:
//   whole vectors: bfloat16 never (1x4 n = 65536 2.6 / 2.4, 4x4 131072 3.6 /
//   3.1, 2x5 100000 4.1 / 3.2); binary32 from 8 workers (1x4 65536 2.9 / 2.4,
//   131072 3.2 / 2.8; 2x4 40000 0.76, 262144 0.88 of it; 4x4 65536 3.4 / 4.6),
//   beyond 4096 elements (4x4: 1024; n = 1000: 1.2 of it, every layout);
//   ragged vectors: bfloat16 always (1x1 n = 40001 0.89 of it, 1x4 0.85, 4x4
//   0.56); binary32 from 2 workers beyond 4096 elements (1x1 1.04, 1x2 0.93 to
//   1.04, 1x4 10007 0.79, 4x4 2003 0.64), more than 8 workers from 1024.
// More workers or no compile-time kernel (split / the other one):
//   bfloat16: 8x8 n = 262144 10.8 / 10.8; but more than 64 whole ones only up
//   to 3 * 2^16 (16x8 185360 0.85 of it, 262144 21.0 / 18.2; ragged 262141
//   22.1 / 76.5);
//   binary32 of more than 16 workers: up to 3 * 2^17 (370727: 8x8 18.7 / 25.3,
//   16x8 41.3 / 46.1, 10x4 13.4 / 17.7, unequal 16 groups of 30 25.9 / 24.4;
//   524288: 8x8 28.4 / 26.8, 16x8 59.0 / 48.8, unequal 34.7 / 24.8).
inline bool split_serves(int64_t n, int n_workers, bool bf16, bool compile_time) {
    const bool whole = n % (bf16 ? 8 : 4) == 0;
    if (compile_time && n_workers <= 16) {
        if (n > int64_t{1} << 18) return false;
        if (bf16) return !whole;
        return n_workers >= (whole ? 8 : 2) && n > (n_workers > 8 ? 1024 : 4096);
    }
    if (bf16) return n <= (compile_time && whole && n_workers > 64 ? int64_t{3} << 16 : int64_t{1} << 18);
    return n <= (n_workers > 16 ? int64_t{3} << 17 : int64_t{1} << 18);
}

}  // namespace lsgd
