// The table of schedule variants: what every row's knobs are.  One list per part: attn_kernels.hip compiles
// the kernels of one part, so that the build runs its parts side by side (the kernels take four
// minutes to compile one after the other).
#pragma once
#include "attn_kernel.h"

namespace attn {

typedef void (*KernelFn)(const uint16_t*, const uint16_t*, const uint16_t*, uint16_t*, float*, uint64_t, uint64_t, uint64_t, int);

// The kernels of one variant for one head dimension, by [dtype][causal]; defined in attn_kernels.hip.
template <int D, class KN>
struct KernelSet {
    static const KernelFn fn[2][2];
};

}  // namespace attn

// BOTH, D64, D128 (bn, nw, qb, occ, ldp, pipe, pf, prio, ilv, ldpos): a variant built for both head
// dimensions, or for one.  The position in the lists, one after the other, is the variant's id.
#define ATTN_VARIANTS_0(BOTH, D64, D128) \
    BOTH(64, 4, 1, 2, 1, 0, 4, 0, 0, 0) /* 0: the hand-written first schedule */ \
    BOTH(64, 4, 1, 2, 1, 0, 2, 0, 0, 0) \
    BOTH(64, 4, 1, 2, 1, 0, 6, 0, 0, 0) \
    BOTH(64, 4, 1, 2, 1, 0, 4, 1, 0, 0)

#define ATTN_VARIANTS_1(BOTH, D64, D128) \
    BOTH(64, 4, 1, 2, 0, 0, 4, 0, 0, 0) \
    BOTH(32, 4, 1, 2, 1, 0, 4, 0, 0, 0) \
    BOTH(32, 4, 1, 2, 1, 0, 2, 0, 0, 0)

#define ATTN_VARIANTS_2(BOTH, D64, D128) \
    BOTH(64, 8, 1, 1, 1, 0, 4, 0, 0, 0) \
    BOTH(64, 8, 1, 1, 1, 0, 6, 0, 0, 0) \
    BOTH(64, 8, 1, 1, 1, 1, 2, 0, 0, 0)

#define ATTN_VARIANTS_3(BOTH, D64, D128) \
    BOTH(64, 8, 1, 1, 1, 1, 4, 0, 0, 0) \
    BOTH(64, 8, 1, 1, 1, 1, 4, 1, 0, 0) \
    BOTH(64, 8, 1, 1, 0, 1, 4, 0, 0, 0)

#define ATTN_VARIANTS_4(BOTH, D64, D128) \
    BOTH(64, 4, 2, 1, 1, 0, 4, 0, 0, 0) \
    D64(128, 4, 1, 2, 1, 0, 4, 0, 0, 0) \
    D128(64, 8, 1, 1, 1, 2, 2, 1, 0, 0) /* 15, 16: MFMA work in both ping-pong clusters */ \
    D128(64, 8, 1, 1, 1, 2, 4, 1, 0, 0) \
    D64(64, 4, 1, 3, 1, 0, 4, 0, 0, 0) /* 17 .. 19: three free-running workgroups per CU (d = 64) */ \
    D64(64, 4, 1, 3, 1, 0, 4, 1, 0, 0)

#define ATTN_VARIANTS_5(BOTH, D64, D128) \
    D64(64, 4, 1, 3, 1, 0, 2, 1, 0, 0) \
    BOTH(64, 8, 1, 1, 1, 1, 4, 2, 0, 0) /* 20: ping-pong, priority raised while a wave issues tile loads */ \
    D128(64, 8, 1, 1, 0, 3, 4, 0, 0, 0) /* 21 .. 29: the interleaved order, tiles through registers */ \
    D128(64, 8, 1, 1, 0, 3, 4, 0, 0, 1) \
    D128(64, 8, 1, 1, 0, 3, 4, 0, 0, 2)

#define ATTN_VARIANTS_6(BOTH, D64, D128) \
    D128(64, 8, 1, 1, 0, 3, 2, 0, 0, 1) \
    D128(64, 8, 1, 1, 0, 3, 8, 0, 0, 1) \
    D128(64, 8, 1, 1, 0, 3, 4, 1, 0, 1) \
    D128(64, 8, 1, 1, 0, 3, 4, 2, 0, 1) \
    D128(64, 8, 1, 1, 0, 3, 4, 0, 1, 1) \
    D128(64, 8, 1, 1, 0, 3, 4, 0, 2, 1) \
    D128(64, 8, 1, 1, 1, 3, 4, 0, 0, 0) /* 30 .. 32: the interleaved order, tiles straight to LDS (32: one knob from 16, the lattice stays connected) */

#define ATTN_VARIANTS_7(BOTH, D64, D128) \
    D128(64, 8, 1, 1, 1, 3, 4, 0, 0, 1) \
    D128(64, 8, 1, 1, 1, 3, 4, 1, 0, 0) \
    D128(64, 8, 1, 1, 1, 1, 4, 1, 1, 0) /* 33, 34: ping-pong with other orders of the softmax instructions (a second pinned one, the compiler's) */ \
    D128(64, 8, 1, 1, 1, 1, 4, 1, 2, 0) \
    D128(64, 8, 1, 1, 1, 1, 4, 1, 0, 1) /* 35, 36: ping-pong with three K/V buffers, loads one tile further ahead, one barrier per tile */ \
    D128(64, 8, 1, 1, 1, 1, 2, 1, 0, 1)

#define ATTN_VARIANTS_8(BOTH, D64, D128) \
    BOTH(32, 4, 1, 2, 1, 0, 4, 0, 0, 1) /* 37, 38: free-running, the waves split the keys instead of the queries */ \
    BOTH(32, 8, 1, 1, 1, 0, 4, 0, 0, 1) \
    BOTH(64, 8, 1, 1, 1, 0, 4, 0, 0, 2) /* 39, 40: two wave groups of 128 query rows, four of 64, that split the keys of every tile */ \
    BOTH(128, 8, 1, 1, 1, 0, 4, 0, 1, 2)

#define ATTN_ALL_VARIANTS(BOTH, D64, D128) \
    ATTN_VARIANTS_0(BOTH, D64, D128) \
    ATTN_VARIANTS_1(BOTH, D64, D128) \
    ATTN_VARIANTS_2(BOTH, D64, D128) \
    ATTN_VARIANTS_3(BOTH, D64, D128) \
    ATTN_VARIANTS_4(BOTH, D64, D128) \
    ATTN_VARIANTS_5(BOTH, D64, D128) \
    ATTN_VARIANTS_6(BOTH, D64, D128) \
    ATTN_VARIANTS_7(BOTH, D64, D128) \
    ATTN_VARIANTS_8(BOTH, D64, D128)
