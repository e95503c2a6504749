// Host side of the fused GEMM + LeakyReLU library entry points: choice of the tile, variant table,
// argument checks, launches, timing, kernels loaded from code objects.  The kernels are in gemm_block.h
// (what gemm_lrelu launches) and gemm_kernel.h (the schedule search's table).
#include "../../include/gemm_lrelu.h"
#include "../../include/gemm_workspace.h"

#include <stdio.h>

#include "gemm_block.h"
#include "gemm_kernel.h"

namespace gemm {

// ---- host side -----------------------------------------------------------------------------
typedef void (*KernelFn)(Params);
struct Variant {
    int wk, bkw, stages, rot;
    KernelFn fn[2];  // by dtype
};
#define GEMM_VARIANT(WK, BKW, S, ROT) \
    { WK, BKW, S, ROT, { gemm_lrelu_kernel<attn::F16, Knobs<WK, BKW, S, ROT>>, gemm_lrelu_kernel<attn::BF16, Knobs<WK, BKW, S, ROT>> } }
static const Variant kVariants[] = {
    GEMM_VARIANT(4, 32, 8, 0),   // 0
    GEMM_VARIANT(4, 32, 4, 0),   // 1
    GEMM_VARIANT(4, 32, 10, 0),  // 2
    GEMM_VARIANT(4, 64, 4, 0),   // 3
    GEMM_VARIANT(4, 64, 3, 0),   // 4
    GEMM_VARIANT(8, 32, 4, 0),   // 5
    GEMM_VARIANT(8, 32, 3, 0),   // 6
    GEMM_VARIANT(2, 64, 8, 0),   // 7
    GEMM_VARIANT(2, 64, 4, 0),   // 8
    GEMM_VARIANT(2, 32, 8, 0),   // 9
    GEMM_VARIANT(1, 64, 8, 0),   // 10
    GEMM_VARIANT(2, 32, 4, 0),   // 11
    GEMM_VARIANT(4, 32, 4, 1),   // 12
    GEMM_VARIANT(4, 32, 8, 1),   // 13
    GEMM_VARIANT(4, 64, 3, 1),   // 14
    GEMM_VARIANT(4, 64, 4, 1),   // 15
    GEMM_VARIANT(8, 32, 3, 1),   // 16
    GEMM_VARIANT(8, 32, 4, 1),   // 17
    GEMM_VARIANT(4, 32, 3, 0),   // 18
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
constexpr int kDefault = 1;  // where the schedule search starts

// Tiles of `size` (a power of two) that cover n >= 1 (n may be the largest int).  Shifts, here and below: the choices
// run on every call, and their forty divisions took 0.1 us of it.
static int cover(int n, int size) { return 1 + ((n - 1) >> __builtin_ctz(size)); }
// Of any size.
static int cover_any(int n, int size) { return 1 + (n - 1) / size; }

static int check_args(const void* a, const void* b, const void* c, int M, int N, int K, int dtype, int variant_id) {
    if (!a || !b || !c) return GEMM_EINVAL;
    if (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) return GEMM_EINVAL;
    if (M < 1 || N < 8 || K < 8 || (N & 7) || (K & 7) || N >= (1 << 24) || K >= (1 << 24)) return GEMM_EINVAL;
    if ((long long)cover(M, 32) * cover(N, 32) > 0x7fffffffLL) return GEMM_EINVAL;
    if (dtype != GEMM_F16 && dtype != GEMM_BF16) return GEMM_EINVAL;
    // C is written while other workgroups still read A and B: it must not overlap them
    const uintptr_t c0 = (uintptr_t)c, c1 = c0 + (size_t)M * N * 2;
    const uintptr_t a0 = (uintptr_t)a, a1 = a0 + (size_t)M * K * 2, b0 = (uintptr_t)b, b1 = b0 + (size_t)K * N * 2;
    if ((c0 < a1 && a0 < c1) || (c0 < b1 && b0 < c1)) return GEMM_EINVAL;
    if (variant_id < 0 || variant_id >= kNumVariants) return GEMM_EINVAL;
    return GEMM_OK;
}

// ---- the tiles gemm_lrelu chooses from, with the cost model that chooses.  With n tiles on the busiest
// of the 256 compute units a tile shape takes about
//     ceil(K / kstage) * max(ceil(n / occ) * alone, n * full) + n * ends       (us)
// (alone: a stage of one tile, latency included; full: its share when the unit's tiles run side by
// side; ends: prologue and epilogue).  The three numbers are fitted to 85 shapes over M 1 .. 8192, N
// and K 64 .. 8192, ragged and whole, timed with every tile shape.  On 60 other shapes drawn from the same
// ranges the model's choice is 1.4 % (mean) above the best of the other seven, most of it the noise of calls of
// 3.5 us (above 5 us: 0.2 %, 8 % at most); always 32 x 32 tiles: 31 %.
// (The 64 x 64 tile on eight waves, two groups of four that split K, came later; its numbers are from 36 to 144 tiles
// with K from 2056 to 8200.  It pays while a unit has one tile: four waves there draw 60 to 65 GB/s, as much as one wave per SIMD
// has LDS reads and loads in flight for, eight 83.  768 x 768 x 3072 14.8 -> 12.2 us, 533 x 1152 x 3976 18.8 -> 16.3, 3802 x 200 x
// 2560 13.5 -> 12.9.  Rings of six and nine stages in place of three: nothing.
// The model takes it for 130 to 256 tiles from K of about 1100 on.  Time against the four waves', 500 shapes there, one set of buffers /
// five: with K a multiple of 64, where the rows of A start on whole lines, 0.98 / 0.97 at 1120, 0.95 at 1600, 0.90 / 0.92 from 2080 on; with
// other K 1.05 / 1.03 below 1440, 1.03 / 1.03 at 1600, 1.02 at 1920, 1.00 / 1.01 at 2080 and 0.99 / 1.00 from 2240 on (979 x 912 x 1272 8.35 us
// on four waves, 9.1 on eight; 3676 x 232 x 1456 8.6 and 9.5): there from 2112 on.  Above 2600: 0.96 over 56 shapes.)
struct BlockShape {
    int bm, bn, bk, wk, threads, occ;
    int ragged;  // the least K that it is taken for where K is no multiple of 64
    float alone, full, ends;
    struct Large { float alone, full, load, off, ends; } large;  // of the model for large calls (large_us)
    BlockFn fn[2], lines[2];  // by dtype; the second, where there is one, takes A by whole lines
    BlockFn split[2], split_lines[2];  // the same for a range of K (or null)
    int lines_from;  // the least K that whole lines are taken for
    bool off_lines(const void* a, int K) const;
    const BlockFn& whole_for(int dtype, const void* a, int K) const { return lines[dtype] && off_lines(a, K) ? lines[dtype] : fn[dtype]; }
    const BlockFn& range_for(int dtype, const void* a, int K) const { return split_lines[dtype] && off_lines(a, K) ? split_lines[dtype] : split[dtype]; }
};
template <class BL>
constexpr BlockShape block_shape(float alone, float full, float ends, BlockShape::Large large, int ragged = 0) {
    return {BL::BM, BL::BN, BL::BK, BL::WK, BL::WM * BL::WN * BL::WK * 64, BL::OCC, ragged, alone, full, ends, large,
            {gemm_block_kernel<Mfma16F16, BL>, gemm_block_kernel<Mfma16BF16, BL>}, {nullptr, nullptr}, {nullptr, nullptr}, {nullptr, nullptr}, 0};
}
// (the same tile with A by whole lines too; measured at `Block`)
template <class BL>
constexpr BlockShape lines_shape(float alone, float full, float ends, BlockShape::Large large, int ragged = 0, int lines_from = 768) {
    using Lines = Block<BL::BM, BL::BN, BL::BK, BL::WM, BL::WN, BL::WK, BL::NB, BL::OCC, true>;
    BlockShape s = block_shape<BL>(alone, full, ends, large, ragged);
    s.lines[0] = gemm_block_kernel<Mfma16F16, Lines>;
    s.lines[1] = gemm_block_kernel<Mfma16BF16, Lines>;
    s.lines_from = lines_from;
    return s;
}
template <class BL, bool LINES>
constexpr BlockShape with_split(BlockShape s) {
    s.split[0] = gemm_block_kernel<Mfma16F16, BL, true>;
    s.split[1] = gemm_block_kernel<Mfma16BF16, BL, true>;
    if constexpr (LINES) {
        using Lines = Block<BL::BM, BL::BN, BL::BK, BL::WM, BL::WN, BL::WK, BL::NB, BL::OCC, true>;
        s.split_lines[0] = gemm_block_kernel<Mfma16F16, Lines, true>;
        s.split_lines[1] = gemm_block_kernel<Mfma16BF16, Lines, true>;
    }
    return s;
}
// Whether A is taken by whole lines: its rows do not all start on one, and K is long enough for what that costs: the line that the first
// stage needs in addition, and in every stage a lane's choice between two of them.  Time without over time with, mean over 7 shapes each
// of K about 530 / 790 / 1050 / 1300 / 1560 / 2060, on buffers that exceed the caches and, in brackets, on the same ones:
//   64 x 128   0.98 / 1.00 / 1.02 / 1.04 / 1.03 / 1.04  (0.92 / 0.92 / 0.95 / 0.95 / 1.02 / 1.04): from 1280 on
//   128 x 128  1.01 / 1.05 / 1.06 / 1.08 / 1.10 / 1.15  (0.93 / 0.97 / 0.98 / 1.00 / 1.06 / 1.12)
//   128 x 256  1.03 / 1.04 / 1.04 / 1.06 / 1.07 / 1.07  (1.00 / 1.00 / 1.00 / 1.01 / 1.01 / 1.01)
//   256 x 256  1.03 / 1.05 / 1.06 / 1.07 / 1.08 / 1.09  (1.00 / 1.00 / 1.01 / 1.01 / 1.01 / 1.01)
//   192 x 128  1.04 / 1.10 / 1.11 / 1.17 / 1.20 / 1.21  (0.98 / 1.00 / 1.04 / 1.07 / 1.09 / 1.10)
//   192 x 256  1.01 / 1.04 / 1.03 / 1.03 / 1.02 / 1.05  (0.99 / 1.01 / 1.03 / 1.04 / 1.04 / 1.05)
//   96 x 64    taken from K of about 1100 on: 1.09 / 1.12 / 1.14 / 1.17  (1.03 / 1.03 / 1.09 / 1.14)
//   64 x 64 on eight waves, at 2600: 1.12 (1.08)
// (Not for the three smallest tiles: of the 64 x 64 tiles on four waves the longer ring costs the third workgroup of a unit, and the
// others are held by latency, 32 x 64: 0.93 to 1.02 of the time.)
// The base counts only where the order of the sums stays the same, so that the bits of C do not depend on where A lies: two groups
// of waves take alternate stages of K without whole lines and a run of stages each with them.  (Base 64 bytes off a line, us, without /
// with: 768 x 768 x 3072 13.5 / 12.2, 961 x 1096 x 2048 14.9 / 12.5, 247 x 4160 x 1664 10.9 / 9.6; on a line 12.0, 12.2 and 9.2.)
bool BlockShape::off_lines(const void* a, int K) const { return K >= lines_from && ((K & 63) || (wk == 1 && ((uintptr_t)a & 127))); }
static constexpr BlockShape kBlocks[] = {
    with_split<Block<32, 32, 32, 1, 1, 4, 4, 2>, false>(block_shape<Block<32, 32, 32, 1, 1, 4, 4, 2>>(0.21f, 0.22f, 0.5f, {0.275f, 0.253f, 0.02f, 0.15f, 0.17f})),
    with_split<Block<32, 64, 64, 1, 2, 2, 3, 2>, false>(block_shape<Block<32, 64, 64, 1, 2, 2, 3, 2>>(0.27f, 0.31f, 0.58f, {0.229f, 0.288f, 0.06f, 0.25f, 0.11f})),
    with_split<Block<64, 64, 64, 2, 2, 1, 3, 3>, false>(block_shape<Block<64, 64, 64, 2, 2, 1, 3, 3>>(0.24f, 0.17f, 0.22f, {0.215f, 0.181f, 0.25f, 0.16f, 0.f})),
    lines_shape<Block<64, 64, 64, 2, 2, 2, 4, 1>>(0.40f, 0.f, 0.9f, {0.310f, 0.f, 0.61f, 0.17f, 0.37f}, 2112),
    lines_shape<Block<64, 128, 64, 1, 4, 1, 3, 2>>(0.27f, 0.28f, 0.88f, {0.261f, 0.213f, 0.54f, 0.09f, 0.32f}, 0, 1280),
    with_split<Block<128, 128, 64, 2, 4, 1, 4, 1>, true>(lines_shape<Block<128, 128, 64, 2, 4, 1, 4, 1>>(0.41f, 0.f, 0.9f, {0.327f, 0.f, 0.62f, 0.09f, 1.02f})),
    lines_shape<Block<128, 256, 64, 2, 4, 1, 3, 1>>(0.64f, 0.f, 1.8f, {0.502f, 0.f, 0.80f, 0.f, 2.39f}),
    lines_shape<Block<256, 256, 64, 2, 4, 1, 2, 1>>(1.1f, 0.f, 3.0f, {0.982f, 0.f, 0.66f, 0.01f, 4.20f}),
};
// Tiles for large calls only: heights between the powers of two, for the calls whose tiles of those leave units
// without work or fill the units a little more than once.
static constexpr BlockShape kLargeBlocks[] = {
    lines_shape<Block<96, 64, 64, 2, 2, 2, 3, 1>>(0.f, 0.f, 0.f, {0.382f, 0.f, 0.60f, 0.15f, 0.77f}),
    with_split<Block<192, 128, 64, 2, 4, 1, 3, 1>, true>(lines_shape<Block<192, 128, 64, 2, 4, 1, 3, 1>>(0.f, 0.f, 0.f, {0.443f, 0.f, 0.56f, 0.05f, 1.83f})),
    lines_shape<Block<192, 256, 64, 2, 4, 1, 2, 1>>(0.f, 0.f, 0.f, {0.768f, 0.f, 0.77f, 0.06f, 2.94f}),
};

// 128 x 128 tiles with two workgroups on a unit, each with a ring of two stages, for the calls of more than one round and a K below
// 640: one multiplies while the other waits for its first stages or stores its tile, which is most of such a tile's time.  us, one
// workgroup / two: 2744 x 6672 x 112 19.9 / 15.4, 5826 x 2944 x 128 19.5 / 15.3, 4722 x 1584 x 104 9.1 / 7.4, 3499 x 5696 x 320 26.3 / 22.3,
// 3656 x 2080 x 448 12.2 / 10.8; over 37 shapes of 270 to 4032 tiles 1.10 to 1.39 at K up to 504, 1.02 to 1.25 up to 624, 0.99 to 1.13 from
// 704 on, and with longer K the shorter ring is the slower one (1504 x 5624 x 2272 0.88).
static constexpr BlockShape kShortBlock = block_shape<Block<128, 128, 64, 2, 4, 1, 2, 2>>(0.f, 0.f, 0.f, {0.579f, 0.395f, 0.39f, 0.05f, 0.41f});

constexpr unsigned long long kComputeUnits = 256;

static const BlockShape& choose_table(int M, int N, int K) {
    const BlockShape* best = &kBlocks[0];
    float best_us = 0.f;
    for (const BlockShape& s : kBlocks) {
        if ((long long)(s.bm - 1) * K * 2 + s.bk * 2 + 128 >= (long long)kBufferSize) continue;  // 32-bit offsets in a tile's rows
        if (K < s.ragged && (K & 63)) continue;
        const unsigned long long tiles = (unsigned long long)cover(M, s.bm) * cover(N, s.bn);
        const long long n = (tiles + kComputeUnits - 1) / kComputeUnits, stages = cover(K, s.bk * s.wk);
        const float alone = (float)(n <= s.occ ? 1 : (n + s.occ - 1) / s.occ) * s.alone, full = (float)n * s.full;
        const float us = (float)stages * (alone > full ? alone : full) + (float)n * s.ends;
        if (&s == &kBlocks[0] || us < best_us) best = &s, best_us = us;
    }
    return *best;
}

// ---- large calls: a second model, of more terms, puts the choice above against the tiles of kLargeBlocks.  With n tiles on the
// busiest unit, and f of the units' n rounds filled, a tile shape takes about
//     ceil(K / kstage) * max(ceil(n / occ) * alone, n * full) * (1 + load * f) * (1 + off) + n * ends + 2.7      (us)
// (load: what the units take from each other, in memory and clock; off: only where N is no multiple of 64, where every row of
// a piece of B begins and ends inside a line; 2.7: the launch).  Fitted to 190 shapes of 3e8 products and more, M 33 .. 8192, N 64 ..
// 8192 and K 256 .. 8192, a third of them with N and K multiples of 64, each timed with every tile, bfloat16; the
// standard deviation of the time over the model is 6 to 13 % by tile, so one of the new tiles has to be 5 % ahead, or, with a short
// K, where what is not a stage weighs more, 11 %.  Of those shapes 26 take another tile and run in 0.89 of the time (geometric
// mean; one takes longer, 3 %); of 250 drawn ones that do, each in 0.84 to 0.86 on several sets of buffers and on one (with whole lines of A where
// it has them), the slowest 1.01 on several (3219 x 5360 x 608) and 1.09 on one (2394 x 600 x 1240 8.0 -> 8.7; 13.8 -> 12.4 on several).  us:
//   96 x 64    247 x 4160 x 1704 12.0 -> 10.1, 3353 x 384 x 1264 9.6 -> 8.3, 1138 x 1088 x 2880 16.8 -> 14.0, 1000 x 1032 x 2056 14.2 -> 12.6
//   192 x 128  7798 x 2280 x 1000 52.8 -> 49.0, 1504 x 5624 x 2272 62.8 -> 51.8, 3430 x 1536 x 1856 25.3 -> 20.1
//   192 x 256  5963 x 1528 x 1272 36.0 -> 31.9, 7028 x 1216 x 4608 107.9 -> 93.7, 4297 x 2176 x 576 18.6 -> 16.2
static float large_us(const BlockShape& s, int M, int N, int K) {
    const unsigned long long tiles = (unsigned long long)cover_any(M, s.bm) * cover(N, s.bn);
    const long long n = (long long)((tiles + kComputeUnits - 1) / kComputeUnits), stages = cover(K, s.bk * s.wk);
    const float alone = (float)(n <= s.occ ? 1 : (n + s.occ - 1) / s.occ) * s.large.alone, full = (float)n * s.large.full;
    const float filled = (float)tiles / (float)(n * (long long)kComputeUnits);
    return (float)stages * (alone > full ? alone : full) * (1.f + s.large.load * filled) * (N & 63 ? 1.f + s.large.off : 1.f) + (float)n * s.large.ends + 2.7f;
}
static bool is_large(int M, int N, int K) { return M > 32 && K >= 256 && (double)M * N * K >= 3e8; }

static const BlockShape& choose_block(int M, int N, int K) {
    const BlockShape* best = &choose_table(M, N, K);
    if (best == &kBlocks[5] && K < 640 && (unsigned long long)cover(M, 128) * cover(N, 128) > kComputeUnits) best = &kShortBlock;
    if (!is_large(M, N, K)) return *best;
    float best_us = (K < 960 ? 0.89f : 0.95f) * large_us(*best, M, N, K);
#pragma unroll
    for (const BlockShape& s : kLargeBlocks) {
        if ((long long)(s.bm - 1) * K * 2 + s.bk * 2 + 128 >= (long long)kBufferSize) continue;
        const float us = large_us(s, M, N, K);
        if (us < best_us) best = &s, best_us = us;
    }
    return *best;
}

// ---- few tiles and a long K: the workgroups split K as well, and a second kernel adds their parts.
// A compute unit draws about 50 bytes a clock from memory however many loads it keeps in flight, so 128
// tiles on 128 units read the weights at half the card's rate and three tiles at a hundredth.  The second
// launch costs 2.1 us, so K has to be long.  Measured, whole / split, on one set of buffers and, in
// brackets, on sets that together exceed the last-level cache, us:
//   32 x 32   4 x 72 x 8136       9.9 / 6.3 (13.7 / 6.6)     2 x 880 x 7528     11.8 / 6.8 (20.1 / 8.5)
//             520 x 72 x 5192     7.7 / 7.7 (14.3 / 8.9)     222 x 280 x 4512    7.0 / 8.1 (13.4 / 9.1)
//   32 x 64   24 x 4096 x 4096   12.2 / 8.3 (21.1 / 12.6)    3 x 2480 x 5072    10.5 / 7.6 (16.7 / 10.1)
//             30 x 5592 x 4248   14.9 / 13.1 (21.4 / 17.8)   10 x 7472 x 7680   19.3 / 21.0 (28.4 / 24.6)
//   64 x 64   428 x 728 x 6168   22.4 / 16.3 (28.3 / 18.9)   170 x 456 x 4736   12.4 / 8.9 (14.1 / 9.5)
//             130 x 2448 x 6576  23.7 / 21.1 (30.0 / 27.0)   64 x 4096 x 4096   13.4 / 12.4 (20.7 / 14.8)
// Over 60 random shapes that the rule below takes: 1.2 times as fast on one set, 1.7 on fresh ones.
struct Split {
    const BlockShape* shape;
    int ranges, kc;           // ranges of kc values of k; 0: not split
    const BlockShape* whole;  // choose_block's, where the choice had to ask for it, or null
};
static Split choose_few(int M, int N, int K) {
    if (K < 4000) return {nullptr, 0, K, nullptr};
    auto tiles = [&](int s) { return (long long)cover(M, kBlocks[s].bm) * cover(N, kBlocks[s].bn); };
    const int s = tiles(0) <= 64 ? 0 : M <= 32 ? 1 : 2;
    const long long n = tiles(s);
    if (K < (s == 0 ? 4864 : M <= 64 ? 4000 : 4608) || n > (s == 1 ? 96 : 128) || K > (1 << 16)) return {nullptr, 0, K, nullptr};
    long long ranges = 256 / n;  // one workgroup per compute unit
    ranges = ranges < K / 512 ? ranges : K / 512;
    ranges = ranges < (s == 0 ? 16 : 8) ? ranges : s == 0 ? 16 : 8;
    const int step = kBlocks[s].bk * kBlocks[s].wk, kc = (int)((K + ranges - 1) / ranges + step - 1) / step * step;
    return {&kBlocks[s], (K + kc - 1) / kc, kc, nullptr};
}

// Large calls that the rule above leaves whole: tiles of 128 x 128 or 192 x 128, which read A and B the fewest times but are
// too few, or of 64 x 64, with K split into up to 8 ranges of 512 and more, one workgroup per unit.  The time is modelled as
//     stages of a range * alone * (1 + load * f) * (1 + off) + ends + 2.7 + second (the second launch) + per_mb per MB of parts   (us)
// and has to be 7 % below that of the call in one piece (64 x 64: 10 %).  At most 24 MiB of parts: a tile of 192 x 128 floats for each unit.  Whole / split, us, on sets of
// buffers that exceed the caches of the XCDs and, in brackets, on one:
//   128 x 128   969 x 664 x 7256  28.8 / 21.5     2335 x 216 x 7256  44.4 / 21.1 (33.5 / 18.7)    998 x 528 x 4552   21.8 / 16.0 (21.8 / 15.8)
//               118 x 7464 x 5592 35.7 / 27.2     91 x 5920 x 4112   23.5 / 18.3 (19.0 / 16.1)    2080 x 352 x 4504  20.7 / 17.3 (20.8 / 17.4)
//               a model's ratio of 0.89 and 0.94: 339 x 2256 x 4288  18.2 / 18.9,  451 x 1184 x 3648  14.7 / 16.2 (14.6 / 16.0; not taken)
//   192 x 128   180 x 2880 x 8192 37.5 / 23.8     167 x 3656 x 6536  40.9 / 23.6 (32.0 / 21.1)    3115 x 136 x 5296  30.2 / 19.3 (25.0 / 17.2)
//   64 x 64     162 x 800 x 4512  12.4 / 10.1 (12.0 / 8.9)    78 x 1264 x 3560  11.7 / 10.1 (10.4 / 8.7)    214 x 888 x 3960  13.4 / 11.2 (12.9 / 11.1)
//               not below 512 columns: 410 x 200 x 3800  11.8 / 8.1 (6.6 / 7.0),  2114 x 64 x 3992  11.4 / 9.8 (6.9 / 8.3)
// 250 drawn calls, split over whole, means on several sets (on one): 128 x 128 0.67 (0.81), 192 x 128 0.67 (0.82), 64 x 64 0.67 (0.86).  On
// several sets none is slower; on one 17 are by more than 3 %, those whose whole call finds A and B in the caches: 1420 x 176 x 4304
// 21.2 / 14.4 (9.7 / 12.7), 182 x 512 x 3456 15.0 / 9.1 (5.8 / 7.4).
// (128 x 256 and 256 x 128 tiles with K split: within 3 % of these; the parts in the accumulators' own order, 1 KB a store: the same.)
static Split choose_large_split(int M, int N, int K) {
    Split best = {nullptr, 0, K, nullptr};
    if (!is_large(M, N, K) || K > (1 << 16)) return best;
    static constexpr struct { const BlockShape* shape; float alone, load, off, ends, second, per_mb, ahead; double least; int width; } kRanges[] = {
        {&kBlocks[2], 0.179f, 0.67f, 0.08f, 0.55f, 2.5f, 0.22f, 0.90f, 3e8, 512},
        {&kBlocks[5], 0.325f, 0.59f, 0.01f, 1.28f, 2.3f, 0.40f, 0.93f, 1e9, 8},
        {&kLargeBlocks[1], 0.523f, 0.20f, 0.f, 1.21f, 2.3f, 0.40f, 0.93f, 1e9, 8}};
    const double products = (double)M * N * K;
    float best_us = 0.f, whole_us = 0.f;
#pragma unroll
    for (const auto& s : kRanges) {
        const long long tiles = (long long)cover_any(M, s.shape->bm) * cover(N, s.shape->bn);
        if (products < s.least || N < s.width || (long long)(s.shape->bm - 1) * K * 2 + s.shape->bk * 2 + 128 >= (long long)kBufferSize) continue;
        if (tiles * 2 > (long long)kComputeUnits || 1024 > K) continue;
        if (!best.whole) best.whole = &choose_block(M, N, K), whole_us = large_us(*best.whole, M, N, K);
        const float off = N & 63 ? 1.f + s.off : 1.f, parts_us = s.per_mb * 1e-6f * (float)M * (float)N, limit_us = s.ahead * whole_us;
        // no number of ranges comes below this (each takes 6 ns to look at)
        if ((float)K * (1.f / 512) * s.alone + s.ends + 2.7f + s.second + parts_us * 8.f >= 1.0001f * limit_us) continue;
#pragma unroll
        for (int r = 2; r <= 8; ++r) {
            if (tiles * r > (long long)kComputeUnits || r * 512 > K) break;
            const int kc = ((K + r - 1) / r + 63) / 64 * 64;
            if ((r - 1) * kc >= K) continue;
            const float filled = (float)((int)tiles * r) / (float)kComputeUnits;
            const float loop = (float)(kc / 64) * s.alone * (1.f + s.load * filled) * off;
            const float us = loop + s.ends + 2.7f + s.second + parts_us * (float)(4 * r);
            if (us < limit_us && (!best.ranges || us < best_us)) best = {s.shape, r, kc, best.whole}, best_us = us;
        }
    }
    return best;
}

static Split choose_split(int M, int N, int K) {
    const Split few = choose_few(M, N, K);
    return few.ranges ? few : choose_large_split(M, N, K);
}

static int launch_split(const Split& sp, const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype,
                        void* stream, void* workspace) {
    const BlockShape& s = *sp.shape;
    int ranges = sp.ranges;
    Arguments to(a, b, workspace, M, N, K, sp.kc, slope);
    unsigned chunks = (unsigned)((long long)M * N / 8);
    void* args[] = {&to.pointers_m_n, &to.k_kc_slope};
    void* sum_args[] = {&workspace, &c, &ranges, &chunks, &slope};
    const void* const sum = dtype == GEMM_F16 ? (const void*)gemm_sum_kernel<Mfma16F16> : (const void*)gemm_sum_kernel<Mfma16BF16>;
    const dim3 grid(cover_any(M, s.bm) * cover(N, s.bn) * ranges);
    if (hipLaunchKernel((const void*)s.range_for(dtype, a, K), grid, dim3(s.threads), args, 0, (hipStream_t)stream) != hipSuccess ||
        hipLaunchKernel(sum, dim3((chunks + 63) / 64), dim3(64), sum_args, 0, (hipStream_t)stream) != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ELAUNCH;
    }
    return GEMM_OK;
}

// (arguments checked by the caller)
static int launch_block(const BlockShape& s, const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream) {
    Arguments to(a, b, c, M, N, K, K, slope);
    void* args[] = {&to.pointers_m_n, &to.k_kc_slope};
    const dim3 grid(cover_any(M, s.bm) * cover(N, s.bn));
    if (hipLaunchKernel((const void*)s.whole_for(dtype, a, K), grid, dim3(s.threads), args, 0, (hipStream_t)stream) != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ELAUNCH;
    }
    return GEMM_OK;
}

static int launch(const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream,
                  int variant_id, hipFunction_t module_fn = nullptr) {
    const int rc = check_args(a, b, c, M, N, K, dtype, variant_id);
    if (rc != GEMM_OK) return rc;
    Params p;
    p.a = (const char*)a;
    p.b = (const char*)b;
    p.c = (uint16_t*)c;
    p.M = M, p.N = N, p.K = K;
    p.ntm = cover(M, 32), p.ntn = cover(N, 32);
    p.slope = slope;
    const Variant& v = kVariants[variant_id];
    void* args[] = {&p};
    const hipError_t e =
        module_fn ? hipModuleLaunchKernel(module_fn, (unsigned)(p.ntm * p.ntn), 1, 1, v.wk * 64, 1, 1, 0, (hipStream_t)stream, args, nullptr)
                  : hipLaunchKernel((const void*)v.fn[dtype], dim3(p.ntm * p.ntn), dim3(v.wk * 64), args, 0, (hipStream_t)stream);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ELAUNCH;
    }
    return GEMM_OK;
}

// ---- kernels loaded from code objects: the same kernel after its instructions were reordered
// outside the compiler.  A handle remembers which variant (launch shape) and type it replaces.
struct LoadedKernel {
    hipModule_t module = nullptr;
    hipFunction_t fn = nullptr;
    int variant_id = -1, dtype = 0;
};
constexpr int kMaxLoaded = 64;
static LoadedKernel g_loaded[kMaxLoaded];

template <class LaunchFn>
static int time_back_to_back(LaunchFn&& do_launch, void* stream, int warmup, int iters, float* ms_total) {
    if (!ms_total || iters < 1 || warmup < 0) return GEMM_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    for (int i = 0; i < warmup; ++i) {
        const int rc = do_launch();
        if (rc != GEMM_OK) return rc;
    }
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return GEMM_ELAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) {
        hipEventDestroy(e0);
        return GEMM_ELAUNCH;
    }
    int rc = hipEventRecord(e0, s) == hipSuccess ? GEMM_OK : GEMM_ELAUNCH;
    for (int i = 0; i < iters && rc == GEMM_OK; ++i) rc = do_launch();
    if (rc == GEMM_OK &&
        (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
         hipEventElapsedTime(ms_total, e0, e1) != hipSuccess))
        rc = GEMM_ELAUNCH;
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    return rc;
}

}  // namespace gemm

extern "C" {

int gemm_lrelu_num_variants(void) { return gemm::kNumVariants; }
int gemm_lrelu_default_variant(int, int, int) { return gemm::kDefault; }

int gemm_lrelu_variant_knobs(int variant_id, int* knobs) {
    if (!knobs || variant_id < 0 || variant_id >= gemm::kNumVariants) return GEMM_EINVAL;
    knobs[0] = gemm::kVariants[variant_id].wk;
    knobs[1] = gemm::kVariants[variant_id].bkw;
    knobs[2] = gemm::kVariants[variant_id].stages;
    knobs[3] = gemm::kVariants[variant_id].rot;
    return GEMM_OK;
}

int gemm_lrelu_variant(const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream,
                       int variant_id) {
    return gemm::launch(a, b, c, M, N, K, slope, dtype, stream, variant_id);
}

int gemm_lrelu(const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream) {
    const int rc = gemm::check_args(a, b, c, M, N, K, dtype, 0);
    return rc == GEMM_OK ? gemm::launch_block(gemm::choose_block(M, N, K), a, b, c, M, N, K, slope, dtype, stream) : rc;
}

static long long parts_bytes(const gemm::Split& sp, int M, int N) { return (long long)sp.ranges * M * N * 4; }

long long gemm_lrelu_workspace(int M, int N, int K) {
    return M < 1 || N < 8 || K < 8 ? 0 : parts_bytes(gemm::choose_split(M, N, K), M, N);
}

// (one look at the shape for the scratch memory, the tile and the launch: with a query for the bytes ahead of it the choice took 203 ns of
// a call of 512 x 512 x 2048 and 313 of 704 x 704 x 4000, now 60 and 89; without large calls' tiles and ranges it was 34)
int gemm_lrelu_with(const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream,
                    gemm_scratch_fn scratch, void* owner) {
    const int rc = gemm::check_args(a, b, c, M, N, K, dtype, 0);
    if (rc != GEMM_OK) return rc;
    const gemm::Split sp = gemm::choose_split(M, N, K);
    const long long need = parts_bytes(sp, M, N);
    void* const workspace = need && scratch ? scratch(owner, need) : nullptr;
    if (!workspace) return gemm::launch_block(sp.whole ? *sp.whole : gemm::choose_block(M, N, K), a, b, c, M, N, K, slope, dtype, stream);
    const uintptr_t w0 = (uintptr_t)workspace, w1 = w0 + need;
    auto meets = [&](const void* p, size_t bytes) { return w0 < (uintptr_t)p + bytes && (uintptr_t)p < w1; };
    if ((w0 & 15) || meets(a, (size_t)M * K * 2) || meets(b, (size_t)K * N * 2) || meets(c, (size_t)M * N * 2)) return GEMM_EINVAL;
    return gemm::launch_split(sp, a, b, c, M, N, K, slope, dtype, stream, workspace);
}

int gemm_lrelu_in(const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream,
                  void* workspace, long long workspace_bytes) {
    struct Given {
        void* p;
        long long bytes;
    } given = {workspace, workspace_bytes};
    const gemm_scratch_fn enough = [](void* owner, long long bytes) { return ((Given*)owner)->bytes < bytes ? nullptr : ((Given*)owner)->p; };
    return gemm_lrelu_with(a, b, c, M, N, K, slope, dtype, stream, enough, &given);
}

int gemm_lrelu_capturing(void* stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing((hipStream_t)stream, &status) != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return status != hipStreamCaptureStatusNone;
}

// The tile of C that gemm_lrelu uses for a shape (for the tests; not part of the interface).
int gemm_lrelu_block_of(int M, int N, int K, int* bm, int* bn) {
    if (!bm || !bn || M < 1 || N < 1 || K < 1) return GEMM_EINVAL;
    const gemm::BlockShape& s = gemm::choose_block(M, N, K);
    *bm = s.bm;
    *bn = s.bn;
    return GEMM_OK;
}

// The threads of its workgroups (the same).
int gemm_lrelu_block_threads_of(int M, int N, int K) { return M < 1 || N < 1 || K < 1 ? GEMM_EINVAL : gemm::choose_block(M, N, K).threads; }

// What gemm_lrelu (scratch 0) or gemm_lrelu_in with scratch memory (1) launches for A at `base` bytes behind a line (the same): tile,
// threads, workgroups per unit, 1 for A by whole lines, ranges of K (0: whole) and their kc.
int gemm_lrelu_launch_of(int M, int N, int K, int base, int scratch, int* out) {
    if (!out || M < 1 || N < 8 || K < 8 || base < 0) return GEMM_EINVAL;
    const gemm::Split sp = scratch ? gemm::choose_split(M, N, K) : gemm::Split{nullptr, 0, K, nullptr};
    const gemm::BlockShape& s = sp.ranges ? *sp.shape : gemm::choose_block(M, N, K);
    const void* const a = (const void*)(uintptr_t)base;
    const bool lines = sp.ranges ? s.range_for(0, a, K) == s.split_lines[0] : s.whole_for(0, a, K) == s.lines[0];
    const int what[7] = {s.bm, s.bn, s.threads, s.occ, lines, sp.ranges, sp.kc};
    for (int i = 0; i < 7; ++i) out[i] = what[i];
    return GEMM_OK;
}

int gemm_lrelu_time(const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream,
                    int variant_id, int warmup, int iters, float* ms_total) {
    return gemm::time_back_to_back([&] { return gemm::launch(a, b, c, M, N, K, slope, dtype, stream, variant_id); }, stream,
                                   warmup, iters, ms_total);
}

int gemm_lrelu_codeobj_load(const char* path, const char* kernel_name, int variant_id, int dtype) {
    using namespace gemm;
    if (!path || !kernel_name || variant_id < 0 || variant_id >= kNumVariants) return GEMM_EINVAL;
    if (dtype != GEMM_F16 && dtype != GEMM_BF16) return GEMM_EINVAL;
    int slot = -1;
    for (int i = 0; i < kMaxLoaded; ++i)
        if (!g_loaded[i].fn) {
            slot = i;
            break;
        }
    if (slot < 0) return GEMM_EINVAL;  // table full: unload something first
    // A failed runtime call leaves its status behind for whoever asks next: look at the file
    // first, and consume the status of a load that fails anyway.
    if (FILE* f = fopen(path, "rb")) fclose(f);
    else return GEMM_ELAUNCH;
    LoadedKernel lk;
    if (hipModuleLoad(&lk.module, path) != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ELAUNCH;
    }
    if (hipModuleGetFunction(&lk.fn, lk.module, kernel_name) != hipSuccess) {
        (void)hipGetLastError();
        hipModuleUnload(lk.module);
        return GEMM_ELAUNCH;
    }
    lk.variant_id = variant_id;
    lk.dtype = dtype;
    g_loaded[slot] = lk;
    return slot;
}

int gemm_lrelu_codeobj_unload(int handle) {
    using namespace gemm;
    if (handle < 0 || handle >= kMaxLoaded || !g_loaded[handle].fn) return GEMM_EINVAL;
    const hipError_t e = hipModuleUnload(g_loaded[handle].module);
    g_loaded[handle] = LoadedKernel();
    return e == hipSuccess ? GEMM_OK : GEMM_ELAUNCH;
}

int gemm_lrelu_codeobj(int handle, const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype,
                       void* stream) {
    using namespace gemm;
    if (handle < 0 || handle >= kMaxLoaded || !g_loaded[handle].fn || g_loaded[handle].dtype != dtype) return GEMM_EINVAL;
    return launch(a, b, c, M, N, K, slope, dtype, stream, g_loaded[handle].variant_id, g_loaded[handle].fn);
}

int gemm_lrelu_time_codeobj(int handle, const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype,
                            void* stream, int warmup, int iters, float* ms_total) {
    using namespace gemm;
    if (handle < 0 || handle >= kMaxLoaded || !g_loaded[handle].fn || g_loaded[handle].dtype != dtype) return GEMM_EINVAL;
    const LoadedKernel lk = g_loaded[handle];
    return time_back_to_back([&] { return launch(a, b, c, M, N, K, slope, dtype, stream, lk.variant_id, lk.fn); }, stream,
                             warmup, iters, ms_total);
}

int gemm_lrelu_tile_of_block(int block, int ntm, int ntn, int* tm, int* tn) {
    if (!tm || !tn || ntm < 1 || ntn < 1 || (long long)ntm * ntn > 0x7fffffffLL) return GEMM_EINVAL;
    if (block < 0 || block >= ntm * ntn) return GEMM_EINVAL;
    gemm::tile_of_block(block, ntm, ntn, *tm, *tn);
    return GEMM_OK;
}

}  // extern "C"
