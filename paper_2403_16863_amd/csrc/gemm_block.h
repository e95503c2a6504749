// Block-tiled fused GEMM + LeakyReLU for gfx950 (MI355X): the kernel behind gemm_lrelu.
//
// The 32 x 32 tiles of gemm_kernel.h read (32 + 32) * 2 bytes per k for 2048 flops: the compute
// unit's path from L2 (64 bytes per clock at most, about 80 GB/s per unit once all 256 pull) holds
// them below 300 TFLOP/s whatever the size.  Here the tile of C grows with the problem, from 32 x 32
// (few tiles: latency decides) to 256 x 256 (the matrix cores decide); the host picks (gemm_lrelu.hip).
//
//  * 16x16x32 MFMA, transposed product C^T += B^T A^T as in gemm_kernel.h: the A operand (n) comes
//    from the row-major B piece through the transposing LDS read, the B operand (m) is a 16-byte read
//    of an A row, and a lane of the accumulator holds four consecutive n of one row m of C.  (At the
//    power limit the 16x16x32 form runs 12 % faster than 32x32x16: half the accumulator traffic.)
//  * A ring of NB stages of BK k values in LDS, filled by direct global -> LDS buffer loads.  A stage is
//    BK / 32 steps; in each step a wave multiplies the fragments it read one step ago and reads those
//    of the next step, so there is no MFMA that waits for a read issued just before it.  The one
//    barrier of a stage stands ahead of its last step: by then every fragment of the stage is in
//    registers (its buffer is free, the loads of stage t + NB go there) and the wait in front of it,
//    counted, says that the wave's share of stage t + 1 has landed.
//  * The loads are dealt out between the MFMAs, because a wave is held while the texture path takes
//    one (about 16 clocks each).  With NB >= 3 they run from behind the barrier to the next one; with
//    NB = 2 they all go out in the step behind the barrier, or they would land late.  Measured,
//    4096 x 4096 x 4096, 256 x 256 tile, NB = 2: 98 us this way, 107 us spread; 128 x 128 tile with
//    NB = 4 on 2048 x 2048 x 2048: 18.7 us spread, 19.9 us in one step.
//  * BK = 64 because rows of A in a stage are then 128 bytes, a whole line: with 32 (64-byte rows) the
//    256 x 256 tile takes 102 us instead of 98 on the 4096 cube, the 128 x 256 tile 122 instead of 112.
//  * By whole lines (LINES), for rows of A that do not all start on a 128-byte line (K no multiple of 64, or a base off
//    the line): 64 k values of a row then lie in two lines, and a load instruction, 8 rows of 128 bytes, is 16 requests to the
//    texture path in place of 8, which is what holds every tile but the largest.  So a stage loads the line that the
//    row's next k values END in, of which the stage behind it reads the rest, and the ring of A holds one stage more.
//    A fragment read takes each 16-byte chunk from one stage or the next, by a lane's own row (rows 16 apart
//    agree), and a chunk's place in its LDS row goes by its k as in the form without lines: by its place in the line, the
//    fragment reads of odd K / 8 met in banks (2573 x 512 x 840: 304 k of 761 k LDS clocks, now none of 457 k).  bfloat16, us
//    before and after: 1394 x 7384 x 5480 144.7 -> 127.3 (256 x 256 tiles), 2622 x 1016 x 6224 72.3 -> 61.4 (128 x 128), 4096 x
//    4096 x 4088 114.7 -> 105.2, 5963 x 1528 x 1272 39.7 -> 36.2 (128 x 256), 1000 x 1032 x 2056 15.0 -> 14.2 (64 x 128), 1000 x
//    1024 x 2056 10.8 -> 10.1 (64 x 64 on eight waves).  Where the rows start on lines the longer ring costs 0 to 3 %: such calls
//    keep the ring without.  (B has no such form: its rows would need a line each in addition, so N off the line costs the
//    wider tiles least.)
//  * Workgroups of WK > 1 groups split K between the groups, each with a ring of its own (a group of
//    one wave then needs no barrier at all), and sum in LDS at the end, in group order.
//
// Measured (bfloat16, 4096 cube, 256 tiles of 256 x 256, one per compute unit): 98 us = 1400 TFLOP/s,
// from 480 us with the 32 x 32 tiles; a large product of the vendor library reaches 1280 on the same
// card.  The bound is the power limit (the clock falls to about 1.6 GHz), not the 64 LDS-bytes per clock
// of the loads (a 256 x 256 stage moves 64 KB in 2048 clocks of matrix work) nor the fragment reads.
#pragma once
#include "gemm_kernel.h"

namespace gemm {

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct Mfma16F16 {
    static __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(attn::f16x8, a), __builtin_bit_cast(attn::f16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ unsigned pack2(float a, float b) { return attn::F16::pack2(a, b); }
};
struct Mfma16BF16 {
    static __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(attn::bf16x8, a), __builtin_bit_cast(attn::bf16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ unsigned pack2(float a, float b) { return attn::BF16::pack2(a, b); }
};

template <int BM_, int BN_, int BK_, int WM_, int WN_, int WK_, int NB_, int OCC_, bool LINES_ = false>
struct Block {
    static constexpr int BM = BM_, BN = BN_;  // tile of C of one workgroup
    static constexpr int BK = BK_;            // k extent of one stage: 32 or 64
    static constexpr int WM = WM_, WN = WN_;  // its waves, as a grid over that tile
    static constexpr int WK = WK_;            // groups of WM x WN waves that split K between them, each with a ring of its own
    static constexpr int NB = NB_;            // stages of a ring
    static constexpr int OCC = OCC_;          // workgroups per compute unit
    static constexpr bool LINES = LINES_;     // A by whole lines (below)
};

// Size of the descriptors and, as a lane's offset, the mark of a chunk outside the matrix.  Real offsets
// stay below it: (BM - 1) * K * 2 and (BK - 1) * N * 2, checked by the host.
constexpr unsigned kBufferSize = 0x80000000u;

// SPLIT: workgroup b computes the products of k range b / (ntm ntn) (kc values of k, a multiple of 64 WK) into its
// part of the workspace, [range][M][N] floats; gemm_sum_kernel adds them.  `out` is C, or that workspace.
// The arguments arrive in scalar registers (see Params in attn_kernel.h), packed into two vectors: a launch costs the host 20 ns
// for every further argument, and calls that end sooner than the next launch can be made are bound by that.  Six
// arguments 2.74 us a launch, these two 2.62, one struct, which is not preloaded, 2.61.
typedef unsigned u32x8 __attribute__((ext_vector_type(8)));
struct Arguments {
    u32x8 pointers_m_n;   // A, B, `out`, M, N
    u32x4 k_kc_slope;
    Arguments(const void* a, const void* b, const void* out, int M, int N, int K, int kc, float slope) {
        const uint64_t p[3] = {(uint64_t)a, (uint64_t)b, (uint64_t)out};
        for (int i = 0; i < 3; ++i) pointers_m_n[2 * i] = (unsigned)p[i], pointers_m_n[2 * i + 1] = (unsigned)(p[i] >> 32);
        pointers_m_n[6] = (unsigned)M, pointers_m_n[7] = (unsigned)N;
        k_kc_slope = u32x4{(unsigned)K, (unsigned)kc, __builtin_bit_cast(unsigned, slope), 0u};
    }
};
typedef void (*BlockFn)(u32x8 pointers_m_n, u32x4 k_kc_slope);

template <class T, class BL, bool SPLIT = false>
__global__ __launch_bounds__(BL::WM * BL::WN * BL::WK * 64, (BL::OCC * BL::WM * BL::WN * BL::WK + 3) / 4) void gemm_block_kernel(
    u32x8 pointers_m_n, u32x4 k_kc_slope) {
    auto address = [&](int i) __attribute__((always_inline)) { return (uint64_t)pointers_m_n[2 * i + 1] << 32 | pointers_m_n[2 * i]; };
    const char* const a = reinterpret_cast<const char*>(address(0));
    const char* const b = reinterpret_cast<const char*>(address(1));
    // (named global: of an address made of two numbers the compiler does not know it)
    char __attribute__((address_space(1)))* const out = (char __attribute__((address_space(1)))*)address(2);
    const int M = (int)pointers_m_n[6], N = (int)pointers_m_n[7], K = (int)k_kc_slope[0], kc = (int)k_kc_slope[1];
    const float slope = __builtin_bit_cast(float, (unsigned)k_kc_slope[2]);
    constexpr int BM = BL::BM, BN = BL::BN, WM = BL::WM, WN = BL::WN, WK = BL::WK, NB = BL::NB;
    constexpr int NW = WM * WN, BK = BL::BK, KS = BK / 32;
    constexpr bool LINES = BL::LINES;
    constexpr int NA = NB + LINES;  // stages of the ring of A
    constexpr int TM = BM / WM, TN = BN / WN, MT = TM / 16, NT = TN / 16;
    constexpr int A_STAGE = BM * BK * 2, B_STAGE = BN * BK * 2;
    constexpr int LA = A_STAGE / 1024 / NW, LB = B_STAGE / 1024 / NW, LPS = LA + LB;
    constexpr int CPA = BK / 8, CPB = BN / 8, SLOTS = BN / 16;
    constexpr int RING = NA * A_STAGE + NB * B_STAGE;
    static_assert(LA * 1024 * NW == A_STAGE && LB * 1024 * NW == B_STAGE, "whole load instructions per wave");
    static_assert(NT % 2 == 0, "C is stored in pairs of 16-column tiles");
    static_assert(NB >= 2 && (NB - 1) * LPS <= 63, "the counted waits must fit s_waitcnt's field");
    static_assert(!LINES || BK == 64, "a line of A per row and stage");
    static_assert(WK == 1 || RING >= BM * BN * 4, "a ring also holds its group's partial sums");

    __shared__ __attribute__((aligned(256))) u32x4 smem[WK * RING / 16];
    char* const smem_b = reinterpret_cast<char*>(smem);

    const int lane = threadIdx.x & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave_wg / NW, wave = wave_wg % NW;
    const unsigned lds0 = lds_address(smem_b) + wk * RING;
    const int wm = wave / WN, wn = wave % WN;
    const int ntm = 1 + (M - 1) / BM, ntn = 1 + (N - 1) / BN;
    int tm, tn, range = 0, k0 = 0, K1 = K;  // (K1: end of the k range)
    if constexpr (SPLIT) {
        const int tiles = ntm * ntn;
        range = (int)blockIdx.x / tiles;
        tile_of_block((int)blockIdx.x - range * tiles, ntm, ntn, tm, tn);
        k0 = range * kc;
        K1 = min(K, k0 + kc);
    } else {
        tile_of_block((int)blockIdx.x, ntm, ntn, tm, tn);
    }
    const int m0 = tm * BM, n0 = tn * BN;
    // a group's k: every WK-th stage, or, by lines, a run of stages
    const int nkt = (K1 - k0 + WK * BK - 1) / (WK * BK), step = LINES ? BK : WK * BK;
    k0 += wk * (LINES ? nkt * BK : BK);
    if (LINES) K1 = min(K1, k0 + nkt * BK);
    // 16-byte chunks from the start of a line to a row of A.  (The same for rows 16 apart: K is a multiple of 8.  m0 and k0
    // do not change it either.)
    auto shift = [&](int row) __attribute__((always_inline)) { return LINES ? (int)(((unsigned)((uintptr_t)a >> 4) + (unsigned)row * ((unsigned)K >> 3)) & 7) : 0; };
    constexpr int BEFORE = LINES ? 7 * 16 : 0;  // bytes of a line that can lie ahead of a row

    // B piece: rows (k) of 32-byte slots, one slot per 16 columns.  The transposing read takes 4 rows x 32
    // bytes per 16 lanes and two such groups, 8 rows apart, per clock: the slot index is XOR-ed with a
    // code that puts those 8 rows into different eighths of the LDS's 256 bytes.
    auto b_code = [](int row) {
        const int hi = (row >> 3) & 1;
        return SLOTS >= 8 ? ((row & 3) | (hi << 2)) : SLOTS == 4 ? (((row >> 1) & 1) | (hi << 1)) : hi;
    };

    // What each lane loads: load i of a piece fills its physical chunks i*64 .. i*64+63 in wave order.
    // Rows past M and columns past N deliver zeros.
    unsigned voffA[LA], voffB[LB];
    int kA[LA], kB[LB];  // k of the lane's chunk inside a stage
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int ci = (wave * LA + i) * 64 + lane, row = ci / CPA;
        const int ch = (ci % CPA) ^ a_code<CPA>(row);  // of the row's k; by lines, the one of the line that lies as far behind the row's start
        kA[i] = (ch + shift(row) < CPA ? ch : ch - CPA) * 8;
        voffA[i] = m0 + row < M ? (unsigned)row * (unsigned)(K * 2) + (unsigned)(kA[i] * 2 + BEFORE) : kBufferSize;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int ci = (wave * LB + i) * 64 + lane, row = ci / CPB, pos = ci % CPB;
        const int col = ((((pos >> 1) ^ b_code(row)) << 1) | (pos & 1)) * 8;
        kB[i] = row;
        voffB[i] = n0 + col < N ? (unsigned)row * (unsigned)(N * 2) + col * 2 : kBufferSize;
    }
    const char* pa = a + (size_t)m0 * K * 2 + (size_t)k0 * 2 - BEFORE;
    const char* pb = b + (size_t)n0 * 2 + (size_t)k0 * N * 2;
    int kload = k0;  // first k of the next stage to be requested
    auto issue_a = [&](unsigned voff, int i, unsigned buf, u32x4 r) __attribute__((always_inline)) {
        attn::buffer_to_lds_16(r, voff, lds0 + buf * A_STAGE + (wave * LA + i) * 1024);
    };
    auto issue_b = [&](int i, unsigned buf, u32x4 r) __attribute__((always_inline)) {
        attn::buffer_to_lds_16(r, voffB[i], lds0 + NA * A_STAGE + buf * B_STAGE + (wave * LB + i) * 1024);
    };
    if constexpr (LINES) {  // line 0: nothing ahead of the row
        const u32x4 r = attn::buffer_resource(pa, kBufferSize);
#pragma unroll
        for (int i = 0; i < LA; ++i) issue_a(kA[i] < 0 || k0 + kA[i] >= K1 ? kBufferSize : voffA[i], i, 0, r);
        pa += BK * 2;
    }
    // the last, partial stage: chunks past K deliver zeros on both sides
    auto clip_tail = [&]() __attribute__((always_inline)) {
        if (kload + (1 + LINES) * BK > K1) {
#pragma unroll
            for (int i = 0; i < LA; ++i) if (kload + LINES * BK + kA[i] >= K1) voffA[i] = kBufferSize;
#pragma unroll
            for (int i = 0; i < LB; ++i) if (kload + kB[i] >= K1) voffB[i] = kBufferSize;
        }
    };
    auto advance = [&]() __attribute__((always_inline)) {
        pa += step * 2;
        pb += (size_t)step * N * 2;
        kload += step;
    };

    unsigned a_base[KS];
    bool a_next[KS];  // the chunk lies in the next line
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        const int chunk = j * 4 + (lane >> 4);
        a_next[j] = LINES && chunk + shift(lane & 15) >= CPA;
        a_base[j] = lds0 + (wm * TM + (lane & 15)) * (BK * 2) + ((chunk ^ a_code<CPA>(lane & 15)) * 16);
    }
    unsigned b_base[NT];
    {
        const int i16 = lane & 15, row = 8 * (lane >> 4) + (i16 >> 2);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            b_base[nt] = lds0 + NA * A_STAGE + row * (BN * 2) + (((wn * NT + nt) ^ b_code(row)) * 32) + (i16 & 3) * 8;
    }
    typedef const u32x4 __attribute__((address_space(3))) * lds_u32x4_ptr;
    auto a_address = [&](int j, unsigned buf) __attribute__((always_inline)) {
        return a_base[j] + (a_next[j] ? (buf + 1 == NA ? 0 : buf + 1) : buf) * A_STAGE;
    };
    auto read_a = [&](int mt, unsigned address) __attribute__((always_inline)) -> u32x4 {
        return *(lds_u32x4_ptr)(unsigned long)(address + mt * 16 * (BK * 2));
    };
    auto read_b = [&](int nt, int j, unsigned buf) __attribute__((always_inline)) -> u32x4 {
        const unsigned a = b_base[nt] + buf * B_STAGE + j * 32 * (BN * 2);
        const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(unsigned long)a));
        const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(unsigned long)(a + 4 * BN * 2)));
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    };

    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The loads l = 0 .. LPS-1 of a stage go out one by one between the MFMAs, from the step behind the
    // barrier on and through the steps ahead of the next one; load l behind MFMA number slot(l).
    constexpr int FIRST = NB == 2 ? 0 : KS == 1 ? MT * NT / 2 : MT * NT / 4, SPAN = (NB == 2 ? 1 : KS) * MT * NT;
    auto slot = [](int l) constexpr { return FIRST + l * (SPAN - FIRST) / LPS; };
    auto first_loads = [=]() constexpr { int n = 0; for (int l = 0; l < LPS; ++l) n += slot(l) < MT * NT; return n; };
    unsigned lbuf = 0, lbuf_a = 0;  // the stage being requested: its buffers (by lines, of A the line behind the stage's first) and sources
    u32x4 ra, rb;
    auto next_stage = [&](int t) __attribute__((always_inline)) {
        clip_tail();
        const unsigned size = t < nkt ? kBufferSize : 0u;
        ra = attn::buffer_resource(pa, size), rb = attn::buffer_resource(pb, size);
        advance();
    };
    auto issue = [&](auto l_c) __attribute__((always_inline)) {
        constexpr int l = decltype(l_c)::value;
        if constexpr (l < LA) issue_a(voffA[l], l, LINES ? lbuf_a : lbuf, ra);
        else issue_b(l - LA, lbuf, rb);
    };
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        next_stage(t);
        lbuf = t, lbuf_a = t + LINES;
        attn::static_for<LPS>([&](auto l_c) __attribute__((always_inline)) {
            if (t < NB - 1 || slot(decltype(l_c)::value) < MT * NT) issue(l_c);
        });
    }
    u32x4 fa[2][MT], fb[2][NT];
    auto meet = []() __attribute__((always_inline)) { if constexpr (NW > 1) asm volatile("s_barrier" ::: "memory"); };
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 2) * LPS + first_loads()) : "memory");
    meet();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) fb[0][nt] = read_b(nt, 0, 0);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) fa[0][mt] = read_a(mt, a_address(0, 0));

    unsigned buf = 0, line = 0;  // t % NB, and by lines t % NA
    auto stage = [&](auto par_c, int t) __attribute__((always_inline)) {
        const unsigned nbuf = buf + 1 == NB ? 0 : buf + 1, abuf = LINES ? line : buf, nabuf = abuf + 1 == NA ? 0 : abuf + 1;
        attn::static_for<KS>([&](auto j_c) __attribute__((always_inline)) {
            constexpr int j = decltype(j_c)::value, P = (decltype(par_c)::value + j) & 1, Q = P ^ 1;
            constexpr bool LAST = j == KS - 1;
            constexpr int nj = LAST ? 0 : j + 1;
            const unsigned rbuf = LAST ? nbuf : buf;
            if constexpr (LAST) {
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NB - 2) * LPS) : "memory");
                meet();
                next_stage(t + NB);
                lbuf = buf, lbuf_a = abuf;
            }
            const unsigned from_a = LINES ? a_address(nj, LAST ? nabuf : abuf) : 0;
            attn::static_for<MT * NT>([&](auto i_c) __attribute__((always_inline)) {
                constexpr int i = decltype(i_c)::value, mt = i / NT, nt = i % NT;
                acc[mt][nt] = T::mfma(fb[P][nt], fa[P][mt], acc[mt][nt]);
                // fragment reads spread over the first half of the step, loads over the second
                constexpr int R = MT + NT, STEPS = MT * NT / 2 > R ? R : (MT * NT + 1) / 2;
                attn::static_for<R>([&](auto r_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(r_c)::value;
                    if constexpr (i == q * STEPS / R) {
                        if constexpr (q < NT) fb[Q][q] = read_b(q, nj, rbuf);
                        else fa[Q][q - NT] = read_a(q - NT, LINES ? from_a : a_base[nj] + rbuf * A_STAGE);
                    }
                });
                attn::static_for<LPS>([&](auto l_c) __attribute__((always_inline)) {
                    if constexpr (slot(decltype(l_c)::value) == (LAST ? 0 : j + 1) * MT * NT + i) issue(l_c);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        buf = nbuf;
        if constexpr (LINES) line = nabuf;
    };
    if constexpr (KS % 2 == 0) {
        for (int t = 0; t < nkt; ++t) stage(std::integral_constant<int, 0>{}, t);
    } else {
        for (int t = 0; t < nkt; t += 2) {
            stage(std::integral_constant<int, 0>{}, t);
            stage(std::integral_constant<int, 1>{}, t + 1);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (stages past the end were requested empty)

    // ---- a lane holds rows n = 4g .. 4g+3 of each 16 x 16 tile of C^T; exchanged between the odd and even
    // 16-lane groups of two neighbouring tiles it has eight consecutive n: one 16-byte store.
    const int g = lane >> 4;
    auto act = [&](float x) __attribute__((always_inline)) { return x >= 0.f ? x : slope * x; };
    auto store_pair = [&](int mt, int nt, f32x4 x, f32x4 y) __attribute__((always_inline)) {
        const int m = m0 + wm * TM + mt * 16 + (lane & 15);
        if constexpr (SPLIT) {
            const int n = n0 + wn * TN + nt * 16 + g * 4;
            auto* const row = (float __attribute__((address_space(1)))*)out + ((size_t)range * M + m) * N;
            if (m < M && n < N) *(f32x4 __attribute__((address_space(1)))*)(row + n) = x;
            if (m < M && n + 16 < N) *(f32x4 __attribute__((address_space(1)))*)(row + n + 16) = y;
            return;
        }
        const auto s0 = __builtin_amdgcn_permlane16_swap(T::pack2(act(x[0]), act(x[1])), T::pack2(act(y[0]), act(y[1])), false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(T::pack2(act(x[2]), act(x[3])), T::pack2(act(y[2]), act(y[3])), false, false);
        const int n = n0 + wn * TN + nt * 16 + (g & 1) * 16 + (g >> 1) * 8;
        if (m < M && n < N) *(u32x4 __attribute__((address_space(1)))*)(out + ((size_t)m * N + n) * 2) = u32x4{s0[0], s1[0], s0[1], s1[1]};
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; nt += 2) store_pair(mt, nt, acc[mt][nt], acc[mt][nt + 1]);
    } else {
        constexpr int PAIRS = MT * NT / 2;
        if constexpr (NW > 1) __syncthreads();  // the ring is shared by the group's waves
        f32x4* const mine = reinterpret_cast<f32x4*>(smem_b + wk * RING + wave * (TM * TN * 4)) + lane;
#pragma unroll
        for (int i = 0; i < MT * NT; ++i) mine[i * 64] = acc[i / NT][i % NT];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < (PAIRS + WK - 1) / WK; ++q) {
            const int pr = q * WK + wk;
            if (PAIRS % WK != 0 && pr >= PAIRS) break;
            f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < WK; ++w) {
                const f32x4* part = reinterpret_cast<const f32x4*>(smem_b + w * RING + wave * (TM * TN * 4)) + lane;
                x += part[2 * pr * 64];
                y += part[(2 * pr + 1) * 64];
            }
            store_pair(pr / (NT / 2), pr % (NT / 2) * 2, x, y);
        }
    }
}

// C = leaky_relu(sum of the parts), in range order; one thread per eight consecutive elements.
template <class T>
__global__ __launch_bounds__(64) void gemm_sum_kernel(const float* parts, uint16_t* c, int ranges, unsigned chunks, float slope) {
    const unsigned i = blockIdx.x * 64 + threadIdx.x;
    if (i >= chunks) return;
    const f32x4* src = reinterpret_cast<const f32x4*>(parts) + (size_t)i * 2;
    f32x4 x = src[0], y = src[1];
#pragma unroll 4
    for (int r = 1; r < ranges; ++r) {
        src += (size_t)chunks * 2;
        x += src[0];
        y += src[1];
    }
    auto act = [&](float v) __attribute__((always_inline)) { return v >= 0.f ? v : slope * v; };
    reinterpret_cast<u32x4*>(c)[i] = u32x4{T::pack2(act(x[0]), act(x[1])), T::pack2(act(x[2]), act(x[3])),
                                           T::pack2(act(y[0]), act(y[1])), T::pack2(act(y[2]), act(y[3]))};
}

}  // namespace gemm
