// C ABI of the fused attention-forward library: argument checking, the table of
// schedule variants (the search space of Sec. 3.1 as compile-time instantiations of
// one kernel) and the event-timed measurement used as search feedback (Sec. 3.3).
#include "attn_variants.h"

#include <math.h>
#include <stdio.h>
#include <string.h>

#include "../../include/attn.h"

namespace {

using attn::Params;

struct Variant {
    int bn, nw, qb, occ, ldp, pipe, pf, prio, ilv, ldpos;  // knob values
    int coords[10];                                     // lattice coordinates (indices into the knob value lists)
    // kernels by [dtype][causal] for head dimension 64 and 128; null = not built for it
    const attn::KernelFn (*fn64)[2];
    const attn::KernelFn (*fn128)[2];
    int resident[2], mirrored;                          // what schedule_item takes, head dimension 64 and 128
    bool keysplit() const { return pipe == 0 && ldpos == 1; }
    int groups() const { return keysplit() ? nw : pipe == 0 && ldpos == 2 ? 2 << ilv : 1; }  // of waves that split the keys
    int bm() const { return 32 * qb * nw / groups(); }  // query rows of a work item
    attn::KernelFn fn(int d, int dtype, int causal) const {
        const attn::KernelFn(*f)[2] = d == 128 ? fn128 : fn64;
        return f ? f[dtype][causal ? 1 : 0] : nullptr;
    }
};

// Knob value lists (lattice axes): bn {32,64,128}  nw {4,8}  qb {1,2}  ldp {0,1}
// pipe {0,1,2,3}  pf {2,4,6,8}  prio {0,1,2}  dense {0,1}  ilv {0,1,2}  ldpos {0,1,2}.  The occupancy
// target follows from nw and qb (two workgroups per CU when one holds four waves of one query block
// each); dense = 1 asks for one workgroup more than that (three waves per SIMD: their vector
// instructions fill the issue slots a single wave leaves empty; d = 64 only, where the registers
// allow it).  ilv = how MFMA, LDS-read, transcendental and other vector instructions are grouped
// in the interleaved order (sched_group_barrier patterns), and for the ping-pong order the order of
// the softmax's vector instructions (0: every exponential followed by a multiply-add, an addition
// and every other time a conversion, pinned; 1: multiply-adds and exponentials alternating, then the
// sums and the conversion, pinned; 2: the compiler's own order); ldpos = where in the interleaved order's stream a
// wave issues its tile loads (all after the barrier, after fixed MFMA slots, after slots that
// depend on the wave): the position of the memory instructions, which is what Sec. 3.1 perturbs.
// On the ping-pong order ldpos 1 moves the tile loads one tile further ahead, into a third pair of
// buffers, which leaves one workgroup barrier per tile instead of two.  On the free-running order
// ldpos 1 is the key split: every wave loads tiles of its own, of the same 32 query rows; ldpos 2 the wave groups,
// which share every tile and split its keys (ilv 0: two groups, 1: four).
const char* const kKnobNames[] = {"bn", "nw", "qb", "ldp", "pipe", "pf", "prio", "dense", "ilv", "ldpos"};
const int kKnobSizes[] = {3, 2, 2, 2, 4, 4, 3, 2, 3, 3};
constexpr int kNumKnobs = 10;

// index helpers for the coordinate lists above
#define IDX_BN(x) ((x) == 32 ? 0 : (x) == 64 ? 1 : 2)
#define IDX_NW(x) ((x) == 4 ? 0 : 1)
#define IDX_QB(x) ((x) == 1 ? 0 : 1)
#define IDX_PF(x) ((x) / 2 - 1)
#define IDX_DENSE(NW, QB, OCC) ((OCC) - (((NW) == 4 && (QB) == 1) ? 2 : 1))
#define VARIANT_HEAD(BN, NW, QB, OCC, LDP, PIPE, PF, PRIO, ILV, LDPOS)                              \
    BN, NW, QB, OCC, LDP, PIPE, PF, PRIO, ILV, LDPOS,                                               \
    {IDX_BN(BN), IDX_NW(NW), IDX_QB(QB), LDP, PIPE, IDX_PF(PF), PRIO, IDX_DENSE(NW, QB, OCC), ILV, LDPOS}

#define VARIANT_DEAL(...) {attn::Knobs<__VA_ARGS__>::resident(64), attn::Knobs<__VA_ARGS__>::resident(128)}, attn::Knobs<__VA_ARGS__>::mirrored()

#define ROW_D64(...) {VARIANT_HEAD(__VA_ARGS__), attn::KernelSet<64, attn::Knobs<__VA_ARGS__>>::fn, nullptr, VARIANT_DEAL(__VA_ARGS__)},
#define ROW_D128(...) {VARIANT_HEAD(__VA_ARGS__), nullptr, attn::KernelSet<128, attn::Knobs<__VA_ARGS__>>::fn, VARIANT_DEAL(__VA_ARGS__)},
#define ROW_BOTH(...) \
    {VARIANT_HEAD(__VA_ARGS__), attn::KernelSet<64, attn::Knobs<__VA_ARGS__>>::fn, attn::KernelSet<128, attn::Knobs<__VA_ARGS__>>::fn, VARIANT_DEAL(__VA_ARGS__)},

const Variant kVariants[] = {ATTN_ALL_VARIANTS(ROW_BOTH, ROW_D64, ROW_D128)};
constexpr int kNumVariants = (int)(sizeof(kVariants) / sizeof(kVariants[0]));

// Compute units of the current device (queried once per device).
int cu_count() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

// Persistent workgroups: as many as the device keeps resident (occ per CU), a multiple of 8
// when every XCD can be given whole heads, never more than there are work items.
// The workgroups of the key split and of the wave groups are not persistent, one per item: they come in the order of the schedule
// as units become free (dealt out ahead, 4 heads x 8000 causal keys, d = 128, took 170 us instead of 122).
long long grid_size(int cus, const Variant& var, int BH, long long nqt) {
    const long long total = (long long)BH * nqt, resident = (long long)cus * var.occ;
    // (513 to 768 items: padded, which costs nothing that can be measured, 0.2 % at most; the schedule does not need it)
    if (var.groups() > 1) return total > 512 && total <= 768 ? 776 : total;
    if ((BH & 7) == 0 && (resident & 7) == 0) {
        const long long per_xcd_items = (long long)(BH >> 3) * nqt, per_xcd_wg = resident >> 3;
        return 8 * (per_xcd_items < per_xcd_wg ? per_xcd_items : per_xcd_wg);
    }
    return total < resident ? total : resident;
}

// A launch counts its threads in 32 bits (the grids of one workgroup per item are the only ones that can get there).
bool launchable(long long grid, const Variant& var) { return grid * var.nw * 64 <= 0xffffffffLL; }

bool aligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + nb && b0 < a0 + na;
}

// Everything that can be rejected without touching the device.
int check_args(const void* q, const void* k, const void* v, void* out, float* lse, int B, int H,
               int N, int d, float scale, int dtype, int variant_id) {
    if (!q || !k || !v || !out || !lse) return ATTN_EINVAL;
    if (B < 1 || H < 1 || N < 1) return ATTN_EINVAL;
    if (dtype != ATTN_F16 && dtype != ATTN_BF16) return ATTN_EINVAL;
    if (!isfinite(scale)) return ATTN_EINVAL;
    if (variant_id < 0 || variant_id >= kNumVariants) return ATTN_EINVAL;
    if (!aligned(q, 16) || !aligned(k, 16) || !aligned(v, 16) || !aligned(out, 16) || !aligned(lse, 4))
        return ATTN_EINVAL;
    if (d != 64 && d != 128) return ATTN_EUNSUPPORTED;
    const unsigned long long elems = (unsigned long long)B * H * N * d;
    if (elems > (1ull << 40)) return ATTN_EUNSUPPORTED;  // keeps every byte offset far inside 64 bits
    const size_t bytes = (size_t)elems * 2;
    if (overlaps(out, bytes, q, bytes) || overlaps(out, bytes, k, bytes) || overlaps(out, bytes, v, bytes))
        return ATTN_EINVAL;
    const size_t lse_bytes = (size_t)B * H * N * 4;
    if (overlaps(lse, lse_bytes, q, bytes) || overlaps(lse, lse_bytes, k, bytes) ||
        overlaps(lse, lse_bytes, v, bytes) || overlaps(lse, lse_bytes, out, bytes))
        return ATTN_EINVAL;
    return ATTN_OK;
}

// Launches the variant's own kernel, or, when `module_fn` is given, a kernel loaded from a
// code object that was derived from that variant's kernel (same arguments, same grid, same
// block, same LDS).
int launch(const void* q, const void* k, const void* v, void* out, float* lse, int B, int H, int N,
           int d, int causal, float scale, int dtype, void* stream, int variant_id,
           hipFunction_t module_fn = nullptr) {
    const int rc = check_args(q, k, v, out, lse, B, H, N, d, scale, dtype, variant_id);
    if (rc != ATTN_OK) return rc;
    const Variant& var = kVariants[variant_id];
    const attn::KernelFn fn = var.fn(d, dtype, causal);
    if (!fn) return ATTN_EUNSUPPORTED;
    const int bm = var.bm();
    const long long nqt = ((long long)N + bm - 1) / bm;
    const long long total = nqt * B * H;
    if (total > 0x7fffffffLL) return ATTN_EUNSUPPORTED;
    // the interleaved order addresses K and V of a head through a buffer descriptor: 32-bit byte offsets
    if (var.pipe == 3 && (long long)N * d * 2 > 0xffffffffLL) return ATTN_EUNSUPPORTED;
    // the key split too, and counts past the end of the keys (two rounds of its waves' tiles)
    if (var.keysplit() && (long long)N * d * 2 > 0x7fffffffLL) return ATTN_EUNSUPPORTED;

    Params p;
    p.q = (const uint16_t*)q;
    p.k = (const uint16_t*)k;
    p.v = (const uint16_t*)v;
    p.out = (uint16_t*)out;
    p.lse = lse;
    p.N = N;
    p.nqt = (int)nqt;
    p.BH = B * H;
    // The kernel tracks the running maximum of the raw dot products, which needs a
    // positive multiplier: a negative scale is moved into the sign of Q, a zero scale
    // into Q = 0.
    p.qmode = scale > 0.f ? 0 : (scale < 0.f ? 1 : 2);
    p.scale = scale > 0.f ? scale : (scale < 0.f ? -scale : 1.0f);
    p.scale_l2 = p.scale * 1.44269504088896340736f;
    const long long grid = grid_size(var.groups() > 1 ? 0 : cu_count(), var, p.BH, nqt);  // (one item per workgroup: no question of the device)
    if (!launchable(grid, var)) return ATTN_EUNSUPPORTED;
    p.grid = (int)grid;
    // The launch's own return code is used (not hipGetLastError, which can report a
    // stale, unrelated status left behind by another library's earlier call).
    // A code object gets the arguments as one block, which is laid out alike whether its kernel takes them one by
    // one or, built before they were split up, as one struct.
    attn::KernelArguments args = attn::kernel_arguments(p);
    size_t bytes = sizeof p;
    void* block[] = {HIP_LAUNCH_PARAM_BUFFER_POINTER, &p, HIP_LAUNCH_PARAM_BUFFER_SIZE, &bytes, HIP_LAUNCH_PARAM_END};
    const hipError_t e =
        module_fn ? hipModuleLaunchKernel(module_fn, (unsigned)grid, 1, 1, var.nw * 64, 1, 1, 0, (hipStream_t)stream, nullptr, block)
                  : hipLaunchKernel((const void*)fn, dim3((unsigned)grid), dim3(var.nw * 64), args.list, 0, (hipStream_t)stream);
    if (e != hipSuccess) fprintf(stderr, "attn: kernel launch failed: %s (%d), grid=%lld block=%d\n", hipGetErrorString(e), (int)e, grid, var.nw * 64);
    return e == hipSuccess ? ATTN_OK : ATTN_ELAUNCH;
}

// ---- kernels loaded from code objects (instruction-level schedule search).  A small fixed
// table; a slot records what the kernel was derived from so that a launch can be refused
// when the shape does not match.
struct LoadedKernel {
    hipModule_t module = nullptr;
    hipFunction_t fn = nullptr;
    int variant_id = -1, d = 0, dtype = 0, causal = 0;
};
constexpr int kMaxLoaded = 64;
LoadedKernel g_loaded[kMaxLoaded];

const LoadedKernel* loaded_for(int handle, int d, int dtype, int causal, int* rc) {
    if (handle < 0 || handle >= kMaxLoaded || !g_loaded[handle].fn) { *rc = ATTN_EINVAL; return nullptr; }
    const LoadedKernel& lk = g_loaded[handle];
    if (lk.d != d || lk.dtype != dtype || lk.causal != (causal ? 1 : 0)) { *rc = ATTN_EUNSUPPORTED; return nullptr; }
    *rc = ATTN_OK;
    return &lk;
}

// Shared by the two timing entry points: `warmup` untimed launches, then `iters` launches
// each bracketed by its own pair of events.
template <class LaunchFn>
int time_launches(LaunchFn&& do_launch, void* stream, int warmup, int iters, float* ms) {
    if (!ms || iters < 1 || warmup < 0) return ATTN_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    for (int i = 0; i < warmup; ++i) {
        const int rc = do_launch();
        if (rc != ATTN_OK) return rc;
    }
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return ATTN_ELAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) { hipEventDestroy(e0); return ATTN_ELAUNCH; }
    int rc = ATTN_OK;
    for (int i = 0; i < iters && rc == ATTN_OK; ++i) {
        if (hipEventRecord(e0, s) != hipSuccess) { rc = ATTN_ELAUNCH; break; }
        rc = do_launch();
        if (rc != ATTN_OK) break;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms[i], e0, e1) != hipSuccess)
            rc = ATTN_ELAUNCH;
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    return rc;
}


// ---- measurement aid: what the MFMA pipe sustains on this device.  Every wave issues
// independent 32x32x16 bf16 MFMAs back to back (four accumulators, operands fixed in
// registers, no memory traffic), two waves per SIMD.  With constant operands this reaches
// the clock-limited peak; with random operands the switching activity makes the device
// lower its clock (power management), which bounds what any kernel fed real data can reach.
__global__ __launch_bounds__(256) void mfma_ceiling_kernel(unsigned long long* counters, int iters, int random_operands) {
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    typedef float f32x16 __attribute__((ext_vector_type(16)));
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    u32x4 a[4], b[4];
    unsigned st = (blockIdx.x * 256 + threadIdx.x) * 2654435761u + 12345u;
    for (int n = 0; n < 4; ++n)
        for (int j = 0; j < 4; ++j) {
            st = st * 1664525u + 1013904223u;
            unsigned ra = st;
            st = st * 1664525u + 1013904223u;
            unsigned rb = st;
            if (!random_operands) {
                ra = rb = 0x3f803f80u;  // 1.0, 1.0
            } else {  // random sign and mantissa, exponent 126 or 127: magnitudes in [0.5, 2)
                ra = (ra & 0x807f807fu) | 0x3f003f00u | ((ra >> 3) & 0x00800080u);
                rb = (rb & 0x807f807fu) | 0x3f003f00u | ((rb >> 5) & 0x00800080u);
            }
            a[n][j] = ra;
            b[n][j] = rb;
        }
    f32x16 acc[4];
    for (int n = 0; n < 4; ++n)
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
    const unsigned long long c0 = clock64(), r0 = wall_clock64();
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int n = 0; n < 4; ++n)
            acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[n]), __builtin_bit_cast(bf16x8, b[n]), acc[n], 0, 0, 0);
    }
    const unsigned long long c1 = clock64(), r1 = wall_clock64();
    float sum = 0;
    for (int n = 0; n < 4; ++n)
        for (int v = 0; v < 16; ++v) sum += acc[n][v];
    if (blockIdx.x == 7 && threadIdx.x == 0) {
        counters[0] = c1 - c0;  // core clock cycles
        counters[1] = r1 - r0;  // ticks of the constant 100 MHz clock
    }
    if (sum == 1.2345e-30f) counters[2] = 1;  // keeps the accumulators alive
}

// ---- measurement aid: what a kernel with this path's instruction mix sustains.  Per 32x32x16 MFMA
// the tile loop reads one 1 KB operand fragment from LDS and issues, for the softmax of the one
// score element a lane owns per MFMA (a wave's 32 x 64 scores take 32 MFMAs), one multiply-add,
// one exp2, one add and half a conversion.  This
// kernel issues exactly that per MFMA, with random operands, fragments read from LDS four steps
// ahead, two waves per SIMD, and nothing else: no tile loads, no barriers, no masks, no item
// boundaries.  The device runs it at its power limit like the attention kernel, so the rate is
// the ceiling of the loop body on this device; mode 0 leaves out the LDS reads and the vector
// work (the MFMA-only rate with two waves per SIMD), mode 1 adds the LDS reads, mode 2 adds both.
template <int MODE>
__global__ __launch_bounds__(512) void mix_ceiling_kernel(unsigned long long* counters, int iters) {
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x16 __attribute__((ext_vector_type(16)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    __shared__ u32x4 lds[4096];  // 64 KB of random 16-bit patterns
    unsigned st = (blockIdx.x * 512 + threadIdx.x) * 2654435761u + 12345u;
    auto rnd = [&]() {  // random sign and mantissa, exponent 126 or 127: magnitudes in [0.5, 2)
        st = st * 1664525u + 1013904223u;
        return (st & 0x807f807fu) | 0x3f003f00u | ((st >> 3) & 0x00800080u);
    };
    for (int i = threadIdx.x; i < 4096; i += 512) lds[i] = u32x4{rnd(), rnd(), rnd(), rnd()};
    __syncthreads();
    u32x4 a[4], b[4];
    for (int n = 0; n < 4; ++n) {
        a[n] = u32x4{rnd(), rnd(), rnd(), rnd()};
        b[n] = u32x4{rnd(), rnd(), rnd(), rnd()};
    }
    f32x16 acc[4];
    for (int n = 0; n < 4; ++n)
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
    float x[16];
    for (int i = 0; i < 16; ++i) x[i] = -0.01f * (float)((st >> (i & 7)) & 255);
    float rs0 = 0.f, rs1 = 0.f;
    unsigned keep = 0;
    const char* lb = reinterpret_cast<const char*>(lds) + ((threadIdx.x * 16) & 0x3ff0);
    u32x4 ring[4];
    for (int n = 0; n < 4; ++n) ring[n] = *reinterpret_cast<const u32x4*>(lb + n * 16384);
    const unsigned long long c0 = clock64(), r0 = wall_clock64();
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            u32x4 av = a[n & 3];
            if constexpr (MODE >= 1) av = ring[n & 3];
            acc[n & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, b[n & 3]), acc[n & 3], 0, 0, 0);
            if constexpr (MODE >= 1) ring[n & 3] = *reinterpret_cast<const u32x4*>(lb + (n & 3) * 16384);
            if constexpr (MODE >= 2) {
                const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x[n], 0.127517f, -0.25f));
                if (n & 1) {
                    rs1 += e;
                    unsigned pk = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{x[n - 1], e}, bf16x2));
                    asm volatile("" : "+v"(pk));
                    keep ^= pk;
                } else {
                    rs0 += e;
                }
                asm volatile("" : "+v"(x[n]));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const unsigned long long c1 = clock64(), r1 = wall_clock64();
    float sum = rs0 + rs1;
    for (int n = 0; n < 4; ++n)
        for (int v = 0; v < 16; ++v) sum += acc[n][v];
    if (blockIdx.x == 7 && threadIdx.x == 0) {
        counters[0] = c1 - c0;  // core clock cycles
        counters[1] = r1 - r0;  // ticks of the constant 100 MHz clock
    }
    if (sum == 1.2345e-30f || keep == 0x12345678u) counters[2] = 1;  // keeps the results alive
}

// ---- measurement aid: the same work in the ping-pong form and nothing else.  Eight waves per workgroup,
// two per SIMD; per "tile" a wave runs one MFMA cluster (32 MFMAs, each with one 1 KB fragment read
// from LDS two steps ahead, the first 16 on four accumulators, the other 16 on two, like PV and S) and
// one vector cluster (per lane 32 multiply-adds, 32 exp2, 32 additions, 16 conversions, in the pinned
// order of the attention kernel), the waves 4..7 in the opposite order, with BARRIERS workgroup
// barriers per tile (2: after every cluster; 1: after every tile).  No tile loads, masks, item
// boundaries or epilogues: what is left is the structure itself, one wave of a SIMD feeding the
// matrix pipe while the other one issues vector instructions.
template <int BARRIERS>
__global__ __launch_bounds__(512) void pingpong_ceiling_kernel(unsigned long long* counters, int iters) {
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x16 __attribute__((ext_vector_type(16)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    __shared__ u32x4 lds[4096];  // 64 KB of random 16-bit patterns
    unsigned st = (blockIdx.x * 512 + threadIdx.x) * 2654435761u + 12345u;
    auto rnd = [&]() {  // random sign and mantissa, exponent 126 or 127: magnitudes in [0.5, 2)
        st = st * 1664525u + 1013904223u;
        return (st & 0x807f807fu) | 0x3f003f00u | ((st >> 3) & 0x00800080u);
    };
    for (int i = threadIdx.x; i < 4096; i += 512) lds[i] = u32x4{rnd(), rnd(), rnd(), rnd()};
    __syncthreads();
    u32x4 b[4];
    for (int n = 0; n < 4; ++n) b[n] = u32x4{rnd(), rnd(), rnd(), rnd()};
    f32x16 acc[6];
    for (int n = 0; n < 6; ++n)
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
    float x[32];
    for (int i = 0; i < 32; ++i) x[i] = -0.01f * (float)((st >> (i & 7)) & 255);
    float rs0 = 0.f, rs1 = 0.f;
    unsigned keep = 0;
    const char* lb = reinterpret_cast<const char*>(lds) + ((threadIdx.x * 16) & 0x3ff0);
    const bool grp_b = threadIdx.x >= 256;
    auto cluster_m = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(2);
        u32x4 ring[2];
        ring[0] = *reinterpret_cast<const u32x4*>(lb);
        ring[1] = *reinterpret_cast<const u32x4*>(lb + 16384);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < 32; ++n) {
            const int a = n < 16 ? (n & 3) : 4 + (n & 1);
            acc[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[n & 1]), __builtin_bit_cast(bf16x8, b[n & 3]), acc[a], 0, 0, 0);
            if (n + 2 < 32) ring[n & 1] = *reinterpret_cast<const u32x4*>(lb + ((n + 2) & 3) * 16384);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    auto cluster_v = [&]() __attribute__((always_inline)) {
        float xa = 0.f, xb = 0.f, ea = 0.f, eb = 0.f;
#pragma unroll
        for (int i = 0; i < 18; ++i) {  // pair i enters, pair i-1 in exp2, pair i-2 leaves
            float na = 0.f, nb = 0.f, fa = 0.f, fb = 0.f;
            if (i >= 1 && i <= 16) { fa = __builtin_amdgcn_exp2f(xa); __builtin_amdgcn_sched_barrier(0); }
            if (i < 16) { na = __builtin_fmaf(x[2 * i], 0.127517f, -0.25f); __builtin_amdgcn_sched_barrier(0); }
            if (i >= 2) { rs0 += ea; __builtin_amdgcn_sched_barrier(0); }
            if (i >= 2) {
                unsigned pk = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{ea, eb}, bf16x2));
                asm volatile("" : "+v"(pk));
                keep ^= pk;
                __builtin_amdgcn_sched_barrier(0);
            }
            if (i >= 1 && i <= 16) { fb = __builtin_amdgcn_exp2f(xb); __builtin_amdgcn_sched_barrier(0); }
            if (i < 16) { nb = __builtin_fmaf(x[2 * i + 1], 0.127517f, -0.25f); __builtin_amdgcn_sched_barrier(0); }
            if (i >= 2) { rs1 += eb; __builtin_amdgcn_sched_barrier(0); }
            xa = na; xb = nb; ea = fa; eb = fb;
        }
#pragma unroll
        for (int i = 0; i < 32; ++i) asm volatile("" : "+v"(x[i]));
    };
    const unsigned long long c0 = clock64(), r0 = wall_clock64();
    if (!grp_b) {
        for (int it = 0; it < iters; ++it) {
            cluster_m();
            if constexpr (BARRIERS == 2) __syncthreads();
            cluster_v();
            __syncthreads();
        }
    } else {
        for (int it = 0; it < iters; ++it) {
            cluster_v();
            if constexpr (BARRIERS == 2) __syncthreads();
            cluster_m();
            __syncthreads();
        }
    }
    const unsigned long long c1 = clock64(), r1 = wall_clock64();
    float sum = rs0 + rs1;
    for (int n = 0; n < 6; ++n)
        for (int v = 0; v < 16; ++v) sum += acc[n][v];
    if (blockIdx.x == 7 && threadIdx.x == 0) {
        counters[0] = c1 - c0;  // core clock cycles
        counters[1] = r1 - r0;  // ticks of the constant 100 MHz clock
    }
    if (sum == 1.2345e-30f || keep == 0x12345678u) counters[2] = 1;  // keeps the results alive
}

// ---- measurement aid: what the vector ALU sustains on the softmax's own instruction mix.  Per
// score element the one-pass softmax issues one fma (scale and shift), one exp2, one add (row sum)
// and half a conversion (two probabilities per packed 16-bit pair); this kernel issues exactly
// that mix on independent data from registers, 16 elements per round like one 32-key half tile,
// with a chosen number of waves per SIMD.  Ordinary scalar float code: the build keeps the compiler
// from forming packed-fp32 instructions.
__global__ __launch_bounds__(256) void valu_ceiling_kernel(unsigned long long* counters, int iters, float scale, float shift) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    float x[16];
    for (int i = 0; i < 16; ++i) x[i] = -0.01f * (float)((threadIdx.x * 16 + i) & 255);
    float rs0 = 0.f, rs1 = 0.f;
    unsigned keep = 0;
    const unsigned long long c0 = clock64(), r0 = wall_clock64();
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(x[i], scale, shift));
            const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(x[i + 1], scale, shift));
            rs0 += e0;
            rs1 += e1;
            unsigned pk = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{e0, e1}, bf16x2));
            asm volatile("" : "+v"(pk));  // the conversion is part of the mix: keep it
            keep ^= pk;
        }
        asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]));
        asm volatile("" : "+v"(x[8]), "+v"(x[9]), "+v"(x[10]), "+v"(x[11]), "+v"(x[12]), "+v"(x[13]), "+v"(x[14]), "+v"(x[15]));
    }
    const unsigned long long c1 = clock64(), r1 = wall_clock64();
    if (blockIdx.x == 7 && threadIdx.x == 0) {
        counters[0] = c1 - c0;  // core clock cycles
        counters[1] = r1 - r0;  // ticks of the constant 100 MHz clock
    }
    if (rs0 + rs1 == 1.2345e-30f || keep == 0x12345678u) counters[2] = 1;  // keeps the results alive
}

}  // namespace

extern "C" {

int attn_num_variants(void) { return kNumVariants; }

int attn_schedule_grid(int variant_id, int compute_units, int B, int H, int N) {
    if (variant_id < 0 || variant_id >= kNumVariants || compute_units < 1 || B < 1 || H < 1 || N < 1) return ATTN_EINVAL;
    const Variant& var = kVariants[variant_id];
    const int bm = var.bm();
    const long long nqt = ((long long)N + bm - 1) / bm, g = grid_size(compute_units, var, B * H, nqt);
    if ((long long)B * H > 0x7fffffffLL / nqt || !launchable(g, var)) return ATTN_EUNSUPPORTED;
    return (int)g;
}

// The item for either mask: causal + 2 * resident + 16 * mirrored (exported for the tests; not part of the interface).
int attn_schedule_item_of(int grid, int workgroup, int BH, int nqt, int round, int causal, int* bh, int* qt) {
    if (grid < 1 || workgroup < 0 || workgroup >= grid || BH < 1 || nqt < 1 || round < 0 || causal < 0 || !bh || !qt) return ATTN_EINVAL;
    int b = 0, q = 0;
    if (!attn::schedule_item(grid, workgroup, BH, nqt, round, b, q, (causal & 1) != 0, causal >> 1 & 7, causal >> 4)) return 0;
    *bh = b;
    *qt = q;
    return 1;
}

// The item that a launch of this variant takes (the same).
int attn_schedule_item_launched(int variant_id, int d, int causal, int grid, int workgroup, int BH, int nqt, int round, int* bh, int* qt) {
    if (variant_id < 0 || variant_id >= kNumVariants || (d != 64 && d != 128)) return ATTN_EINVAL;
    const Variant& v = kVariants[variant_id];
    return attn_schedule_item_of(grid, workgroup, BH, nqt, round, (causal ? 1 : 0) + 2 * v.resident[d == 128] + 16 * v.mirrored, bh, qt);
}

int attn_schedule_item(int grid, int workgroup, int BH, int nqt, int round, int* bh, int* qt) {
    return attn_schedule_item_of(grid, workgroup, BH, nqt, round, 1, bh, qt);
}

int attn_variant_supported(int variant_id, int d, int dtype, int causal) {
    if (variant_id < 0 || variant_id >= kNumVariants) return ATTN_EINVAL;
    if ((d != 64 && d != 128) || (dtype != ATTN_F16 && dtype != ATTN_BF16)) return 0;
    return kVariants[variant_id].fn(d, dtype, causal) != nullptr;
}

int attn_variant_desc(int variant_id, char* buf, int buflen) {
    if (variant_id < 0 || variant_id >= kNumVariants || !buf || buflen < 1) return ATTN_EINVAL;
    const Variant& v = kVariants[variant_id];
    return snprintf(buf, (size_t)buflen, "bm=%d bn=%d nw=%d qb=%d occ=%d ldp=%d pipe=%d pf=%d prio=%d ilv=%d ldpos=%d",
                    v.bm(), v.bn, v.nw, v.qb, v.occ, v.ldp, v.pipe, v.pf, v.prio, v.ilv, v.ldpos);
}

int attn_num_knobs(void) { return kNumKnobs; }

const char* attn_knob_name(int knob) { return (knob < 0 || knob >= kNumKnobs) ? nullptr : kKnobNames[knob]; }

int attn_knob_size(int knob) { return (knob < 0 || knob >= kNumKnobs) ? ATTN_EINVAL : kKnobSizes[knob]; }

int attn_variant_coords(int variant_id, int* coords) {
    if (variant_id < 0 || variant_id >= kNumVariants || !coords) return ATTN_EINVAL;
    for (int i = 0; i < kNumKnobs; ++i) coords[i] = kVariants[variant_id].coords[i];
    return ATTN_OK;
}

int attn_variant_from_coords(const int* coords) {
    if (!coords) return ATTN_EINVAL;
    for (int id = 0; id < kNumVariants; ++id)
        if (memcmp(kVariants[id].coords, coords, sizeof(int) * kNumKnobs) == 0) return id;
    return ATTN_EINVAL;
}

// Defaults chosen from the measured search over the variant table on MI355X: the
// two-cluster ping-pong order (256-row query tiles) wins for head_dim 128, in its form with
// three buffers, one barrier per tile and an LDS prefetch distance of 2 (about 1 % ahead of the
// two-buffer form, variant 11, on both long workloads, every time the two were timed alternately);
// long sequences with head_dim 64 run three free-running workgroups per compute unit, short ones
// have too few 256-row tiles to go round and run the free-running order on 128-row tiles.
// (Ids index kVariants.)
constexpr int kDefaultD128 = 36;
constexpr int kDefaultD64Long = 18;
constexpr int kDefaultD64Short = 3;

// The choice by the number of query tiles, measured on 256 units, us (heads x keys; g = tiles of 32 rows, the
// key split's; j = tiles of 128 rows).  Calls back to back, after 70 ms of the same: out of idle every one is up to
// 20 % slower, the key split most.
// The key split (37: four waves, two workgroups per compute unit, 38: eight waves, one) against the defaults; where two
// figures stand they are of two cards, which differ by up to 15 % here and by 1 % for the others:
//   d = 128          32 x 512 (g 512)  15.2 / 37: 11.0 / 38: 12.9     3 x 5000 (471)    87.4 / 60.5 / 66.0
//   d = 128, causal  32 x 512 (512)    15.8 /  8.9 / 12.6             6 x 5753 (1080)  101.2 / 83.2
//                    40 x 768 (960)    20.4 / 16.8, 18.2              48 x 768 (1152)   20.9 / 19.8, 22.1
//                    36 x 1024 (1152)  25.7 / 23.6                    32 x 1150 (1152)  26.8 / 25.0, 27.0
//                    64 x 350 (704)    13.8 / 12.0                    96 x 286 (864)    12.8 / 12.5
//   d = 64           24 x 512 (384)     8.9 /  6.7 /  8.5             4 x 5259 (660)    59.7 / 51.0
//                    40 x 554 (720)    10.2 / 10.3
//   d = 64, causal   8 x 4065 (1024)   47.2 / 33.6 / 36.7             24 x 2048 (1536)  27.2 / 24.4, 26.0
//                    64 x 512 (1024)   10.2 / 10.5                    64 x 600 (1216)   12.7 / 12.4
//                    64 x 620 (1280)   12.7 / 11.5                    70 x 610 (1400)   13.4 / 15.5
//                    72 x 640 (1440)   12.4 / 12.3, 13.8              60 x 768 (1440)   15.1 / 13.1
//                    64 x 768 (1536)   13.9 / 13.4, 15.3              48 x 1024 (1536)  16.9 / 15.6, 17.6
//                    48 x 905 (1392)   15.9 / 13.9, 15.7              40 x 1200 (1520)  18.6 / 17.0
// The lines lie where the slower card's two sides meet: a masked tile is half as heavy on average while the
// default's time is that of its heaviest; with few keys the split's start and its sum at the end count for more.
// Eight waves pay while each workgroup has a compute unit to itself (4 x 2048, d = 64: 9.5 against 10.9), and
// under a mask a little beyond, where the units' sums are uneven anyway (g; 37 / 38 at d = 64, at d = 128):
//   2 x 6000 (376)  26.1 / 25.2, 40.4 / 40.8    2 x 6656 (416)   29.2 / 30.7, 45.4 / 49.4    2 x 8000 (500)  36.8 / 41.7, 57.4 / 67.3
//   1 x 12000 (375) 47.9 / 38.1, 75.6 / 63.2    1 x 14000 (438)  57.5 / 51.9, 92.3 / 86.7    1 x 16000 (500) 68.6 / 66.2, 110.4 / 111.0
// d = 128 between the split and full rounds of 256-row tiles, on 128-row tiles of the free-running order (1):
//   12 x 1486 (j 144)  32.8 -> 29.6    64 x 329 (192)  14.2 -> 11.7    32 x 1011 (256)  25.5 -> 23.4;  33 x 1000 (264)  27.1 -> 34.2
//   a second round of few tiles either way: 10 x 7000 (550)  306 -> 298    96 x 751 (576)  47.5 -> 42.3    64 x 1250 (640)  68.7 -> 63.4
//   causal  128 x 256 (256)  12.3 -> 10.6    32 x 1270 (320)  29.6 -> 27.5    8 x 6159 (392)  112.3 -> 107.9    32 x 1984 (512)  45.8 -> 44.9
//           96 x 767 (576)  27.4 -> 26.6;  64 x 1196 (640)  35.2 -> 36.5
// d = 64, three workgroups per unit (18) against two (3): 4 x 16384 (j 512)  281 / 281, 6 x 10900 (516)  257 / 286, 24 x 2809 (528)  70.4 / 77.5;
//   causal  26 x 3000 (624)  43.1 / 41.5, 16 x 6000 (752)  85.4 / 83.4, 40 x 2400 (760)  39.2 / 39.6, 36 x 2800 (792)  45.5 / 46.8,
//           48 x 2300 (864)  38.2 / 40.2, 64 x 1706 (896)  34.3 / 35.9, 96 x 1397 (1056)  34.7 / 37.4.
// The wave groups (39: two groups, 128 rows; 40: four, 64 rows), one workgroup of eight waves per compute unit, two at
// d = 64: they pay where the tiles of their rows fill the units about once, under a mask, where they come by weight, up to twice;
// there 128-row tiles of four waves leave half the waves of a unit out and the key split reads K and V two to four times as
// often.  us, graphs of sixteen calls replayed in shuffled order; heads x keys (g, or tiles of 64 rows t, or j): the key split on four
// waves / 39 / 40 / the best of the long launches, on both sides of each line
//   d = 128          256 < g, t <= 256           12 x 617 (g 240)   8.4 / 13.6 / 10.6 / 15.2     15 x 558 (270)     10.6 / 12.9 / 10.5 / 14.5
//                                                32 x 512 (t 256)  11.1 / 12.9 / 10.6 / 13.6     24 x 666 (264)     13.3 / 15.7 / 22.5 / 17.3
//                    512 < g, j <= 256           32 x 1015 (j 256) 31.6 / 23.0 / 29.4 / 24.5     36 x 1024 (288)    37.3 / 39.2 / 41.0 / 28.9
//                    400 <= N for both           32 x 364 (g 384)   9.2 / 11.0 /  8.9 / 11.4     80 x 248 (640)     11.7 / 10.3 / 14.6 / 10.3
//                                                40 x 414 (g 520)  14.9 / 12.3 / 18.0 / 12.8
//   d = 128, causal  39: g > 700, N < 640        36 x 519 (g 612)  12.5 / 13.7 / 14.4 / 15.3     48 x 512 (768)     14.5 / 13.9 / 15.0 / 14.9
//                    g > 800, N < 900            28 x 819 (g 728)  16.2 / 17.0 / 16.9 / 19.9     40 x 660 (840)     16.2 / 15.5 / 16.6 / 16.9
//                    g > 960, N >= 900           28 x 970 (g 868)  19.8 / 20.1 / 20.5 / 23.6     28 x 1126 (1008)   23.4 / 22.4 / 22.4 / 26.2
//                    j <= 256, N < 1200          80 x 313 (j 240)  12.3 / 10.8 / 13.3 / 11.0     96 x 296 (288)     12.8 / 15.3 / 14.1 / 11.8
//                    j <= 480, N >= 1200         40 x 1308 (j 440) 38.2 / 32.2 / 38.8 / 32.4     40 x 1536 (480)    46.8 / 36.0 / 46.8 / 36.7
//                                                48 x 1349 (j 528) 51.2 / 43.1 / 50.0 / 35.8     18 x 3690 (522)   108.4 / 78.4 / 97.2 / 76.8
//                    40: g > 768, N >= 1500      14 x 1692 (g 742) 23.4 / 28.0 / 23.5 / 33.3     16 x 1617 (816)    22.9 / 26.6 / 22.4 / 31.6
//                    t <= 512                    16 x 2048 (t 512) 33.1 / 33.4 / 30.2 / 39.3     16 x 2061 (528)    32.7 / 32.9 / 35.1 / 39.8
//   d = 64           g > 300, N >= 960            6 x 1496 (g 282) 12.5 / 19.0 / 12.3 / 19.8      8 x 1280 (320)    11.1 / 16.5 / 10.8 / 16.9
//                                                15 x 896 (g 420)   9.1 / 13.1 /  9.0 / 13.0     16 x 1024 (512)    10.6 / 14.5 / 10.2 / 14.6
//                    t <= 256                     5 x 3142 (t 250) 24.3 / 35.4 / 22.2 / 39.3      9 x 2048 (288)    21.6 / 24.7 / 22.7 / 25.9
//                    (N >= 6000: g <= 768)        4 x 4599 (t 288) 42.8 / 49.4 / 42.5 / 55.6      3 x 6144 (288)    54.7 / 61.5 / 52.4 / 69.6
//                    g > 768, N >= 700           16 x 1536 (g 768) 19.2 / 20.9 / 19.7 / 21.5     12 x 2113 (804)    29.6 / 27.3 / 25.6 / 29.8
//                    (860 for heads that divide  38 x 700 (g 836)  13.7 / 13.0 / 13.1 / 13.9     36 x 768 (864)     13.9 / 12.7 / 12.6 / 13.2
//                    by 8: on one XCD each       40 x 768 (g 960)  14.3 / 13.3 / 13.1 / 13.0     32 x 830 (832)     15.2 / 14.4 / 14.4 / 14.2
//                    in the long launches)       40 x 694 (g 880)  13.6 / 12.9 / 12.9 / 12.6     32 x 878 (896)     15.4 / 14.4 / 14.0 / 14.2
//                    j <= 256                    32 x 969 (j 256)  17.0 / 16.1 / 15.4 / 16.1     18 x 2048 (288)    34.8 / 38.1 / 34.5 / 33.3
//   d = 64, causal   g > 1536, 1250 <= N < 2000  28 x 1697 (1512)  23.5 / 25.9 / 23.6 / 27.3     28 x 1943 (1708)   27.8 / 28.7 / 27.1 / 30.7
//                    g > 960, N >= 2000           9 x 3376 (g 954) 25.4 / 37.7 / 26.4 / 42.7     15 x 2141 (1005)   20.3 / 26.5 / 20.1 / 29.8
//                    g <= 1800, N < 2000         36 x 1500 (1692)  23.4 / 23.8 / 23.3 / 25.1     46 x 1300 (1886)   26.3 / 23.8 / 24.2 / 24.6
//                    g <= 2050, N < 4000         24 x 2637 (1992)  37.5 / 36.0 / 35.4 / 38.2     28 x 2461 (2156)   39.9 / 37.8 / 37.9 / 37.4
//                    g <= 2200, N >= 4000         8 x 8634 (2160) 110.1 / 102  / 94.1 / 110.0    18 x 4096 (2304)   67.6 / 57.2 / 57.8 / 58.6
// (Not taken, though measured: 40 for one head from 12000 keys at d = 64, 1 x 12500 75.2 / 68.7.)
// d = 64, causal, 37 / 3 / 18: 64 x 500 (1024)  8.8 / 10.5 / 10.5   120 x 400 (g 1560)  15.2 / 10.1 / 10.1;  3 and 18 between j = 410 and 512: alike,
// within 1 %; beyond, up to 1600 keys: 112 x 640 (j 560) 16.3 / 13.9.
// Eight waves (38) against four (37) where each has a unit to itself: d = 64 8 x 427 (112) 5.5 / 5.3, 12 x 224 (84) 4.3 / 4.5;
// causal 8 x 199 4.3 / 4.2, 8 x 1957 (496) 12.5 / 11.2, 3 x 3663 (345) 17.5 / 16.0, 8 x 2076 (520) 13.3 / 13.1; d = 128 causal
// 4 x 2085 (264) 17.4 / 15.1, 5 x 2002 (315) 17.7 / 16.6, 4 x 2682 (336) 21.1 / 19.8, 4 x 2871 (360) 22.5 / 22.6; d = 128 9 x 790 (225) 9.7 / 9.1, 12 x
// 617 (240) 8.4 / 8.2, 2 x 4096 (256) 30.8 / 27.0, 10 x 819 (260) 12.9 / 16.1.
constexpr int kKeySplit4 = 37, kKeySplit8 = 38, kGroups2 = 39, kGroups4 = 40, kRows128 = 1;

// d = 128 beyond those lines: 128-row tiles (two workgroups of four waves per unit) against 256-row tiles (one of eight), where
// neither has many rounds and the larger tiles leave more of the last one, or of a head's last tile, empty.  Time of the busiest
// unit, us, with tiles of 64 keys per item (nk; causal: of the items that a unit is dealt, heaviest first, forward and backward, in sum):
//   256 rows   1.40 nk + 9.4 a round;                                               causal  1.51 per tile + 8.05 an item
//   128 rows   1.70 nk + 6.9 a round (0.86 nk with one workgroup on every unit);    causal  1.87 per tile of a workgroup's mean share + 6.17 a round
// Fitted to 181 and 188 launches of 24 to 128 heads, 257 to 8000 keys and up to 16 rounds (standard deviation of the time over the
// model 3 to 7 %).  128 rows have to be 6 % ahead; under a mask that is the model of heads that divide by 8, which stay on an XCD
// each (schedule_item).  Of other heads, whose tiles every XCD reads, 128 rows take up to 1.16 of the time where they are modelled 6 to
// 18 % ahead (45 launches; 12 of them more than 1.02 on one set of buffers and on several), unless the keys are few: from 640 on
// they have to be 18 % ahead.  Time against 256 rows', one set / several, mean and largest: without a mask (173 launches) 0.89 / 0.87, 1.07 /
// 1.03; under it 0.92 / 0.91, 1.00 / 0.99 (70 of heads that divide by 8) and 0.94 / 0.91, 1.02 / 0.99 (48 others).  256 / 128 rows, us, several sets:
//   96 x 599  43.9 / 27.1    128 x 642  48.5 / 40.4    128 x 1041  97.9 / 86.7    24 x 3790  172 / 170 (not taken, as all beyond 3000 keys)
//   causal  128 x 561  32.9 / 27.5    96 x 846  38.0 / 32.7    128 x 1101  70.1 / 60.5    48 x 2111  69.5 / 65.7    64 x 1545  57.9 / 55.8
//           17 x 4256  98.9 / 90.7    119 x 568  32.2 / 28.7    not taken: 43 x 2059  65.2 / 71.7    90 x 1811  110.7 / 117.8
static bool rows128_sooner(long long heads, int N, int causal) {
    if (N <= 256 || N > (causal ? 8000 : 3000)) return false;
    const long long nq = (N + 255) / 256, items = heads * nq, rounds = (items + 255) / 256;
    const long long n128 = (N + 127) / 128, j = heads * n128;
    if (rounds > 16) return false;
    const float nk = (float)((N + 63) / 64);
    if (!causal) {
        const long long full = j / 512, rest = j % 512;
        const float t128 = (float)full * (1.70f * nk + 6.9f) + (rest ? (rest <= 256 ? 0.86f : 1.70f) * nk + 6.9f : 0.f);
        return t128 < 0.94f * (float)rounds * (1.40f * nk + 9.4f);
    }
    float t256 = 0.f;
    for (int unit = 0; unit < 256; unit += 255) {
        float t = 0.f;
        for (long long r = 0; r < rounds; ++r) {
            const long long rank = r * 256 + (r & 1 ? 255 - unit : unit);
            if (rank >= items) break;
            const long long keys = (nq - rank / heads) * 256;
            t += 1.51f * (float)(((keys < N ? keys : N) + 63) / 64) + 8.05f;
        }
        t256 = t > t256 ? t : t256;
    }
    const float tiles = (float)heads * ((float)(n128 * (n128 - 1)) + nk);
    return 1.87f * tiles / 512.f + 6.17f * (float)((j + 511) / 512) < (heads % 8 == 0 || N < 640 ? 0.94f : 0.82f) * t256;
}

static int choose_variant(long long heads, int N, int d, int causal) {
    const long long g = heads * ((N + 31LL) / 32), t = heads * ((N + 63LL) / 64), j = heads * ((N + 127LL) / 128);
    const int most = d == 128 ? (!causal ? 512 : N < 768 ? 736 : N < 1024 ? 1056 : 1152)
                              : !causal ? (N < 640 ? 704 : 768) : N < 300 ? 960 : N < 600 ? 1100 : N < 768 ? 1280 : N < 1200 ? 1440 : 1536;
    // the wave groups
    if (d == 128 && !causal) {
        if (N >= 400 && g > 256 && t <= 256) return kGroups4;
        if (N >= 400 && g > 512 && j <= 256) return kGroups2;
    } else if (d == 128) {
        if (N >= 1500 && g > 768 && t <= 512) return kGroups4;
        if (N >= 300 && g > (N < 640 ? 700 : N < 900 ? 800 : 960) && j <= (N < 1200 ? 256 : 480)) return kGroups2;
    } else if (!causal) {
        if (N >= 960 && N < 12000 && g > 300 && (t <= 256 || (N >= 6000 && g <= most))) return kGroups4;
        if (N >= (heads & 7 ? 700 : 860) && g > most && j <= 256) return N >= 960 ? kGroups4 : kGroups2;
    } else if (N >= 1250 && g > (N < 2000 ? most : 960) && g <= (N < 2000 ? 1800 : N < 4000 ? 2050 : 2200)) {
        return kGroups4;
    }
    // the key split: eight waves up to the line `alone`
    const int alone = causal && N >= 6000 ? (N >= 12000 ? 512 : 384)
                      : causal && d == 64 && N >= 1200 && N <= 5000 ? 512
                      : causal && d == 128 && N >= 2000 && N <= 5500 ? 352 : 256;
    if (g <= most) return N >= (d == 128 ? 512 : causal ? 160 : 400) && g <= alone ? kKeySplit8 : kKeySplit4;
    if (d == 128) return (causal ? j <= 576 : j <= 256 || (j > 512 && j <= 640)) || rows128_sooner(heads, N, causal) ? kRows128 : kDefaultD128;
    return j > (!causal ? 512 : N >= 256 && N < 1600 ? 410 : 755) ? kDefaultD64Long : kDefaultD64Short;
}

int attn_choose_variant(int B, int H, int N, int d, int dtype, int causal) {
    if (B < 1 || H < 1 || N < 1 || (dtype != ATTN_F16 && dtype != ATTN_BF16)) return ATTN_EINVAL;
    if (d != 64 && d != 128) return ATTN_EUNSUPPORTED;
    return choose_variant((long long)B * H, N, d, causal);
}

int attn_default_variant(int N, int d, int dtype, int causal) {
    (void)dtype;
    if (N < 1024) return choose_variant(8, N, d, causal);
    return d == 128 ? kDefaultD128 : N >= 2048 ? kDefaultD64Long : kDefaultD64Short;
}

int attn_fwd_variant(const void* q, const void* k, const void* v, void* out, float* lse, int B, int H,
                     int N, int d, int causal, float scale, int dtype, void* stream, int variant_id) {
    return launch(q, k, v, out, lse, B, H, N, d, causal, scale, dtype, stream, variant_id);
}

// ---- deployed schedules (Sec. 4.1): what attn_fwd launches instead of the default, by shape
// class.  A small fixed table searched newest first; handle >= 0 names a loaded code object.
struct Deployment {
    bool used = false;
    int variant_id = -1, handle = -1, d = 0, dtype = 0, causal = 0, n_min = 0, n_max = 0;
};
constexpr int kMaxDeployed = 16;
static Deployment g_deployed[kMaxDeployed];
static int g_num_deployed = 0;

static const Deployment* deployed_for(int N, int d, int dtype, int causal) {
    for (int i = g_num_deployed - 1; i >= 0; --i) {
        const Deployment& e = g_deployed[i];
        if (e.used && e.d == d && e.dtype == dtype && e.causal == (causal ? 1 : 0) && N >= e.n_min && N <= e.n_max) return &e;
    }
    return nullptr;
}

static int add_deployment(const Deployment& e) {
    if (g_num_deployed == kMaxDeployed) {  // reuse the room of removed entries, keeping the order
        int n = 0;
        for (int i = 0; i < kMaxDeployed; ++i)
            if (g_deployed[i].used) g_deployed[n++] = g_deployed[i];
        for (int i = n; i < kMaxDeployed; ++i) g_deployed[i] = Deployment();
        g_num_deployed = n;
        if (n == kMaxDeployed) return ATTN_EUNSUPPORTED;
    }
    g_deployed[g_num_deployed++] = e;
    return ATTN_OK;
}

int attn_fwd(const void* q, const void* k, const void* v, void* out, float* lse, int B, int H, int N,
             int d, int causal, float scale, int dtype, void* stream) {
    if (g_num_deployed > 0) {
        if (const Deployment* e = deployed_for(N, d, dtype, causal)) {
            const int rc = launch(q, k, v, out, lse, B, H, N, d, causal, scale, dtype, stream, e->variant_id,
                                  e->handle >= 0 ? g_loaded[e->handle].fn : nullptr);
            if (rc != ATTN_EUNSUPPORTED) return rc;
        }
    }
    return launch(q, k, v, out, lse, B, H, N, d, causal, scale, dtype, stream,
                  choose_variant((long long)B * H, N, d, causal));
}

int attn_deploy_variant(int variant_id, int d, int dtype, int causal, int n_min, int n_max) {
    if (variant_id < 0 || variant_id >= kNumVariants || n_min < 1 || n_max < n_min) return ATTN_EINVAL;
    if ((d != 64 && d != 128) || (dtype != ATTN_F16 && dtype != ATTN_BF16)) return ATTN_EINVAL;
    if (!kVariants[variant_id].fn(d, dtype, causal)) return ATTN_EUNSUPPORTED;
    Deployment e;
    e.used = true;
    e.variant_id = variant_id;
    e.d = d;
    e.dtype = dtype;
    e.causal = causal ? 1 : 0;
    e.n_min = n_min;
    e.n_max = n_max;
    return add_deployment(e);
}

int attn_deploy_codeobj(int handle, int n_min, int n_max) {
    if (handle < 0 || handle >= kMaxLoaded || !g_loaded[handle].fn || n_min < 1 || n_max < n_min) return ATTN_EINVAL;
    const LoadedKernel& lk = g_loaded[handle];
    Deployment e;
    e.used = true;
    e.variant_id = lk.variant_id;
    e.handle = handle;
    e.d = lk.d;
    e.dtype = lk.dtype;
    e.causal = lk.causal;
    e.n_min = n_min;
    e.n_max = n_max;
    return add_deployment(e);
}

int attn_deploy_clear(void) {
    for (int i = 0; i < kMaxDeployed; ++i) g_deployed[i] = Deployment();
    g_num_deployed = 0;
    return ATTN_OK;
}

int attn_deployed(int N, int d, int dtype, int causal, int* variant_id, int* handle) {
    if (N < 1 || (d != 64 && d != 128) || (dtype != ATTN_F16 && dtype != ATTN_BF16)) return ATTN_EINVAL;
    const Deployment* e = deployed_for(N, d, dtype, causal);
    if (variant_id) *variant_id = e ? e->variant_id : attn_default_variant(N, d, dtype, causal);
    if (handle) *handle = e ? e->handle : -1;
    return e ? 1 : 0;
}

int attn_time_variant(const void* q, const void* k, const void* v, void* out, float* lse, int B, int H,
                      int N, int d, int causal, float scale, int dtype, void* stream, int variant_id,
                      int warmup, int iters, float* ms) {
    return time_launches([&] { return launch(q, k, v, out, lse, B, H, N, d, causal, scale, dtype, stream, variant_id); },
                         stream, warmup, iters, ms);
}

int attn_codeobj_load(const char* path, const char* kernel_name, int variant_id, int d, int dtype, int causal) {
    if (!path || !kernel_name || variant_id < 0 || variant_id >= kNumVariants) return ATTN_EINVAL;
    if ((d != 64 && d != 128) || (dtype != ATTN_F16 && dtype != ATTN_BF16)) return ATTN_EINVAL;
    if (!kVariants[variant_id].fn(d, dtype, causal)) return ATTN_EUNSUPPORTED;
    int slot = -1;
    for (int i = 0; i < kMaxLoaded; ++i)
        if (!g_loaded[i].fn) { slot = i; break; }
    if (slot < 0) return ATTN_EUNSUPPORTED;  // table full: unload something first
    // A failed runtime call leaves its status behind for whoever asks next (another library in
    // the process would report it as its own): look at the file first, and consume the status
    // of a load that fails anyway.
    if (FILE* f = fopen(path, "rb")) fclose(f);
    else return ATTN_ELAUNCH;
    LoadedKernel lk;
    if (hipModuleLoad(&lk.module, path) != hipSuccess) {
        (void)hipGetLastError();
        return ATTN_ELAUNCH;
    }
    if (hipModuleGetFunction(&lk.fn, lk.module, kernel_name) != hipSuccess) {
        (void)hipGetLastError();
        hipModuleUnload(lk.module);
        return ATTN_ELAUNCH;
    }
    lk.variant_id = variant_id;
    lk.d = d;
    lk.dtype = dtype;
    lk.causal = causal ? 1 : 0;
    g_loaded[slot] = lk;
    return slot;
}

int attn_codeobj_unload(int handle) {
    if (handle < 0 || handle >= kMaxLoaded || !g_loaded[handle].fn) return ATTN_EINVAL;
    for (int i = 0; i < kMaxDeployed; ++i)  // attn_fwd must not launch a kernel that is gone
        if (g_deployed[i].used && g_deployed[i].handle == handle) g_deployed[i] = Deployment();
    const hipError_t e = hipModuleUnload(g_loaded[handle].module);
    g_loaded[handle] = LoadedKernel();
    return e == hipSuccess ? ATTN_OK : ATTN_ELAUNCH;
}

int attn_fwd_codeobj(int handle, const void* q, const void* k, const void* v, void* out, float* lse,
                     int B, int H, int N, int d, int causal, float scale, int dtype, void* stream) {
    int rc;
    const LoadedKernel* lk = loaded_for(handle, d, dtype, causal, &rc);
    if (!lk) return rc;
    return launch(q, k, v, out, lse, B, H, N, d, causal, scale, dtype, stream, lk->variant_id, lk->fn);
}

int attn_time_codeobj(int handle, const void* q, const void* k, const void* v, void* out, float* lse,
                      int B, int H, int N, int d, int causal, float scale, int dtype, void* stream,
                      int warmup, int iters, float* ms) {
    int rc;
    const LoadedKernel* lk = loaded_for(handle, d, dtype, causal, &rc);
    if (!lk) return rc;
    return time_launches([&] { return launch(q, k, v, out, lse, B, H, N, d, causal, scale, dtype, stream, lk->variant_id, lk->fn); },
                         stream, warmup, iters, ms);
}

int attn_mfma_ceiling(int random_operands, int iters, void* stream, unsigned long long* counters,
                      double* tflops, double* core_ghz) {
    if (iters < 1 || !counters || !tflops || !core_ghz) return ATTN_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const int blocks = 2 * cu_count();  // 8 waves per CU
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return ATTN_ELAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) { hipEventDestroy(e0); return ATTN_ELAUNCH; }
    int rc = ATTN_OK;
    float ms = 0.f;
    unsigned long long h[2] = {0, 0};
    void* args[] = {&counters, &iters, &random_operands};
    if (hipEventRecord(e0, s) != hipSuccess ||
        hipLaunchKernel((const void*)mfma_ceiling_kernel, dim3(blocks), dim3(256), args, 0, s) != hipSuccess ||
        hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess ||
        hipMemcpy(h, counters, sizeof h, hipMemcpyDeviceToHost) != hipSuccess)
        rc = ATTN_ELAUNCH;
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (rc != ATTN_OK) return rc;
    *tflops = (double)blocks * 4 * (double)iters * 4 * 32768.0 / ((double)ms * 1e-3) / 1e12;
    *core_ghz = h[1] ? (double)h[0] / ((double)h[1] * 10.0) : 0.0;
    return ATTN_OK;
}

int attn_mix_ceiling(int mode, int iters, void* stream, unsigned long long* counters, double* tflops, double* core_ghz) {
    if (mode < 0 || mode > 4 || iters < 1 || !counters || !tflops || !core_ghz) return ATTN_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const int blocks = cu_count();  // one workgroup of 8 waves per CU: two waves per SIMD
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return ATTN_ELAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) { hipEventDestroy(e0); return ATTN_ELAUNCH; }
    int rc = ATTN_OK;
    float ms = 0.f;
    unsigned long long h[2] = {0, 0};
    void* args[] = {&counters, &iters};
    const void* kernels[5] = {(const void*)mix_ceiling_kernel<0>, (const void*)mix_ceiling_kernel<1>, (const void*)mix_ceiling_kernel<2>,
                              (const void*)pingpong_ceiling_kernel<2>, (const void*)pingpong_ceiling_kernel<1>};
    // one untimed launch first: from idle the device takes tens of milliseconds to reach the clock it sustains
    if (hipLaunchKernel(kernels[mode], dim3(blocks), dim3(512), args, 0, s) != hipSuccess ||
        hipEventRecord(e0, s) != hipSuccess ||
        hipLaunchKernel(kernels[mode], dim3(blocks), dim3(512), args, 0, s) != hipSuccess ||
        hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess ||
        hipMemcpy(h, counters, sizeof h, hipMemcpyDeviceToHost) != hipSuccess)
        rc = ATTN_ELAUNCH;
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (rc != ATTN_OK) return rc;
    *tflops = (double)blocks * 8 * (double)iters * (mode >= 3 ? 32 : 16) * 32768.0 / ((double)ms * 1e-3) / 1e12;
    *core_ghz = h[1] ? (double)h[0] / ((double)h[1] * 10.0) : 0.0;
    return ATTN_OK;
}

int attn_valu_ceiling(int waves_per_simd, int iters, void* stream, unsigned long long* counters,
                      double* elements_per_s, double* core_ghz) {
    if (waves_per_simd < 1 || waves_per_simd > 4 || iters < 1 || !counters || !elements_per_s || !core_ghz) return ATTN_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const int blocks = waves_per_simd * cu_count();  // 256 threads: one wave on each SIMD of a CU
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return ATTN_ELAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) { hipEventDestroy(e0); return ATTN_ELAUNCH; }
    int rc = ATTN_OK;
    float ms = 0.f, scale = 0.127517f, shift = -0.25f;
    unsigned long long h[2] = {0, 0};
    void* args[] = {&counters, &iters, &scale, &shift};
    if (hipEventRecord(e0, s) != hipSuccess ||
        hipLaunchKernel((const void*)valu_ceiling_kernel, dim3(blocks), dim3(256), args, 0, s) != hipSuccess ||
        hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess ||
        hipMemcpy(h, counters, sizeof h, hipMemcpyDeviceToHost) != hipSuccess)
        rc = ATTN_ELAUNCH;
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (rc != ATTN_OK) return rc;
    *elements_per_s = (double)blocks * 256.0 * (double)iters * 16.0 / ((double)ms * 1e-3);
    *core_ghz = h[1] ? (double)h[0] / ((double)h[1] * 10.0) : 0.0;
    return ATTN_OK;
}

const char* attn_strerror(int code) {
    switch (code) {
        case ATTN_OK: return "ok";
        case ATTN_EINVAL: return "invalid argument";
        case ATTN_EUNSUPPORTED: return "unsupported shape or variant";
        case ATTN_ELAUNCH: return "HIP launch or event call failed";
        default: return "unknown error code";
    }
}

}  // extern "C"
