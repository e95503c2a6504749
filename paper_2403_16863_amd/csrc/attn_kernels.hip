// The attention kernels of one part of the variant table (compile with -DATTN_PART=0 .. 8).
#include "attn_variants.h"

namespace attn {

template <int D, class KN>
const KernelFn KernelSet<D, KN>::fn[2][2] = {
    {(KernelFn)attn_fwd_kernel<F16, D, false, KN>, (KernelFn)attn_fwd_kernel<F16, D, true, KN>},
    {(KernelFn)attn_fwd_kernel<BF16, D, false, KN>, (KernelFn)attn_fwd_kernel<BF16, D, true, KN>}};

#define SET_D64(...) template struct KernelSet<64, Knobs<__VA_ARGS__>>;
#define SET_D128(...) template struct KernelSet<128, Knobs<__VA_ARGS__>>;
#define SET_BOTH(...) SET_D64(__VA_ARGS__) SET_D128(__VA_ARGS__)
#define PART_(n) ATTN_VARIANTS_##n(SET_BOTH, SET_D64, SET_D128)
#define PART(n) PART_(n)
PART(ATTN_PART)

}  // namespace attn
