/* C ABI of the fused GEMM + LeakyReLU with scratch memory from the caller (gemm_lrelu.h has the operation, its
 * argument rules and the error codes). */
#ifndef PAPER_2403_16863_GEMM_WORKSPACE_H
#define PAPER_2403_16863_GEMM_WORKSPACE_H

#ifdef __cplusplus
extern "C" {
#endif

/* gemm_lrelu with scratch memory to use where that is faster: with few tiles of C and a long K (in
 * a large call, few tiles of 64 x 64, 128 x 128 or 192 x 128) the workgroups split K and write fp32 parts, which a
 * second kernel on the same stream adds in a fixed order.
 * gemm_lrelu_workspace names the bytes a shape asks for (0: none, at most 24 MiB).  workspace: device memory
 * aligned to 16 bytes that meets none of A, B, C, with any contents, not used by anybody else until the
 * call's two kernels have run (a pool that goes by the stream's handle does not see to that where a handle
 * is several queues, as the per-thread stream's, or is destroyed while its work runs); null or fewer
 * bytes than asked for make it the plain call. */
long long gemm_lrelu_workspace(int M, int N, int K);
int gemm_lrelu_in(const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream,
                  void* workspace, long long workspace_bytes);

/* The same for callers that take the memory call by call, with one look at the shape: `scratch` is called at most once, with
 * `owner` and the bytes that the shape asks for, after the arguments have been checked and only where there are any.
 * It returns memory as above or null, which makes it the plain call, and must not throw; null in its place: no memory. */
typedef void* (*gemm_scratch_fn)(void* owner, long long bytes);
int gemm_lrelu_with(const void* a, const void* b, void* c, int M, int N, int K, float slope, int dtype, void* stream,
                    gemm_scratch_fn scratch, void* owner);

/* 1 while the stream records a graph (or cannot say), else 0: memory taken per call has no place in a graph. */
int gemm_lrelu_capturing(void* stream);

#ifdef __cplusplus
}
#endif
#endif
