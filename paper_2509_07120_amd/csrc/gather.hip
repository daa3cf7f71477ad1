// Data movement around the layer.
//
// Token gather: dst[h, i, :] = src[h, index[i], :] (Sec. 4.2: the tokens are split into patch
// tokens and special tokens; this reorders a [heads, n, 64] tensor so that each kind is contiguous,
// and back).  HBM-bound: every row (128 B in bf16, 256 B in fp32) is read once and written once,
// 16 bytes per lane, so consecutive lanes cover whole rows and both sides move full cache lines.
#include "bsga_internal.h"

namespace bsga {
namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <int CHUNKS>  // 16-byte chunks per row
__global__ __launch_bounds__(256) void gather_kernel(const u32x4* __restrict__ src, const int32_t* __restrict__ index,
                                                     u32x4* __restrict__ dst, int64_t n_src, int64_t n_dst) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t i = t / CHUNKS;
  const int c = static_cast<int>(t % CHUNKS);
  if (i >= n_dst) return;
  int64_t j = index[i];
  j = j < 0 ? 0 : (j >= n_src ? n_src - 1 : j);  // an out-of-range index cannot read outside the tensor
  const int64_t h = blockIdx.y;
  dst[(h * n_dst + i) * CHUNKS + c] = src[(h * n_src + j) * CHUNKS + c];
}

// Heads of a projection's output made contiguous, and back: dst[ph][i] = src[index[i]][ph] for the ph of
// [parts][heads], and dst[i][h] = src[h][index[i]].  The same rows of 128 (256) bytes, each read and written once;
// with the reordering of Sec. 4.2 in the same pass there is no separate gather of the tokens.  10,992 tokens,
// 3 x 16 heads, bf16 (135 MB): 23 us, where a strided copy took 51 and gathering the tokens 18 more.
template <int CHUNKS>
__global__ __launch_bounds__(256) void split_heads_kernel(const u32x4* __restrict__ src, const int32_t* __restrict__ index,
                                                          u32x4* __restrict__ dst, int64_t n) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t i = t / CHUNKS;
  const int c = static_cast<int>(t % CHUNKS);
  if (i >= n) return;
  const int64_t j = index != nullptr ? min(max(int64_t(index[i]), int64_t(0)), n - 1) : i;
  const int64_t ph = blockIdx.y, all = gridDim.y;
  dst[(ph * n + i) * CHUNKS + c] = src[(j * all + ph) * CHUNKS + c];
}

template <int CHUNKS>
__global__ __launch_bounds__(256) void merge_heads_kernel(const u32x4* __restrict__ src, const int32_t* __restrict__ index,
                                                          u32x4* __restrict__ dst, int64_t n, int heads) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t ih = t / CHUNKS;
  const int c = static_cast<int>(t % CHUNKS);
  if (ih >= n * heads) return;
  const int64_t i = ih / heads;
  const int64_t h = ih - i * heads;
  const int64_t j = index != nullptr ? min(max(int64_t(index[i]), int64_t(0)), n - 1) : i;
  dst[t] = src[(h * n + j) * CHUNKS + c];
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_heads(const char* fn, const void* src, const void* dst, int dtype, int64_t n, int columns, int head_dim) {
  clear_error();
  if (!src || !dst) return fail(BSGA_ERR_INVALID_ARG, "%s: src and dst must be non-null", fn);
  if (!aligned16(src) || !aligned16(dst)) return fail(BSGA_ERR_INVALID_ARG, "%s: src and dst must be 16-byte aligned", fn);
  if (dtype != BSGA_BF16 && dtype != BSGA_FP32) return fail(BSGA_ERR_INVALID_ARG, "%s: unknown dtype %d", fn, dtype);
  if (head_dim != 64) return fail(BSGA_ERR_UNSUPPORTED, "%s: head_dim must be 64, got %d", fn, head_dim);
  if (columns < 1 || columns > 65535)
    return fail(BSGA_ERR_INVALID_ARG, "%s: the number of heads (times parts) must be in [1, 65535], got %d", fn, columns);
  if (n < 1 || n > (int64_t(1) << 24))
    return fail(BSGA_ERR_INVALID_ARG, "%s: n_tokens must be in [1, 2^24], got %lld", fn, static_cast<long long>(n));
  if (n * columns * 16 > int64_t(0x7fffffff) * 256)
    return fail(BSGA_ERR_UNSUPPORTED, "%s: n_tokens * heads is too large", fn);
  return BSGA_OK;
}

}  // namespace

int launch_gather(const void* src, int dtype, int heads, int64_t n_src, const int32_t* index, int64_t n_dst,
                  void* dst, hipStream_t stream) {
  const int chunks = dtype == BSGA_BF16 ? 8 : 16;
  const dim3 grid(static_cast<unsigned>(ceil_div(n_dst * chunks, 256)), heads);
  const u32x4* s = static_cast<const u32x4*>(src);
  u32x4* d = static_cast<u32x4*>(dst);
  if (dtype == BSGA_BF16) {
    hipLaunchKernelGGL(gather_kernel<8>, grid, dim3(256), 0, stream, s, index, d, n_src, n_dst);
  } else {
    hipLaunchKernelGGL(gather_kernel<16>, grid, dim3(256), 0, stream, s, index, d, n_src, n_dst);
  }
  return check_hip(hipGetLastError(), "bsga_gather_tokens launch");
}

}  // namespace bsga

using namespace bsga;

extern "C" {

int bsga_split_heads(const void* src, int dtype, int64_t n_tokens, int parts, int heads, int head_dim, const int32_t* index,
                     void* dst, void* stream) {
  const char* fn = "bsga_split_heads";
  const int64_t columns = int64_t(parts) * heads;
  if (int rc = check_heads(fn, src, dst, dtype, n_tokens,
                           parts < 1 || heads < 1 || columns > 65535 ? 0 : static_cast<int>(columns), head_dim))
    return rc;
  const int chunks = dtype == BSGA_BF16 ? 8 : 16;
  const dim3 grid(static_cast<unsigned>(ceil_div(n_tokens * chunks, 256)), static_cast<unsigned>(columns));
  const u32x4* s = static_cast<const u32x4*>(src);
  u32x4* d = static_cast<u32x4*>(dst);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == BSGA_BF16) hipLaunchKernelGGL(split_heads_kernel<8>, grid, dim3(256), 0, st, s, index, d, n_tokens);
  else hipLaunchKernelGGL(split_heads_kernel<16>, grid, dim3(256), 0, st, s, index, d, n_tokens);
  return check_hip(hipGetLastError(), "bsga_split_heads launch");
}

int bsga_merge_heads(const void* src, int dtype, int heads, int64_t n_tokens, int head_dim, const int32_t* index, void* dst,
                     void* stream) {
  const char* fn = "bsga_merge_heads";
  if (int rc = check_heads(fn, src, dst, dtype, n_tokens, heads, head_dim)) return rc;
  const int chunks = dtype == BSGA_BF16 ? 8 : 16;
  const dim3 grid(static_cast<unsigned>(ceil_div(n_tokens * heads * chunks, 256)));
  const u32x4* s = static_cast<const u32x4*>(src);
  u32x4* d = static_cast<u32x4*>(dst);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == BSGA_BF16) hipLaunchKernelGGL(merge_heads_kernel<8>, grid, dim3(256), 0, st, s, index, d, n_tokens, heads);
  else hipLaunchKernelGGL(merge_heads_kernel<16>, grid, dim3(256), 0, st, s, index, d, n_tokens, heads);
  return check_hip(hipGetLastError(), "bsga_merge_heads launch");
}

}  // extern "C"
