// Block average pooling P^b(x) (Sec. 4.1, "Predicting Block Masks").
//
// One workgroup per (head, block): 256 threads stream the block's b x 64 elements with 16-byte
// loads (a block is one contiguous run of memory), add them up in float64 and write the 64
// block means.  The kernel is bound by HBM reads: 2 bytes (bf16) or 4 bytes (fp32) per element,
// each read exactly once.  Q and K go in one launch: of a short layer a second one is a tenth (16 heads x 1,374 tokens,
// the layer 36.4 -> 33.9 us).
//
// With the special-token split (Sec. 4.2) Q, K and V are put into working order first.  GATHER does that in the same pass, all three in
// one launch: rows are read through the token order, written, and those of Q and K summed, so they are not read a second time.
// The layer with the split at rho = 0.75, 16 heads: 2 frames 73.7 -> 57.6 us, 8 frames 202 -> 182, 100 frames 16.36 -> 16.29 ms.
#include "bsga_internal.h"

namespace bsga {
namespace {

constexpr int kThreads = 256;
constexpr int kD = 64;

__device__ inline void widen8(const uint4& raw, double* acc) {
  // eight bf16 values packed in 16 bytes -> added into acc[0..7]
  const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc[2 * i] += static_cast<double>(__uint_as_float(w[i] << 16));
    acc[2 * i + 1] += static_cast<double>(__uint_as_float(w[i] & 0xffff0000u));
  }
}

__device__ inline void widen4(const uint4& raw, double* acc) {
  acc[0] += static_cast<double>(__uint_as_float(raw.x));
  acc[1] += static_cast<double>(__uint_as_float(raw.y));
  acc[2] += static_cast<double>(__uint_as_float(raw.z));
  acc[3] += static_cast<double>(__uint_as_float(raw.w));
}

// Up to three tensors, one to each of blockIdx.z; pooled may be null.
struct PoolTensors {
  const uint4* x[3];
  double* pooled[3];
  uint4* ordered[3];     // GATHER: [heads][n_tokens], token i from x[heads][n_src] at index[i]
  const int32_t* index;
  int64_t n_src;
};

// ELEM_BYTES: 2 = bf16, 4 = fp32.
template <int ELEM_BYTES, int B, bool GATHER>
__global__ __launch_bounds__(kThreads) void pool_kernel(PoolTensors a, int64_t n_tokens, int64_t n_first, int nb1, int nb) {
  const uint4* const x = a.x[blockIdx.z];
  double* const pooled = a.pooled[blockIdx.z];
  constexpr int E = 16 / ELEM_BYTES;     // elements per 16-byte chunk
  constexpr int CH = kD / E;             // chunks per token row
  constexpr int TL = kThreads / CH;      // tokens covered per pass
  constexpr int PASSES = B / TL;
  __shared__ double red[TL][kD + 1];

  const int I = blockIdx.x;
  const int h = blockIdx.y;
  const int t = threadIdx.x;
  const int cg = t % CH;
  const int tl = t / CH;
  // blocks 0 .. nb1-1 tile tokens [0, n_first), the others tokens [n_first, n_tokens)
  const int64_t tok0 = I < nb1 ? int64_t(I) * B : n_first + int64_t(I - nb1) * B;
  const int valid = static_cast<int>(min<int64_t>(B, (I < nb1 ? n_first : n_tokens) - tok0));
  double acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.0;

  uint4 raw[PASSES];
  if constexpr (GATHER) {
    int64_t from[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {  // (an index out of range cannot read outside the tensor)
      const int64_t j = a.index[tok0 + min(tl + p * TL, valid - 1)];
      from[p] = (int64_t(h) * a.n_src + (j < 0 ? 0 : (j >= a.n_src ? a.n_src - 1 : j))) * CH + cg;
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) raw[p] = x[from[p]];
    uint4* const to = a.ordered[blockIdx.z] + (int64_t(h) * n_tokens + tok0) * CH + cg;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int tok = tl + p * TL;
      if (tok < valid) to[int64_t(tok) * CH] = raw[p];
      else raw[p] = make_uint4(0, 0, 0, 0);
    }
    if (pooled == nullptr) return;
  } else {
    const uint4* const base = x + (int64_t(h) * n_tokens + tok0) * CH;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int tok = tl + p * TL;
      raw[p] = make_uint4(0, 0, 0, 0);
      if (tok < valid) raw[p] = base[int64_t(tok) * CH + cg];
    }
  }
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    if constexpr (ELEM_BYTES == 2) widen8(raw[p], acc); else widen4(raw[p], acc);
  }
#pragma unroll
  for (int e = 0; e < E; ++e) red[tl][cg * E + e] = acc[e];
  __syncthreads();
  if (t < kD) {
    double s = 0.0;
#pragma unroll 8
    for (int r = 0; r < TL; ++r) s += red[r][t];
    pooled[(int64_t(h) * nb + I) * kD + t] = s / static_cast<double>(valid);
  }
}

template <bool GATHER>
void launch(const PoolTensors& a, int tensors, int dtype, int heads, int64_t n_tokens, int64_t n_first, int block, hipStream_t stream) {
  const int nb = static_cast<int>(split_blocks(n_tokens, n_first, block));
  const int nb1 = static_cast<int>(ceil_div(n_first, block));
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(nb, heads, tensors), dim3(kThreads), 0, stream, a, n_tokens, n_first, nb1, nb); };
  if (dtype == BSGA_BF16) {
    if (block == 64) go(pool_kernel<2, 64, GATHER>);
    else go(pool_kernel<2, 128, GATHER>);
  } else {
    if (block == 64) go(pool_kernel<4, 64, GATHER>);
    else go(pool_kernel<4, 128, GATHER>);
  }
}

}  // namespace

int launch_pool(const void* x0, double* pooled0, const void* x1, double* pooled1, int dtype, int heads, int64_t n_tokens, int64_t n_first,
                int block, hipStream_t stream) {
  PoolTensors a = {};
  a.x[0] = static_cast<const uint4*>(x0);
  a.x[1] = static_cast<const uint4*>(x1);
  a.pooled[0] = pooled0;
  a.pooled[1] = pooled1;
  launch<false>(a, x1 != nullptr ? 2 : 1, dtype, heads, n_tokens, n_first, block, stream);
  return check_hip(hipGetLastError(), "bsga_pool_qk launch");
}

int launch_gather_pool(const void* const (&x)[3], int dtype, int heads, int64_t n_src, const int32_t* index, int64_t n_tokens, int64_t n_first,
                       int block, void* const (&ordered)[3], double* const (&pooled)[3], hipStream_t stream) {
  PoolTensors a = {};
  for (int i = 0; i < 3; ++i) {
    a.x[i] = static_cast<const uint4*>(x[i]);
    a.ordered[i] = static_cast<uint4*>(ordered[i]);
    a.pooled[i] = pooled[i];
  }
  a.index = index;
  a.n_src = n_src;
  launch<true>(a, 3, dtype, heads, n_tokens, n_first, block, stream);
  return check_hip(hipGetLastError(), "bsga_gather_pool launch");
}

}  // namespace bsga
