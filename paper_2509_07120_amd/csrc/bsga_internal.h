// Internal declarations shared by the bsga translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "bsga.h"

namespace bsga {

// Records a message for bsga_last_error() and returns `code`.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

// Turns a HIP status into a bsga return code (records the HIP error string).
int check_hip(hipError_t e, const char* what);

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Number of blocks when tokens [0, n_first) and [n_first, n_tokens) are cut into blocks separately
// (no block crosses n_first).  n_first = n_tokens or 0 gives ceil(n_tokens / block).
inline int64_t split_blocks(int64_t n_tokens, int64_t n_first, int64_t block) {
  return ceil_div(n_first, block) + ceil_div(n_tokens - n_first, block);
}

// Scratch of the bf16 attention kernels.  Every call may use the launch order of the (head, query block)
// rows: one int32 per row, sized for the smaller block size (plus one block for a split sequence), plus a
// [32 classes][heads] table.
inline size_t attn_order_bytes(int heads, int64_t n_tokens) {
  return (static_cast<size_t>(heads) * static_cast<size_t>(ceil_div(n_tokens, 64) + 1) + 32u * static_cast<size_t>(heads) + 4u) *
         sizeof(int32_t);
}
// Calls of few rows share rows between workgroups and then need room for partial results, whatever the
// number of rows: two of 33 KB for each of 512 workgroups, and a table.  Up to 4032 tokens (63 blocks of 64) a
// row is too short to be worth sharing.
constexpr size_t kStreamBytes = 2 * 512 * (2 * 66 * 64 * sizeof(float)) + (size_t(1) << 14);
inline bool attn_stream_shape(int heads, int64_t n_tokens) {
  return n_tokens > 4032 && static_cast<int64_t>(heads) * ceil_div(n_tokens, 128) < 1024;
}
// Kernel launchers.  Arguments are already validated.
int launch_pool(const void* x, int dtype, int heads, int64_t n_tokens, int64_t n_first, int block, double* pooled,
                hipStream_t stream);

int launch_select(const double* q_pool, const double* k_pool, int heads, int nb_q, int nb_k,
                  double score_scale, double tau, double one_minus_rho, const uint8_t* force_q,
                  const uint8_t* force_k, uint32_t* mask_bits, int32_t* kv_idx, int32_t* kv_cnt,
                  int idx_stride, void* workspace, hipStream_t stream);
size_t select_workspace_bytes(int heads, int nb_q, int nb_k);

int launch_gather(const void* src, int dtype, int heads, int64_t n_src, const int32_t* index,
                  int64_t n_dst, void* dst, hipStream_t stream);

// workspace_bytes: of the call's workspace, 0 without one; the launch order alone or more (see attn_order_bytes).
int launch_attn_bf16(const void* q, const void* k, const void* v, int heads, int64_t n_tokens, int64_t n_first,
                     int block, int block_k, float softmax_scale, const int32_t* kv_idx, const int32_t* kv_cnt,
                     int idx_stride, void* out, float* lse, void* workspace, size_t workspace_bytes, hipStream_t stream);

int launch_attn_fp32(const float* q, const float* k, const float* v, int heads, int64_t n_tokens, int64_t n_first,
                     int block, float softmax_scale, const int32_t* kv_idx, const int32_t* kv_cnt,
                     int idx_stride, float* out, float* lse, hipStream_t stream);

int launch_probe_mfma(int pattern, int mix, int iters, float* sink, size_t sink_bytes, double* flops,
                      hipStream_t stream);

}  // namespace bsga
