// Host-side check of the C-ABI glue (argument validation, block arithmetic, workspace sizing, error
// strings) under AddressSanitizer / UndefinedBehaviorSanitizer.  The kernel launchers are replaced
// by the stubs below, which only check the invariants the real launchers rely on, so the program
// runs on a machine without a GPU.  Built and run by tests/test_hostglue_sanitized.py.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <string>
#include <vector>

#include "bsga.h"
#include "bsga_internal.h"

static int g_calls = 0;
static int g_fail = 0;
static int g_pooled = 0;              // tensors of the last pooling launch
static size_t g_workspace_bytes = 0;  // of the last attention launch
#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      fprintf(stderr, "FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond);    \
      ++g_fail;                                                            \
    }                                                                      \
  } while (0)

namespace bsga {
// ---- stubs: the launchers' preconditions, as the API layer must establish them -------------------
int launch_pool(const void* x0, double* pooled0, const void* x1, double* pooled1, int dtype, int heads, int64_t n_tokens,
                int64_t n_first, int block, hipStream_t) {
  ++g_calls;
  g_pooled = x1 ? 2 : 1;
  CHECK(x0 && pooled0 && !x1 == !pooled1 && heads >= 1 && n_tokens >= 1 && n_first >= 0 && n_first <= n_tokens);
  CHECK((block == 64 || block == 128) && (dtype == BSGA_BF16 || dtype == BSGA_FP32));
  return BSGA_OK;
}
size_t select_workspace_bytes(int heads, int nb_q, int nb_k) { return size_t(heads) * nb_q * nb_k * sizeof(double); }
int launch_select(const double* q_pool, const double* k_pool, int heads, int nb_q, int nb_k, double, double tau,
                  double one_minus_rho, const uint8_t*, const uint8_t*, uint32_t* mask_bits, int32_t* kv_idx,
                  int32_t* kv_cnt, int idx_stride, void* workspace, hipStream_t) {
  ++g_calls;
  CHECK(q_pool && k_pool && workspace && heads >= 1 && nb_q >= 1 && nb_k >= 1 && nb_k <= 8192);
  CHECK(tau >= 0.0 && one_minus_rho >= 0.0 && one_minus_rho <= 1.0);
  CHECK(mask_bits || kv_idx || kv_cnt);
  CHECK(!kv_idx || idx_stride >= nb_k);
  return BSGA_OK;
}
int launch_gather(const void* src, int, int heads, int64_t n_src, const int32_t* index, int64_t n_dst, void* dst,
                  hipStream_t) {
  ++g_calls;
  CHECK(src && index && dst && heads >= 1 && n_src >= 1 && n_dst >= 1);
  return BSGA_OK;
}
int launch_gather_pool(const void* const (&x)[3], int dtype, int heads, int64_t n_src, const int32_t* index, int64_t n_tokens, int64_t n_first,
                       int block, void* const (&ordered)[3], double* const (&pooled)[3], hipStream_t) {
  ++g_calls;
  for (int i = 0; i < 3; ++i) CHECK(x[i] && ordered[i] && (pooled[i] != nullptr) == (i < 2));
  CHECK((dtype == BSGA_BF16 || dtype == BSGA_FP32) && (block == 64 || block == 128) && heads >= 1 && n_src >= 1 && index);
  CHECK(n_tokens >= 1 && n_first >= 0 && n_first <= n_tokens);
  return BSGA_OK;
}
int launch_linear(const void* x, bool, const void* weight, const void* bias, int64_t n_tokens, int in_features, int out_features, bool,
                  const int32_t* row_index, const void* residual, bool out_heads, void* out, hipStream_t) {
  ++g_calls;
  CHECK(x && weight && bias && out && n_tokens >= 1 && in_features >= 64 && in_features % 64 == 0 && out_features >= 64 && out_features % 64 == 0);
  CHECK(!out_heads || (!row_index && !residual));
  // offsets go up to a tile of 256 features or 192 tokens past the end, in 32 bits
  CHECK((n_tokens + 191) * in_features * 2 < (int64_t(1) << 31) && (int64_t(out_features) + 255) * in_features * 2 < (int64_t(1) << 31));
  CHECK(n_tokens * out_features * 2 < (int64_t(1) << 31));
  return BSGA_OK;
}
int launch_layer_norm(const void* x, const void* weight, const void* bias, float, int64_t n_tokens, int features, const int32_t*, void* out,
                      hipStream_t) {
  ++g_calls;
  CHECK(x && weight && bias && out && n_tokens >= 1 && n_tokens <= (1 << 24) && features >= 8 && features % 8 == 0 && features <= 4096);
  return BSGA_OK;
}
static void check_attn(int heads, int64_t n_tokens, int64_t n_first, int block, int block_k, const int32_t* kv_idx,
                       const int32_t* kv_cnt, int idx_stride) {
  CHECK(heads >= 1 && n_tokens >= 1 && n_first >= 0 && n_first <= n_tokens);
  CHECK((kv_idx == nullptr) == (kv_cnt == nullptr));
  CHECK(!kv_idx || idx_stride >= split_blocks(n_tokens, n_first, block_k));
  CHECK(block == block_k || (block == 128 && block_k == 64));
}
int launch_attn_bf16(const void* q, const void* k, const void* v, int heads, int64_t n_tokens, int64_t n_first, int block,
                     int block_k, float scale, const int32_t* kv_idx, const int32_t* kv_cnt, int idx_stride, void* out,
                     float*, void* workspace, size_t workspace_bytes, hipStream_t) {
  ++g_calls;
  g_workspace_bytes = workspace_bytes;
  CHECK(q && k && v && out && scale > 0.f);
  CHECK((workspace == nullptr) == (workspace_bytes == 0));
  check_attn(heads, n_tokens, n_first, block, block_k, kv_idx, kv_cnt, idx_stride);
  if (workspace) {  // the launch order needs one word per query block plus the class table, the merged class and a counter: touch
                    // it all, and what a choice between rows and pairs takes beyond that
    const int64_t nb = split_blocks(n_tokens, n_first, block);
    const bool choice = block == 128 && kv_idx && chooses_pairs(heads, static_cast<int>(nb), static_cast<int>(split_blocks(n_tokens, n_first, block_k)));
    const size_t words = kv_idx ? size_t(heads) * nb + 32u * heads + 2 + (choice ? 34u * heads + 1 : 0) : 1;
    memset(workspace, 0, words * sizeof(int32_t));  // ASan faults here if the API sized the workspace too small
  }
  return BSGA_OK;
}
int launch_attn_fp32(const float* q, const float* k, const float* v, int heads, int64_t n_tokens, int64_t n_first,
                     int block, float scale, const int32_t* kv_idx, const int32_t* kv_cnt, int idx_stride, float* out,
                     float*, void* workspace, size_t workspace_bytes, hipStream_t) {
  ++g_calls;
  g_workspace_bytes = workspace_bytes;
  CHECK(q && k && v && out && scale > 0.f);
  CHECK((workspace == nullptr) == (workspace_bytes == 0));
  check_attn(heads, n_tokens, n_first, block, block, kv_idx, kv_cnt, idx_stride);
  const size_t parts = size_t(heads) * n_tokens * kPartRow;  // used if it is all there
  if (workspace && workspace_bytes >= parts && parts <= kPartsMaxBytes) memset(workspace, 0, parts);
  return BSGA_OK;
}
int launch_probe_mfma(int pattern, int mix, int iters, float* sink, size_t, double* flops, hipStream_t) {
  ++g_calls;
  CHECK((pattern == 0 || pattern == 1) && mix >= 0 && mix <= 2 && iters >= 1 && sink);
  if (flops) *flops = 1.0;
  return BSGA_OK;
}
}  // namespace bsga

using bsga::chooses_pairs;
using bsga::dense_pairs;
using bsga::pair_differs;
using bsga::pairs_pay;

static bool err_has(const char* what) { return strstr(bsga_last_error(), what) != nullptr; }

int main() {
  alignas(16) static unsigned char buf[1 << 16];
  void* A = buf;  // a real, 16-byte aligned host buffer standing in for device memory (never dereferenced
                  // by the API layer; the stubs only touch the workspace)
  CHECK(bsga_version() == 3);
  CHECK(strlen(bsga_last_error()) == 0);

  // ---- which dense launches take rows in pairs: (heads, blocks per head) at the lines of the rule
  struct { int heads, nb; bool pairs; } dense[] = {
      {16, 22, true}, {16, 33, false}, {16, 54, true}, {16, 65, false}, {16, 86, true}, {16, 128, true},  // the busiest CU: no more rows in pairs
      {32, 16, true}, {64, 15, false}, {64, 16, true}, {32, 48, true}, {64, 24, false}, {64, 32, false}, {128, 16, false},  // long enough for it
      {16, 129, false}, {20, 128, true}, {16, 176, false}, {16, 191, true}, {16, 211, false}, {16, 256, true},  // the last round is full
      {51, 100, true}, {80, 95, false}, {80, 96, true}, {46, 112, false}, {20, 255, true}, {20, 256, true}, {16, 322, true}, {90, 65, false},
      {1, 1, false}, {512, 1, false}, {5120, 1, false}, {65535, 1, false}, {512, 2, false}, {2560, 2, false}, {2000, 3, false}, {640, 8, false}};
  for (const auto& c : dense)
    if (dense_pairs(c.heads, c.nb) != c.pairs) {
      fprintf(stderr, "FAILED dense_pairs(%d, %d)\n", c.heads, c.nb);
      ++g_fail;
    }

  // ---- which sparse launches look at their lists, and what for (lengths in tiles of all blocks, differences of all pairs)
  CHECK(!chooses_pairs(16, 257, 257) && !chooses_pairs(17, 301, 301) && chooses_pairs(18, 301, 301) && chooses_pairs(16, 344, 344));
  CHECK(!chooses_pairs(64, 299, 299) && chooses_pairs(32, 300, 300) && chooses_pairs(2, 4096, 4096) && !chooses_pairs(2, 4097, 4097));
  auto pays = [](long long rows, int nb, int per_tile, double kept, double apart) {  // apart: difference of a pair over its sum
    const long long all = static_cast<long long>(kept * per_tile * nb * rows);
    return pairs_pay(all, static_cast<long long>(apart * all), rows, per_tile * nb, per_tile);
  };
  for (int per_tile : {1, 2}) {
    CHECK(pays(17184, 1074, per_tile, 0.25, 0.0) && pays(17184, 1074, per_tile, 0.7, 0.1) && !pays(17184, 1074, per_tile, 0.8, 0.13));
    CHECK(!pays(17184, 1074, per_tile, 0.24, 0.0) && !pays(16384, 512, per_tile, 0.5, 0.0) && pays(16384, 512, per_tile, 0.51, 0.0));
    CHECK(pays(16384, 1024, per_tile, 0.4, 0.0) && !pays(16383, 1024, per_tile, 0.4, 0.0));
    CHECK(!pays(19264, 301, per_tile, 0.9, 0.05) && pays(19264, 301, per_tile, 0.9, 0.03) && !pays(16384, 512, per_tile, 0.7, 0.07));
    CHECK(pays(8208, 513, per_tile, 0.61, 0.03) && !pays(8208, 513, per_tile, 0.59, 0.03) && !pays(8208, 513, per_tile, 0.9, 0.04));
    CHECK(!pair_differs(0, 16 * per_tile, 0, per_tile) && pair_differs(0, 0, 16 * per_tile + 1, per_tile));  // tiles, not entries
    CHECK(!pair_differs(320, 40 + 16 * per_tile, 20, per_tile) && pair_differs(320, 20, 41 + 16 * per_tile, per_tile));
    // the room of the launch order, sized for blocks of 64, holds what is left of the pairs: two tables and five words
    for (int heads : {1, 16, 28, 400, 65535})
      for (int64_t nb : {300, 301, 513, 4096})
        for (int64_t n : {nb * 128, nb * 128 - 127, (nb - 2) * 128 + 2})  // the last: split, with a ragged block in each part
          CHECK(bsga::attn_order_bytes(heads, n) >= 4 * (heads * (nb + 32 + 34) + 5));
  }

  // ---- pooling
  CHECK(bsga_pool_qk(A, A, 0, 16, 1000, 64, 128, (double*)A, (double*)A, nullptr) == BSGA_OK);
  CHECK(g_calls == 1 && g_pooled == 2);  // one launch
  CHECK(bsga_pool_qk(A, nullptr, 0, 16, 1000, 64, 128, (double*)A, nullptr, nullptr) == BSGA_OK && g_pooled == 1);
  CHECK(bsga_pool_qk(nullptr, A, 0, 16, 1000, 64, 128, nullptr, (double*)A, nullptr) == BSGA_OK && g_calls == 3 && g_pooled == 1);
  CHECK(bsga_pool_qk(nullptr, nullptr, 0, 16, 1000, 64, 128, nullptr, nullptr, nullptr) == BSGA_ERR_INVALID_ARG && err_has("nothing"));
  CHECK(bsga_pool_qk(A, A, 9, 16, 1000, 64, 128, (double*)A, (double*)A, nullptr) == BSGA_ERR_INVALID_ARG && err_has("dtype"));
  CHECK(bsga_pool_qk(A, A, 0, 16, 1000, 64, 96, (double*)A, (double*)A, nullptr) == BSGA_ERR_UNSUPPORTED && err_has("block"));
  CHECK(bsga_pool_qk(buf + 4, A, 0, 16, 1000, 64, 64, (double*)A, (double*)A, nullptr) == BSGA_ERR_INVALID_ARG && err_has("aligned"));
  CHECK(bsga_pool_qk(A, A, 0, 16, (int64_t(1) << 24) + 1, 64, 64, (double*)A, (double*)A, nullptr) == BSGA_ERR_UNSUPPORTED);
  CHECK(bsga_pool_qk_split(A, A, 0, 16, 1000, 0, 64, 64, (double*)A, (double*)A, nullptr) == BSGA_OK);
  CHECK(bsga_pool_qk_split(A, A, 0, 16, 1000, 1000, 64, 64, (double*)A, (double*)A, nullptr) == BSGA_OK);
  CHECK(bsga_pool_qk_split(A, A, 0, 16, 1000, 1001, 64, 64, (double*)A, (double*)A, nullptr) == BSGA_ERR_INVALID_ARG && err_has("n_first"));
  CHECK(bsga_pool_qk_split(A, A, 0, 16, 1000, -1, 64, 64, (double*)A, (double*)A, nullptr) == BSGA_ERR_INVALID_ARG);

  // ---- selection: workspace sizing at the edges
  CHECK(bsga_select_workspace_bytes(16, 1074, 1074) == size_t(16) * 1074 * 1074 * 8);
  CHECK(bsga_select_workspace_bytes(0, 1, 1) == 0 && bsga_select_workspace_bytes(1, -1, 1) == 0);
  CHECK(bsga_select_workspace_bytes(65535, 1 << 18, 8192) == size_t(65535) * (size_t(1) << 18) * 8192 * 8);  // no 32-bit overflow
  const size_t sel_ws = bsga_select_workspace_bytes(2, 9, 9);
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 9, 64, 0.125, 0.9, 1.0, nullptr, nullptr, (uint32_t*)A,
                           (int32_t*)A, (int32_t*)A, 9, A, sel_ws, nullptr) == BSGA_OK);
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 9, 64, 0.125, 0.9, 1.0, nullptr, nullptr, (uint32_t*)A,
                           (int32_t*)A, (int32_t*)A, 9, A, sel_ws - 1, nullptr) == BSGA_ERR_WORKSPACE);
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 9, 64, 0.125, 0.9, 1.0, nullptr, nullptr, (uint32_t*)A,
                           (int32_t*)A, (int32_t*)A, 8, A, sel_ws, nullptr) == BSGA_ERR_INVALID_ARG && err_has("idx_stride"));
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 9, 64, 0.125, -0.1, 1.0, nullptr, nullptr, (uint32_t*)A,
                           (int32_t*)A, (int32_t*)A, 9, A, sel_ws, nullptr) == BSGA_ERR_INVALID_ARG && err_has("tau"));
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 9, 64, 0.125, 0.9, 1.5, nullptr, nullptr, (uint32_t*)A,
                           (int32_t*)A, (int32_t*)A, 9, A, sel_ws, nullptr) == BSGA_ERR_INVALID_ARG && err_has("rho"));
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 8193, 64, 0.125, 0.9, 1.0, nullptr, nullptr, (uint32_t*)A,
                           (int32_t*)A, (int32_t*)A, 8193, A, size_t(1) << 40, nullptr) == BSGA_ERR_UNSUPPORTED);
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 9, 64, 0.125, 0.9, 1.0, nullptr, nullptr, nullptr, nullptr,
                           nullptr, 9, A, sel_ws, nullptr) == BSGA_ERR_INVALID_ARG && err_has("no output"));
  const double nan = __builtin_nan("");
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 9, 64, nan, 0.9, 1.0, nullptr, nullptr, (uint32_t*)A,
                           (int32_t*)A, (int32_t*)A, 9, A, sel_ws, nullptr) == BSGA_ERR_INVALID_ARG);
  CHECK(bsga_select_blocks((double*)A, (double*)A, 2, 9, 9, 64, 0.125, nan, 1.0, nullptr, nullptr, (uint32_t*)A,
                           (int32_t*)A, (int32_t*)A, 9, A, sel_ws, nullptr) == BSGA_ERR_INVALID_ARG);

  // ---- gather
  CHECK(bsga_gather_tokens(A, 0, 3, 100, 64, (int32_t*)A, 50, A, nullptr) == BSGA_OK);
  CHECK(bsga_gather_tokens(A, 0, 3, 100, 64, (int32_t*)A, 0, A, nullptr) == BSGA_OK);
  CHECK(bsga_gather_tokens(A, 0, 3, 0, 64, (int32_t*)A, 5, A, nullptr) == BSGA_ERR_INVALID_ARG);
  CHECK(bsga_gather_tokens(nullptr, 0, 3, 100, 64, (int32_t*)A, 5, A, nullptr) == BSGA_ERR_INVALID_ARG);

  // ---- attention: the workspace the API asks for must cover what the launcher writes, for every
  // shape class (uniform, split with one more block, block 64, block 128)
  for (int64_t n : {1LL, 63LL, 64LL, 129LL, 1000LL, 137400LL}) {
    for (int heads : {1, 16}) {
      const size_t need = bsga_attn_workspace_bytes(BSGA_BF16, heads, n, 64);
      CHECK(need >= (size_t(heads) * ((n + 63) / 64) + 32u * heads + 1) * 4);
      unsigned char* ws = new unsigned char[need + 16];  // exact size: an overrun is an ASan report
      void* wsa = ws + ((16 - (reinterpret_cast<uintptr_t>(ws) & 15)) & 15);
      for (int block : {64, 128}) {
        const int stride = int((n + block - 1) / block) + 1;
        CHECK(bsga_sparse_attn(A, A, A, 0, heads, n, 64, block, 0.125f, (int32_t*)A, (int32_t*)A, stride, A, nullptr, wsa,
                               need, nullptr) == BSGA_OK);
        for (int64_t n_first : {int64_t(0), n / 3, n}) {
          CHECK(bsga_sparse_attn_split(A, A, A, 0, heads, n, n_first, 64, block, block, 0.125f, (int32_t*)A, (int32_t*)A,
                                       stride + 1, A, nullptr, wsa, need, nullptr) == BSGA_OK);
        }
      }
      CHECK(bsga_sparse_attn_qk(A, A, A, 0, heads, n, 64, 128, 64, 0.125f, (int32_t*)A, (int32_t*)A, int((n + 63) / 64), A,
                                nullptr, wsa, need, nullptr) == BSGA_OK);
      if (need > 16)
        CHECK(bsga_sparse_attn(A, A, A, 0, heads, n, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 1 << 20, A, nullptr, wsa,
                               need - 16, nullptr) == BSGA_ERR_WORKSPACE);
      CHECK(bsga_dense_attn(A, A, A, 0, heads, n, 64, 0.125f, A, nullptr, nullptr, 0, nullptr) == BSGA_OK);
      CHECK(bsga_dense_attn(A, A, A, 1, heads, n, 64, 0.125f, A, nullptr, nullptr, 0, nullptr) == BSGA_OK);
      delete[] ws;
    }
  }
  CHECK(bsga_attn_workspace_bytes(BSGA_FP32, 16, 1000, 64) == 0 && bsga_attn_workspace_bytes(0, 0, 1000, 64) == 0);
  CHECK(bsga_sparse_attn(A, A, A, 0, 4, 1000, 64, 128, 0.125f, nullptr, (int32_t*)A, 8, A, nullptr, nullptr, 0, nullptr) == BSGA_ERR_INVALID_ARG);
  CHECK(bsga_sparse_attn(A, A, A, 0, 4, 1000, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 7, A, nullptr, nullptr, 0, nullptr) == BSGA_ERR_INVALID_ARG && err_has("idx_stride"));
  CHECK(bsga_sparse_attn(A, A, A, 0, 4, 1000, 64, 128, 0.f, (int32_t*)A, (int32_t*)A, 8, A, nullptr, nullptr, 0, nullptr) == BSGA_ERR_INVALID_ARG && err_has("softmax_scale"));
  CHECK(bsga_sparse_attn(A, A, A, 0, 4, 1000, 32, 128, 0.125f, (int32_t*)A, (int32_t*)A, 8, A, nullptr, nullptr, 0, nullptr) == BSGA_ERR_UNSUPPORTED);
  CHECK(bsga_sparse_attn_qk(A, A, A, 0, 4, 1000, 64, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 16, A, nullptr, nullptr, 0, nullptr) == BSGA_ERR_UNSUPPORTED);
  CHECK(bsga_sparse_attn_qk(A, A, A, 1, 4, 1000, 64, 128, 64, 0.125f, (int32_t*)A, (int32_t*)A, 16, A, nullptr, nullptr, 0, nullptr) == BSGA_ERR_UNSUPPORTED);
  CHECK(bsga_sparse_attn_split(A, A, A, 0, 4, 1000, 1001, 64, 128, 128, 0.125f, (int32_t*)A, (int32_t*)A, 16, A, nullptr, nullptr, 0, nullptr) == BSGA_ERR_INVALID_ARG);

  // ---- which kernel blocks of 64 go to: the lines that the GPU tests of the ways choose their sizes by
  CHECK(bsga::few_rows(64, 1) && bsga::few_rows(64, 1023) && !bsga::few_rows(64, 1024) && !bsga::few_rows(128, 16));
  CHECK(bsga::pairs_rows(64, 512, 2, 2) && bsga::pairs_rows(64, 1, 4096, 4096) && bsga::pairs_rows(64, 16, 64, 64));
  CHECK(!bsga::pairs_rows(64, 1, 1023, 1023) && !bsga::pairs_rows(64, 1, 4097, 4097) && !bsga::pairs_rows(64, 2000, 1, 1) &&
        !bsga::pairs_rows(128, 16, 172, 172));
  CHECK(bsga::shares_rows(313, 64, 313, false) && !bsga::shares_rows(255, 64, 255, false) && !bsga::shares_rows(401, 64, 401, false));
  for (int nb : {1, 2, 300, 4096, 4097})
    for (int heads = 1; heads < 3000; ++heads) {
      const int64_t rows = int64_t(heads) * nb;
      CHECK(bsga::few_rows(64, rows) + bsga::pairs_rows(64, heads, nb, nb) <= 1);                                   // never two of them
      CHECK((bsga::few_rows(64, rows) || bsga::pairs_rows(64, heads, nb, nb)) == !(rows >= 1024 && (nb == 1 || nb > 4096)));  // else two waves to a block
      CHECK(!bsga::shares_rows(rows, 64, nb, false) || bsga::few_rows(64, rows));                                   // rows are shared out of these alone
    }

  // ---- token order and pooling in one pass, linear layer, layer norm
  {
    const int before = g_calls;
    int refused = 0;
    void *Z = nullptr, *O = buf + 8;  // null, misaligned
    struct GP { const void* q = nullptr; int dt = 0, h = 3; int64_t src = 100; int d = 64; const void* ix = nullptr; int64_t n = 90, first = 80; int b = 64; void *qo, *vo; double *qp, *kp; };
    auto pool = [&](auto change) {
      GP a{A, 0, 3, 100, 64, A, 90, 80, 64, A, A, static_cast<double*>(A), static_cast<double*>(A)};
      change(a);
      const int rc = bsga_gather_pool(a.q, A, A, a.dt, a.h, a.src, a.d, static_cast<const int32_t*>(a.ix), a.n, a.first, a.b, a.qo, A, a.vo, a.qp, a.kp, nullptr);
      refused += rc != BSGA_OK;
      return rc;
    };
    CHECK(pool([](GP&) {}) == BSGA_OK && pool([](GP& a) { a.first = 0; }) == BSGA_OK && pool([](GP& a) { a.first = 90; a.b = 128; a.dt = 1; }) == BSGA_OK);
    CHECK(pool([&](GP& a) { a.q = Z; }) == BSGA_ERR_INVALID_ARG && pool([&](GP& a) { a.q = O; }) == BSGA_ERR_INVALID_ARG && err_has("aligned"));
    CHECK(pool([&](GP& a) { a.vo = Z; }) == BSGA_ERR_INVALID_ARG && pool([&](GP& a) { a.qo = O; }) == BSGA_ERR_INVALID_ARG);
    CHECK(pool([&](GP& a) { a.ix = Z; }) == BSGA_ERR_INVALID_ARG && pool([](GP& a) { a.kp = nullptr; }) == BSGA_ERR_INVALID_ARG && err_has("k_pool"));
    CHECK(pool([](GP& a) { a.dt = 2; }) == BSGA_ERR_INVALID_ARG && pool([](GP& a) { a.h = 0; }) == BSGA_ERR_INVALID_ARG && err_has("heads"));
    CHECK(pool([](GP& a) { a.d = 32; }) == BSGA_ERR_UNSUPPORTED && pool([](GP& a) { a.b = 32; }) == BSGA_ERR_UNSUPPORTED);
    CHECK(pool([](GP& a) { a.src = 0; }) == BSGA_ERR_INVALID_ARG && err_has("n_src") && pool([](GP& a) { a.n = 0; }) == BSGA_ERR_INVALID_ARG);
    CHECK(pool([](GP& a) { a.first = 91; }) == BSGA_ERR_INVALID_ARG && err_has("n_first") && pool([](GP& a) { a.first = -1; }) == BSGA_ERR_INVALID_ARG);

    struct LN { const void *x, *w; int64_t n; int d; void* out; };
    auto norm = [&](LN a) {
      const int rc = bsga_layer_norm(a.x, a.w, A, 1e-5, a.n, a.d, nullptr, a.out, nullptr);
      refused += rc != BSGA_OK;
      return rc;
    };
    CHECK(norm({A, A, 1, 8, A}) == BSGA_OK && norm({A, A, 1 << 24, 4096, A}) == BSGA_OK);
    CHECK(norm({Z, A, 1, 8, A}) == BSGA_ERR_INVALID_ARG && norm({A, O, 1, 8, A}) == BSGA_ERR_INVALID_ARG && norm({A, A, 1, 8, Z}) == BSGA_ERR_INVALID_ARG);
    CHECK(norm({A, A, 0, 8, A}) == BSGA_ERR_INVALID_ARG && norm({A, A, (1 << 24) + 1, 8, A}) == BSGA_ERR_INVALID_ARG && err_has("n_tokens"));
    CHECK(norm({A, A, 1, 12, A}) == BSGA_ERR_UNSUPPORTED && norm({A, A, 1, 4104, A}) == BSGA_ERR_UNSUPPORTED && norm({A, A, 1, 0, A}) == BSGA_ERR_UNSUPPORTED);

    struct Lin { const void *x, *w, *b; int64_t n; int k, f, act; const void *ix, *res; int heads; void* out; };
    auto linear = [&](Lin a) {
      const int rc = bsga_linear(a.x, 0, a.w, a.b, a.n, a.k, a.f, a.act, static_cast<const int32_t*>(a.ix), a.res, a.heads, a.out, nullptr);
      refused += rc != BSGA_OK;
      return rc;
    };
    CHECK(linear({A, A, A, 1, 64, 64, 0, Z, Z, 0, A}) == BSGA_OK && linear({A, A, A, 100, 1024, 3072, 1, Z, Z, 1, A}) == BSGA_OK);
    CHECK(linear({A, A, A, 100, 64, 128, 0, A, A, 0, A}) == BSGA_OK);
    CHECK(linear({Z, A, A, 1, 64, 64, 0, Z, Z, 0, A}) == BSGA_ERR_INVALID_ARG && linear({A, Z, A, 1, 64, 64, 0, Z, Z, 0, A}) == BSGA_ERR_INVALID_ARG);
    CHECK(linear({A, A, O, 1, 64, 64, 0, Z, Z, 0, A}) == BSGA_ERR_INVALID_ARG && linear({A, A, A, 1, 64, 64, 0, Z, O, 0, A}) == BSGA_ERR_INVALID_ARG && err_has("aligned"));
    CHECK(linear({A, A, A, 0, 64, 64, 0, Z, Z, 0, A}) == BSGA_ERR_INVALID_ARG && linear({A, A, A, 1, 64, 64, 2, Z, Z, 0, A}) == BSGA_ERR_INVALID_ARG && err_has("activation"));
    CHECK(linear({A, A, A, 1, 96, 64, 0, Z, Z, 0, A}) == BSGA_ERR_UNSUPPORTED && linear({A, A, A, 1, 64, 32, 0, Z, Z, 0, A}) == BSGA_ERR_UNSUPPORTED && err_has("multiples of 64"));
    CHECK(linear({A, A, A, 1, 64, 64, 0, A, Z, 1, A}) == BSGA_ERR_UNSUPPORTED && linear({A, A, A, 1, 64, 64, 0, Z, A, 1, A}) == BSGA_ERR_UNSUPPORTED && err_has("row_index"));
    // just below 2 GiB with a tile to spare, and at it: x, weight, out
    CHECK(linear({A, A, A, (1 << 18) - 257, 4096, 64, 0, Z, Z, 0, A}) == BSGA_OK && linear({A, A, A, (1 << 18) - 256, 4096, 64, 0, Z, Z, 0, A}) == BSGA_ERR_UNSUPPORTED);
    CHECK(linear({A, A, A, 1, 4096, (1 << 18) - 320, 0, Z, Z, 0, A}) == BSGA_OK && linear({A, A, A, 1, 4096, (1 << 18) - 256, 0, Z, Z, 0, A}) == BSGA_ERR_UNSUPPORTED);
    CHECK(linear({A, A, A, (1 << 18) - 1, 64, 4096, 0, Z, Z, 0, A}) == BSGA_OK && linear({A, A, A, 1 << 18, 64, 4096, 0, Z, Z, 0, A}) == BSGA_ERR_UNSUPPORTED && err_has("2 GiB"));
    CHECK(g_calls - before == 11 && refused == 35);
  }

  // ---- the room for partial results is asked for where some call of the shape can use it, and nowhere else
  for (int heads : {1, 2, 3, 5, 8, 12, 16, 25, 40, 200})
    for (int64_t n = 1; n < 140000; n += n < 5000 ? 97 : 1013) {
      bool used = false;
      for (int64_t n_first : {n, n - 1, n / 2, int64_t(63), int64_t(1)}) {
        if (n_first < 0 || n_first > n) continue;
        for (int block : {64, 128})
          for (int block_k : {64, 128}) {
            if (block_k > block) continue;
            const int64_t tiles = bsga::ceil_div(bsga::split_blocks(n, n_first, block_k), block / block_k);
            used = used || bsga::shares_rows(heads * bsga::split_blocks(n, n_first, block), block, tiles, false);
          }
      }
      used = n > 4032 && (used || bsga::shares_rows(heads * bsga::ceil_div(n, 128), 128, bsga::ceil_div(n, 128), true));
      const size_t order = bsga::attn_order_bytes(heads, n);
      CHECK(bsga_attn_workspace_bytes(0, heads, n, 64) == order + (used ? bsga::kStreamBytes + 256 : 0));
    }
  // a layer of four frames of 1374 tokens, one head of 5000: nothing to share
  CHECK(bsga_attn_workspace_bytes(0, 16, 4 * 1374, 64) < (1 << 20) && bsga_attn_workspace_bytes(0, 1, 5000, 64) < (1 << 20));
  CHECK(bsga_attn_workspace_bytes(0, 2, 32 * 1374, 64) > (32 << 20) && bsga_attn_workspace_bytes(0, 1, 16400, 64) > (32 << 20));

  // ---- the size of a call's workspace reaches its own launch, and no later one's
  {
    const size_t order = bsga::attn_order_bytes(4, 1000);
    CHECK(bsga_sparse_attn(A, A, A, 0, 4, 1000, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 8, A, nullptr, A, sizeof(buf), nullptr) == BSGA_OK);
    CHECK(g_workspace_bytes == sizeof(buf));
    CHECK(bsga_sparse_attn(A, A, A, 0, 4, 1000, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 8, A, nullptr, A, order, nullptr) == BSGA_OK);
    CHECK(g_workspace_bytes == order);
    CHECK(bsga_sparse_attn(A, A, A, 0, 4, 1000, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 8, A, nullptr, nullptr, sizeof(buf), nullptr) == BSGA_OK);
    CHECK(g_workspace_bytes == 0);
  }

  // ---- an fp32 call hands its workspace on, of any size and place; a buffer of what the query says holds the parts
  {
    std::vector<unsigned char> room(bsga_attn_fp32_parts_bytes(3, 4100, 64, 1.0) + 16);
    CHECK(room.size() == size_t(3) * 4100 * 768 + 16);
    unsigned char* const at = reinterpret_cast<unsigned char*>((reinterpret_cast<uintptr_t>(room.data()) + 15) & ~uintptr_t(15));
    const size_t bytes = room.size() - 16;
    auto sparse = [&](void* ws, size_t n) {
      return bsga_sparse_attn(A, A, A, 1, 3, 4100, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 33, A, nullptr, ws, n, nullptr);
    };
    CHECK(sparse(at, bytes) == BSGA_OK && g_workspace_bytes == bytes);
    CHECK(sparse(at, 16) == BSGA_OK && g_workspace_bytes == 16);
    CHECK(sparse(nullptr, bytes) == BSGA_OK && g_workspace_bytes == 0);
    CHECK(bsga_dense_attn(A, A, A, 1, 3, 4100, 64, 0.125f, A, nullptr, at, bytes, nullptr) == BSGA_OK && g_workspace_bytes == bytes);
    CHECK(bsga_dense_attn(A, A, A, 1, 3, 4100, 64, 0.125f, A, nullptr, at, 8, nullptr) == BSGA_OK && g_workspace_bytes == 0);
  }
  // ---- a bf16 call that looks at its lists, in a workspace of the size that the query says
  {
    const int64_t n = int64_t(301) * 128 - 5, first = int64_t(299) * 128 + 1;
    std::vector<unsigned char> room(bsga_attn_workspace_bytes(0, 28, n, 64) + 16);
    void* const at = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(room.data()) + 15) & ~uintptr_t(15));
    CHECK(chooses_pairs(28, 301, 301));
    CHECK(bsga_sparse_attn(A, A, A, 0, 28, n, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 301, A, nullptr, at, room.size() - 16, nullptr) == BSGA_OK);
    CHECK(bsga_sparse_attn_split(A, A, A, 0, 28, n, first, 64, 128, 64, 0.125f, (int32_t*)A, (int32_t*)A, 604, A, nullptr, at, room.size() - 16, nullptr) == BSGA_OK);
  }

  // ---- the entry point on built-in scratch: size limit is checked before any device call; on a
  // machine without a GPU a fitting shape ends in a HIP error, never in a launch
  CHECK(bsga_noalloc_scratch_bytes() == (size_t(2) << 20));
  CHECK(bsga_sparse_attn_noalloc(A, A, A, 0, 4096, 1 << 20, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 1 << 14, A, nullptr, nullptr) == BSGA_ERR_UNSUPPORTED && err_has("scratch"));
  CHECK(bsga_sparse_attn_noalloc(A, A, A, 0, 4, 1000, 64, 128, 0.125f, nullptr, (int32_t*)A, 8, A, nullptr, nullptr) == BSGA_ERR_INVALID_ARG);
  {
    const int before = g_calls;
    const int rc = bsga_sparse_attn_noalloc(A, A, A, 0, 4, 1000, 64, 128, 0.125f, (int32_t*)A, (int32_t*)A, 8, A, nullptr, nullptr);
    CHECK(rc == BSGA_ERR_HIP || rc == BSGA_OK);
    CHECK(rc == BSGA_OK || g_calls == before);
  }

  // ---- probe
  double flops = 0.0;
  CHECK(bsga_probe_mfma(1, 2, 10, A, sizeof(buf), &flops, nullptr) == BSGA_OK && flops == 1.0);
  CHECK(bsga_probe_mfma(3, 0, 10, A, sizeof(buf), nullptr, nullptr) == BSGA_ERR_INVALID_ARG);
  CHECK(bsga_probe_mfma(0, 3, 10, A, sizeof(buf), nullptr, nullptr) == BSGA_ERR_INVALID_ARG);

  // ---- error strings never overflow their buffer
  CHECK(bsga_pool_qk(A, A, 0, 2147483647, 1000, 64, 128, (double*)A, (double*)A, nullptr) == BSGA_ERR_INVALID_ARG);
  CHECK(strlen(bsga_last_error()) < 512);

  printf("hostglue: %d stub launches, %d failed checks\n", g_calls, g_fail);
  return g_fail == 0 ? 0 : 1;
}
