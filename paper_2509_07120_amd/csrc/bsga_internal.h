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
constexpr int kStreamMaxRows = 1024;  // rows of a launch that shares them between workgroups are fewer
// Whether a launch of `rows` rows of at most `tiles` key tiles shares its rows out by tiles.  The plan, the
// partial results and their sum cost 15 to 20 us, so the work must be worth it; what there is to gain is
// idle CUs.  One workgroup per row / rows shared, all tiles kept (a quarter kept):
//  - Blocks of 64 (one workgroup: attn_few.hip): lists of unequal length gain, lists of one length lose.  Lengths uniform, a tenth of the rows full and
//    the rest a tenth, nine tenths kept, a quarter, a tenth: 313 rows of 313 tiles 118 / 80, 123 / 49, 125 / 122, 43 / 48, 24 / 31 us; 400 of 400 153 / 120,
//    157 / 62, 176 / 190, 57 / 67, 29 / 40; with fewer tiles less evens out, 256 of 256 74 / 62, 76 / 46, 77 / 87, 31 / 40, 16 / 28.
//  - Blocks of 128: a CU is busy with one workgroup, so 688 rows (2.7 per CU) gain nothing if they are equal,
//    876 / 897 us at 344 tiles, but 274 / 233 with a quarter kept in lists of unequal length; 344 rows (1.3 per CU)
//    521 / 468 (156 / 134) at 344 tiles, 139 / 131 (47 / 50) at 86; 172 rows of 172 148 / 134 (54 / 52), of 86
//    82 / 81 (36 / 39).
inline bool shares_rows(int64_t rows, int block, int64_t tiles, bool dense) {
  if (rows >= kStreamMaxRows) return false;
  if (block == 64) return rows <= 400 && tiles >= 256;
  const bool idle = 10 * rows < 8 * 256 * ceil_div(rows, 256);
  if (dense) return idle && rows * tiles >= 50 * 512;
  return rows * tiles >= (idle ? 200 : 300) * 512;  // whatever share of the tiles is kept, a tenth at least
}
// Such a launch needs room for partial results, whatever the number of rows: two of 33 KB for each of 512
// workgroups, and a table.
constexpr size_t kStreamBytes = 2 * 512 * (2 * 66 * 64 * sizeof(float)) + (size_t(1) << 14);
// Whether a call of this shape can come to share its rows, whatever its blocks, its lists and its split (which
// may add a block): only then does the workspace query count the room.  Up to 4032 tokens (63 blocks of 64) a row is
// too short to be worth sharing.
inline bool attn_stream_shape(int heads, int64_t n_tokens) {
  if (n_tokens <= 4032) return false;
  const int64_t h = heads, n64 = ceil_div(n_tokens, 64), n128 = ceil_div(n_tokens, 128);
  for (int more_q = 0; more_q < 2; ++more_q)
    for (int more_k = 0; more_k < 2; ++more_k) {
      if (shares_rows(h * (n64 + more_q), 64, n64 + more_k, false)) return true;
      if (shares_rows(h * (n128 + more_q), 128, n128 + more_k, false)) return true;
    }
  return shares_rows(h * n128, 128, n128, true);
}

constexpr int kPairMaxBlocks = 4096;  // key blocks of which two lists fit the LDS beside the tiles
// Whether blocks of 64 rows run with four independent waves to a block (attn_few.hip).  Larger launches go in pairs, or with two waves to a block
// where there are none (heads of one block, more key blocks than pairs take).
// Four waves that share their tiles up to 512 rows, two waves from there on / now, nine tenths kept (a tenth): 22 rows of 22 blocks 15.0 / 10.2 us
// (7.8 / 7.4), 172 of 43 24.0 / 17.1 (8.7 / 7.4), 352 of 22 21.7 / 16.7 (9.7 / 7.8), 512 of 128 82 / 68 (15.9 / 12.7), 688 of 43 45 / 38
// (11.5 / 12.4), 688 of 86 82 / 66.5 (15.5 / 14.6), 880 of 55 61 / 56.5 (14.2 / 15.6), 1,008 of 63 74 / 66.5 (16.3 / 16.1).  More than 512 rows of lists
// of a few blocks lose a microsecond, since the chip holds 512; how long the lists are the host does not know.
inline bool few_rows(int block, int64_t rows) { return block == 64 && rows < 1024; }
// Whether they are taken two to a workgroup (see PAIR).  Fewer than four rows per CU are better off with a
// workgroup each: 688 rows of 43 tiles, nine tenths kept, 49 us, paired 53; a quarter kept 18 and 25.
inline bool pairs_rows(int block, int heads, int nb, int nbk) {
  return block == 64 && int64_t(heads) * nb >= 1024 && nb >= 2 && nbk <= kPairMaxBlocks;
}

// Whether a dense launch takes blocks of 128 two to a workgroup of eight waves (see DUO).  Nothing runs beside the start and the end
// of a pair, so its rows have to be long, and the more so the more pairs a CU takes; and a CU with an odd row left idles half.
// Row by row / in pairs, us:
//  - Up to eight rows per CU, where the busiest CU has no more rows to work on in pairs.  16 heads: 2,748 tokens (1.4 rows) 41.5 / 39.9, 6,870
//    (3.4) 185 / 175, 10,992 (5.4) 431 / 419, 16,300 (8) 895 / 877; but 4,122 (2.1) 88 / 109, 8,244 (4.1) 267 / 312.  Heads of 16 blocks 37 /
//    36.6 (2 rows per CU), 75.3 / 72.7 (4), but of 8 23.5 / 23.9 (2), and of 24 at 6 144 / 146, 32 at 8 243 / 249 (48 at 6 270 / 265,
//    64 at 8 467 / 460).
//  - From there on where the last round of pairs is nearly full.  20,400 tokens (10) 1,401 / 1,361, 32,731 (16) 3,475 / 3,417, 36,827 (18)
//    4,381 / 4,351; but 19,000 (9.3) 1,220 / 1,241, 22,491 (11) 1,669 / 1,718, 27,000 (13.2) 2,401 / 2,440, 35,000 (17.1) 4,010 / 4,045.  51 heads of 100
//    blocks 1,737 / 1,706, 80 of 96 2,488 / 2,463, 80 of 64 1,199 / 1,211.
//  - From twenty rows per CU on rows of 256 blocks and more make up for the rest of a round: 41,179 (20.1) 5,444 / 5,345, 49,371 (24.1) 7,802 /
//    7,722, 137,400 (67) 60.8 / 58.0 ms.  Rows of 112: 46 heads (20.1) 1,956 / 1,966 and, on another card,
//    2,016 / 2,002.
// Short rows lose by the start of the pairs (1,024 heads of 2 blocks 47 / 61), heads of one block run every row twice.
inline bool dense_pairs(int heads, int nb) {
  const int64_t rows = int64_t(heads) * nb, rounds = ceil_div(int64_t(heads) * ((nb + 1) / 2), 256);  // of pairs
  if (rows <= 8 * 256) return nb >= (rows <= 4 * 256 ? 16 : 48) && 2 * rounds <= ceil_div(rows, 256);
  if (rows >= 20 * 256 && nb >= 256) return true;
  return nb >= 96 && 50 * 2 * rounds * 256 <= 51 * rows;
}
// Whether a sparse launch of blocks of 128 is large enough to look at its lists before it takes rows one by one or in pairs, and these fit
// the LDS.  The kernel that then is not meant costs 3 to 5 us (5,504 rows of 344 blocks, a twentieth and a tenth kept 397 -> 400 and 703 ->
// 707 us); what there is to gain (nine tenths kept, lists of one length, 5,764 -> 5,639) is less with fewer rows: 4,816 of 301 4,445 ->
// 4,385, 4,214 of 301 3,872 -> 3,869, 4,112 of 257 3,208 -> 3,238.
inline bool chooses_pairs(int heads, int nb, int nbk) {
  return int64_t(heads) * nb > 20 * 256 && nb >= 300 && nbk <= kPairMaxBlocks;
}
// What it looks for, in the sum of the lists' lengths and the sum of the differences between the two of a pair (half a difference is time
// that one of the two waits, and of a pair that differs by much each row is taken apart, see pair_differs).  One by one / in pairs, ms:
//  - Long rows, which make up for the start of a pair, that nothing runs beside: 16,384 rows of 512 blocks, lists of one length, four tenths
//    kept 11.28 / 11.42, six tenths 17.0 / 16.7, nine 25.2 / 24.6; 17,184 of 1,074, a quarter kept 15.6 / 15.4, half 30.7 / 30.3.
//  - 64 rows per CU and more, rows of 500 tiles: 17,184 rows of 1,074 blocks, nine tenths kept in lists of one length 55.2 / 53.3, lengths
//    within 5 % of eight tenths 52.5 / 50.0, within 12 % 53.7 / 52.7, within 20 % of seven 46.8 / 46.3; uniform, or alternating
//    7 : 9, no gain.
//  - Otherwise less evens out.  Shorter rows: 16,384 of 512 blocks within 20 % of seven tenths 20.8 / 20.9, 19,264 of 301 that alternate 8 : 9
//    17.34 / 17.54; within 5 % of nine 25.5 / 24.2, 17.23 / 16.76.  Fewer: within 20 % of seven tenths 513 blocks 10.35 / 10.47, 700
//    19.5 / 19.6, within 12 % of eight 11.66 / 11.59, 21.97 / 21.77; of one length, half kept, 512 blocks 6.97 / 7.02, 700, four tenths,
//    10.17 / 10.28, six tenths 15.27 / 15.12, nine 22.8 / 22.2, within 5 % of nine 12.60 / 12.13, 23.9 / 22.9.
inline __host__ __device__ bool pairs_pay(long long all, long long apart, long long rows, int nbk, int per_tile) {
  const bool many = rows >= 64 * 256;
  if (all < 260 * per_tile * rows || (!many && 10 * all < 6 * nbk * rows)) return false;
  return (many && all >= 500 * per_tile * rows ? 8 : 32) * apart <= all;
}

// Whether a pair's lists, of which `both` entries are common, differ so much in length that its rows are taken one after the other.  What idles
// is half the difference; another row costs 13 us, which is eight tiles, and the common tiles unshared, 3 % of them.
// (Sixteen entries for key blocks of 64 too: 17,184 rows, lengths within 5 % of eight tenths, 52.04 ms and not 51.80, 8,208 11.74 and not 11.63.)
inline __host__ __device__ bool pair_differs(int both, int alone0, int alone1, int per_tile) {
  const int apart = alone0 < alone1 ? alone1 - alone0 : alone0 - alone1;
  return apart > 16 * per_tile + (both >> 4);
}

constexpr int64_t kFp32FewUnits = 128;  // units of 64 rows, of which an fp32 launch goes to attn_fp32_kernel
// Bytes that K and V of an fp32 call take when they are split in three bf16 parts before the attention and not by every workgroup
// for itself; 0 where that gives nothing.  The pass over K and V costs about 10 us, the attention's steps get a sixth shorter.  Split by the
// workgroups / before, us: 688 rows of 64 that keep 4 tiles each 28 / 35, 9 tiles 48 / 50, 15 85 / 77, 39 203 / 167; 1,376 rows,
// 9 tiles 91 / 92, 17 178 / 162, 77 746 / 626.  Up to 512 rows the chip holds them all at once, and a step is only
// shorter, not cheaper: 344 rows, 15 tiles 49 / 54, 21 67 / 68, 30 93 / 90, 77 228 / 203.  The call uses the room whenever it has
// it; `kept` is what the caller expects the lists to hold of all key blocks.
constexpr int kPartRow = 6 * 64 * 2;  // three parts of a key, then of a value
constexpr size_t kPartsMaxBytes = size_t(256) << 20;  // 21,845 tokens of 16 heads; fp32 is for shorter sequences
inline size_t attn_fp32_parts_bytes(int heads, int64_t n_tokens, double kept) {
  const int64_t tiles = ceil_div(n_tokens, 64), rows = heads * tiles;
  const size_t bytes = static_cast<size_t>(heads) * static_cast<size_t>(n_tokens) * kPartRow;
  if (rows <= kFp32FewUnits || bytes > kPartsMaxBytes) return 0;
  return kept * static_cast<double>(tiles) >= (rows > 512 ? 12.0 : 25.0) ? bytes : 0;
}

// Kernel launchers.  Arguments are already validated.
// One tensor, or (x1 not null) two in one launch.
int launch_pool(const void* x0, double* pooled0, const void* x1, double* pooled1, int dtype, int heads, int64_t n_tokens, int64_t n_first,
                int block, hipStream_t stream);

int launch_select(const double* q_pool, const double* k_pool, int heads, int nb_q, int nb_k,
                  double score_scale, double tau, double one_minus_rho, const uint8_t* force_q,
                  const uint8_t* force_k, uint32_t* mask_bits, int32_t* kv_idx, int32_t* kv_cnt,
                  int idx_stride, void* workspace, hipStream_t stream);
size_t select_workspace_bytes(int heads, int nb_q, int nb_k);
int launch_gather_pool(const void* const (&x)[3], int dtype, int heads, int64_t n_src, const int32_t* index, int64_t n_tokens, int64_t n_first,
                       int block, void* const (&ordered)[3], double* const (&pooled)[3], hipStream_t stream);
int launch_linear(const void* x, bool x_heads, const void* weight, const void* bias, int64_t n_tokens, int in_features, int out_features, bool gelu,
                  const int32_t* row_index, const void* residual, bool out_heads, void* out, hipStream_t stream);
int launch_layer_norm(const void* x, const void* weight, const void* bias, float eps, int64_t n_tokens, int features, const int32_t* index, void* out,
                      hipStream_t stream);

int launch_gather(const void* src, int dtype, int heads, int64_t n_src, const int32_t* index,
                  int64_t n_dst, void* dst, hipStream_t stream);

int launch_attn_few(const void* q, const void* k, const void* v, int heads, int64_t n_tokens, int64_t n_first, float scale_log2,
                    const int32_t* kv_idx, const int32_t* kv_cnt, int idx_stride, void* out, float* lse, hipStream_t stream);
// workspace_bytes: of the call's workspace, 0 without one; the launch order alone or more (see attn_order_bytes).
int launch_attn_bf16(const void* q, const void* k, const void* v, int heads, int64_t n_tokens, int64_t n_first,
                     int block, int block_k, float softmax_scale, const int32_t* kv_idx, const int32_t* kv_cnt,
                     int idx_stride, void* out, float* lse, void* workspace, size_t workspace_bytes, hipStream_t stream);

// workspace: room for K and V split beforehand, kPartRow bytes per token and head; ignored if it is less or misaligned.
int launch_attn_fp32(const float* q, const float* k, const float* v, int heads, int64_t n_tokens, int64_t n_first,
                     int block, float softmax_scale, const int32_t* kv_idx, const int32_t* kv_cnt,
                     int idx_stride, float* out, float* lse, void* workspace, size_t workspace_bytes, hipStream_t stream);

int launch_probe_mfma(int pattern, int mix, int iters, float* sink, size_t sink_bytes, double* flops,
                      hipStream_t stream);

}  // namespace bsga
