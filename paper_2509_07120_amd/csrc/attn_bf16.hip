// bf16 flash-style attention over kept key blocks for gfx950 (Sec. 4.1, Eq. (2); Eq. (1) when no
// index list is given).  bf16 MFMA (32x32x16) for both products, fp32 accumulation, fp32 softmax
// weights in the log2 domain.
//
// Work split.  One workgroup per (head, query block of B rows); it walks the row's kept key
// blocks (tiles of B keys; with key blocks of B/2 keys a tile is two consecutive list entries).
// Blocks are those of a sequence cut in two separately blocked parts (Sec. 4.2; n_first = n_tokens
// is the plain blocking).  Waves are arranged WQ x 2: wave (qi, kh) owns 64 query rows (qi)
// and one half of every key tile (kh), so each K/V operand fetched from LDS into registers feeds
// two MFMAs (register-file traffic, not LDS bandwidth, is what this saves: LDS read data and MFMA
// operands share the VGPR ports).  The two key halves keep independent softmax states that are
// merged once at the end.  Two workgroups share a CU (two waves per SIMD).
// Which workgroup computes which row: see the end of the kernel (launch order, 64 consecutive rows
// per XCD, the last eighth of a large launch handed out at run time).  Launches of few long rows,
// blocks of 64 rows and large launches of blocks of 128 divide the work otherwise: STREAM, PAIR, DUO below;
// launches of few short rows go to attn_few.hip.
//
// Data movement.  K and V tiles go HBM/L2 -> LDS with direct-to-LDS loads (16 bytes per lane, no
// staging registers), double buffered, with one workgroup barrier per tile.  Tiles stay row-major
// [key][64]; only the order of the eight 16-byte chunks inside a row is permuted (XOR swizzle,
// chosen per tensor) so the operand reads below are bank-conflict free.
//
// Register layouts.  Scores are produced transposed, S^T = K Q^T (M = keys, N = queries): in the
// 32x32 accumulator layout lane (n = lane%32, g = lane/32) holds, for query n, the keys
// 8*r4 + 4*g + r (register 4*r4 + r).  A lane owns a whole query column, so row sums need one
// cross-lane step (lane ^ 32) at the very end, and after exponentiation the same registers are,
// with no data movement, the B operand of O^T += V^T P^T if the contraction index is taken in the
// order the accumulator holds the keys.  The matching A operand (V^T: 32 dims x 16 keys) is read
// from the row-major V tile with the LDS transpose read (ds_read_b64_tr_b16): each 16-lane group
// names four keys and gets, per lane, those four keys' values of one dim.
//
// Softmax.  Q is pre-multiplied by softmax_scale*log2(e) when it is loaded.  The fast pass takes
// the weights as exp2 of the raw scaled logits, i.e. with reference 0 for every row: any reference
// gives the same O / l, the choice only matters for range, and the range is checked afterwards
// (see pass()).  Only if that check fails is the workgroup repeated with a running reference
// maximum (SAFE pass).  V is multiplied by the bf16 roundings of the weights.  The pipelined loop
// of blocks of 128 rows sums those same bf16 weights (on the matrix pipe, see fast_loop), so numerator and
// denominator agree exactly; the plain tile code, and everything on blocks of 64 rows, sums the fp32 weights, which
// differ from the bf16 ones by at most one rounding (2^-9 relative), the size of rounding the output itself.
//
// Tile rows that are not keys of the listed block (past the end of a ragged block, or the absent
// second half of a tile of half-size key blocks) get weight exactly 0: their scores are set to -inf
// before they are exponentiated.  Only the plain tile code masks; the pipelined loop runs over the
// row's leading full tiles and hands the rest of the row to the plain code.
#include <stdio.h>
#include <stdlib.h>

#include <type_traits>

#include "bf16_tile.h"
#include "bsga_internal.h"

namespace bsga {
namespace {

constexpr int kD = 64;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRaise = 8.0f;  // SAFE pass: raise the reference maximum when a tile exceeds it by 2^8

template <int V>
using Int = std::integral_constant<int, V>;

__device__ __forceinline__ float xor32(float x) { return __shfl_xor(x, 32); }

// Launch order of the (head, query block) rows.  Rows much longer than the average (more kept key
// blocks) go first, longest first, so that they do not end up alone at the end of the grid; all
// other rows keep the natural order (head-major), because workgroups of equal length that start
// together walk the keys together and share the K/V tiles in L2, and reordering rows of nearly
// equal length would only break that up.  Counting sort by kOrderClasses classes of kept count /
// nb; the classes whose lower bound is below 1.4 x the mean count are merged into one.  Four small
// kernels: per-head class histogram -> merge -> exclusive scan of the [class][head] table ->
// placement.  The rows of the merged class keep their natural order inside a head (neighbouring
// query blocks tend to keep similar key blocks); rows of one of the longer (class, head) groups come
// out in arbitrary order, which only changes which workgroup computes which row.
constexpr int kOrderClasses = 32;

__device__ __forceinline__ int order_class(int cnt, int nb) {  // class 0 holds the longest rows
  const int c = min(max(cnt, 0), nb);
  return (kOrderClasses - 1) - static_cast<int>(static_cast<unsigned>(c) * (kOrderClasses - 1) / static_cast<unsigned>(nb));  // nb <= 2^18
}

// kept count of unit I of head h: of row I, or (pair) of the longer of rows 2I and 2I + 1
__device__ __forceinline__ int unit_count(const int32_t* __restrict__ kv_cnt, int h, int nb, int I, bool pair) {
  const int32_t* c = kv_cnt + int64_t(h) * nb;
  return pair ? max(c[2 * I], c[min(2 * I + 1, nb - 1)]) : c[I];
}

// A launch of pairs whose last ones go row by row has n_pairs units that are pairs, then the rows of the others, two units to each: the
// pair that unit u is of, and which of its rows (-1: both).  An odd head's last pair has a unit with nothing to do.
__device__ __forceinline__ int64_t pair_of(int64_t u, int64_t n_pairs, int& which) {
  which = u < n_pairs ? -1 : static_cast<int>((u - n_pairs) & 1);
  return u < n_pairs ? u : n_pairs + ((u - n_pairs) >> 1);
}

// Whether a large sparse launch of blocks of 128 takes them two to a workgroup (DUO) or one by one is known on the card only,
// because it depends on the lists, see pairs_pay.  The kernels below look at them (above kOrderOneMax rows the order is
// counted both ways and order_merge_kernel goes on with one of them) and leave which in `choice` (else null); both
// attention kernels are launched, of which one finds nothing to do.
// Below: nu = units (rows, or pairs of rows) per head.
__device__ __forceinline__ void read_choice(const int32_t* choice, int nb, int& nu, bool& pair) {
  if (choice == nullptr) return;
  pair = *choice != 0;
  nu = pair ? (nb + 1) >> 1 : nb;
}
// What order_hist_kernel leaves of the pairs: a table as that of the rows, lengths and differences of each head (2^24 at most).
constexpr int kPairsWords = kOrderClasses + 2;  // per head
__global__ __launch_bounds__(256) void order_hist_kernel(const int32_t* __restrict__ kv_cnt, int nb, int nu, bool pair, int nbk,
                                                         int heads, int32_t* __restrict__ table, int32_t* __restrict__ pairs) {
  __shared__ int bins[kOrderClasses], pair_bins[kPairsWords];
  const int h = blockIdx.x;
  const int t = threadIdx.x;
  if (t < kOrderClasses) bins[t] = 0;
  if (t < kPairsWords) pair_bins[t] = 0;
  __syncthreads();
  if (pairs == nullptr) {
    for (int I = t; I < nu; I += 256) atomicAdd(&bins[order_class(unit_count(kv_cnt, h, nb, I, pair), nbk)], 1);
  } else {
    const int32_t* const c = kv_cnt + int64_t(h) * nb;
    int all = 0, apart = 0;
    for (int i = 2 * t; i < nb; i += 512) {
      const int a = min(max(c[i], 0), nbk), b = i + 1 < nb ? min(max(c[i + 1], 0), nbk) : a;
      atomicAdd(&bins[order_class(a, nbk)], 1);
      if (i + 1 < nb) atomicAdd(&bins[order_class(b, nbk)], 1);
      atomicAdd(&pair_bins[order_class(max(a, b), nbk)], 1);
      all += a + b;
      apart += abs(a - b);
    }
    atomicAdd(&pair_bins[kOrderClasses], all);
    atomicAdd(&pair_bins[kOrderClasses + 1], apart);
  }
  __syncthreads();
  if (t < kOrderClasses) table[int64_t(t) * heads + h] = bins[t];
  if (pairs != nullptr && t < kPairsWords) pairs[int64_t(t) * heads + h] = pair_bins[t];
}

// The first class c whose lower bound (31 - c) / 31 is below 1.4 x the mean kept fraction, taking a unit at the
// middle of its class, (31 - c + 1/2) / 31; total(c) = units of class c.  In whole numbers.
template <typename Total>
__device__ __forceinline__ int bulk_class(Total&& total) {
  long long units = 0, mass = 0;  // mass: in units of 1/62
#pragma unroll
  for (int c = 0; c < kOrderClasses; ++c) {
    const long long n = total(c);
    units += n;
    mass += n * (2 * (kOrderClasses - 1 - c) + 1);
  }
  if (units == 0) mass = units = 1;  // nothing to order
  int c = 0;
  while (c < kOrderClasses - 1 && 10 * units * (kOrderClasses - 1 - c) >= 7 * mass) ++c;
  return c;
}

// One workgroup.  Finds the first class c_bulk whose lower bound (31 - c) / 31 is below 1.4 x the
// mean kept fraction, folds every lighter class into it (table rows c > c_bulk are added to row
// c_bulk and zeroed) and leaves c_bulk in table[kOrderClasses * heads].  pairs (or null): what order_hist_kernel has left of
// the pairs; whether the launch takes pairs goes to table[kOrderClasses * heads + 2], and if it does the table becomes theirs.
__global__ __launch_bounds__(256) void order_merge_kernel(int32_t* __restrict__ table, int heads, const int32_t* __restrict__ pairs, int nb,
                                                          int nbk, int per_tile) {
  __shared__ long long total[kOrderClasses];
  __shared__ int c_bulk;
  const int t = threadIdx.x;
  if (pairs != nullptr) {
    if (t < 2) total[t] = 0;
    __syncthreads();
    for (int64_t i = t; i < 2 * int64_t(heads); i += 256)
      atomicAdd(reinterpret_cast<unsigned long long*>(&total[i >= heads]), static_cast<unsigned long long>(pairs[int64_t(kOrderClasses) * heads + i]));
    __syncthreads();
    const bool pay = pairs_pay(total[0], total[1], static_cast<long long>(heads) * nb, nbk, per_tile);
    if (pay)
      for (int64_t i = t; i < int64_t(kOrderClasses) * heads; i += 256) table[i] = pairs[i];
    if (t == 0) table[int64_t(kOrderClasses) * heads + 2] = pay;
    __syncthreads();
  }
  if (t < kOrderClasses) total[t] = 0;
  __syncthreads();
  for (int64_t i = t; i < int64_t(kOrderClasses) * heads; i += 256)
    atomicAdd(reinterpret_cast<unsigned long long*>(&total[i / heads]), static_cast<unsigned long long>(table[i]));
  __syncthreads();
  if (t == 0) {
    const int c = bulk_class([&](int i) { return total[i]; });
    c_bulk = c;
    table[int64_t(kOrderClasses) * heads] = c;
    table[int64_t(kOrderClasses) * heads + 1] = 0;  // the attention kernel's counter of rows handed out at run time
  }
  __syncthreads();
  const int cb = c_bulk;
  for (int h = t; h < heads; h += 256) {
    int sum = 0;
    for (int c = cb; c < kOrderClasses; ++c) {
      sum += table[int64_t(c) * heads + h];
      table[int64_t(c) * heads + h] = 0;
    }
    table[int64_t(cb) * heads + h] = sum;
  }
}

// in-place exclusive scan of table[0 .. n) by one workgroup
__global__ __launch_bounds__(1024) void order_scan_kernel(int32_t* __restrict__ table, int64_t n) {
  __shared__ int part[1024];
  __shared__ int carry;
  const int t = threadIdx.x;
  if (t == 0) carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < n; base += 1024) {
    const int64_t i = base + t;
    const int x = i < n ? table[i] : 0;
    part[t] = x;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int add = t >= o ? part[t - o] : 0;
      __syncthreads();
      part[t] += add;
      __syncthreads();
    }
    const int before = carry;
    if (i < n) table[i] = before + part[t] - x;
    __syncthreads();
    if (t == 1023) carry = before + part[1023];
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void order_place_kernel(const int32_t* __restrict__ kv_cnt, int nb, int nu,
                                                          bool pair, int nbk, int heads, const int32_t* choice,
                                                          const int32_t* __restrict__ table, int32_t* __restrict__ order) {
  read_choice(choice, nb, nu, pair);
  __shared__ int next[kOrderClasses];
  __shared__ int wave_bulk[4];
  const int h = blockIdx.x;
  const int t = threadIdx.x;
  if (t < kOrderClasses) next[t] = table[int64_t(t) * heads + h];
  const int c_bulk = table[int64_t(kOrderClasses) * heads];
  __syncthreads();
  int bulk_next = next[c_bulk];  // every thread keeps its own copy of the bulk group's fill position
  for (int base = 0; base < nu; base += 256) {
    const int I = base + t;
    const int cls = I < nu ? min(order_class(unit_count(kv_cnt, h, nb, I, pair), nbk), c_bulk) : -1;
    // the bulk group keeps the natural order of its rows: rank of this row among the chunk's bulk rows
    const bool bulk = cls == c_bulk;
    const unsigned long long vote = __ballot(bulk);
    const int below = __popcll(vote & ((1ull << (t & 63)) - 1ull));
    if ((t & 63) == 0) wave_bulk[t >> 6] = __popcll(vote);
    __syncthreads();
    int before = 0, chunk = 0;
    for (int w = 0; w < 4; ++w) {
      before += w < (t >> 6) ? wave_bulk[w] : 0;
      chunk += wave_bulk[w];
    }
    if (bulk) order[bulk_next + before + below] = h * nu + I;
    else if (cls >= 0) order[atomicAdd(&next[cls], 1)] = h * nu + I;
    bulk_next += chunk;
    __syncthreads();
  }
}

// The whole launch order in one workgroup, for up to kOrderOneMax units: 5.4 us at 1,376 rows, 10.2 at 5,504 with the choice, where
// the four kernels above take 5 us each whatever the size, a fifth of an 8-frame layer at high sparsity.  The units
// of a thread are consecutive, so the bulk class keeps its order.  choice: where it leaves whether pairs are taken (or null: as `pair` says).
// singly: of the last so many pairs each row is a unit of its own (numbered as the attention kernel does, see pair_of).
constexpr int kOrderOneMax = 8192;
__global__ __launch_bounds__(1024) void order_one_kernel(const int32_t* __restrict__ kv_cnt, int nb, int nu, bool pair, int nbk,
                                                         int heads, int singly, int per_tile, int32_t* choice,
                                                         int32_t* __restrict__ order, int32_t* __restrict__ next_row) {
  constexpr int MAX = kOrderOneMax / 1024;
  __shared__ int total[kOrderClasses], next[kOrderClasses];
  __shared__ int c_bulk_s, wave_bulk[16], sum[2];
  const int t = threadIdx.x;
  if (t < kOrderClasses) total[t] = 0;
  if (choice != nullptr) {
    if (t < 2) sum[t] = 0;
    const int half = (nb + 1) >> 1;
    int all = 0, apart = 0;  // kOrderOneMax lists of kPairMaxBlocks are 2^25
#pragma unroll
    for (int i = 0; i < MAX / 2 + 1; ++i) {  // heads of an odd number of blocks have half a pair more
      const int u = t + i * 1024;
      if (u < heads * half) {
        const int h = u / half, r = 2 * (u - h * half);
        const int32_t* const c = kv_cnt + int64_t(h) * nb;
        const int x = min(max(c[r], 0), nbk), y = r + 1 < nb ? min(max(c[r + 1], 0), nbk) : x;
        all += x + y;
        apart += abs(x - y);
      }
    }
    for (int o = 1; o < 64; o <<= 1) {
      all += __shfl_xor(all, o);
      apart += __shfl_xor(apart, o);
    }
    __syncthreads();
    if ((t & 63) == 0) {
      atomicAdd(&sum[0], all);
      atomicAdd(&sum[1], apart);
    }
    __syncthreads();
    pair = pairs_pay(sum[0], sum[1], static_cast<long long>(heads) * nb, nbk, per_tile);
    if (pair) nu = half;
    if (t == 0) *choice = pair;
  }
  const int n_pairs = heads * nu - singly, units = n_pairs + 2 * singly;
  const int per = (units + 1023) >> 10;
  __syncthreads();
  int cls[MAX];
#pragma unroll
  for (int i = 0; i < MAX; ++i) {
    const int u = t * per + i;
    cls[i] = -1;
    if (i < per && u < units) {
      int which;
      const int p = static_cast<int>(pair_of(u, n_pairs, which)), h = p / nu, I = p - h * nu;
      const int cnt = which < 0 ? unit_count(kv_cnt, h, nb, I, pair) : 2 * I + which < nb ? kv_cnt[int64_t(h) * nb + 2 * I + which] : 0;
      cls[i] = order_class(cnt, nbk);
      atomicAdd(&total[cls[i]], 1);
    }
  }
  __syncthreads();
  if (t < 64) {  // bulk_class and the classes' first places, a class to a lane
    const int n = t < kOrderClasses ? total[t] : 0, weight = 2 * (kOrderClasses - 1 - t) + 1;
    int all = n, mass = n * weight, upto = n;
    for (int o = 1; o < 64; o <<= 1) {
      all += __shfl_xor(all, o);
      mass += __shfl_xor(mass, o);
      const int x = __shfl_up(upto, o);
      if (t >= o) upto += x;
    }
    if (t < kOrderClasses) next[t] = upto - n;
    const unsigned long long longer = __ballot(t < kOrderClasses - 1 && 10 * all * (kOrderClasses - 1 - t) >= 7 * mass);
    if (t == 0) {
      c_bulk_s = __popcll(longer);
      *next_row = 0;  // the attention kernel's counter of rows handed out at run time
    }
  }
  __syncthreads();
  const int c_bulk = c_bulk_s;
  int bulk = 0;
#pragma unroll
  for (int i = 0; i < MAX; ++i) bulk += cls[i] >= c_bulk;
  int upto = bulk;
  for (int o = 1; o < 64; o <<= 1) {
    const int x = __shfl_up(upto, o);
    if ((t & 63) >= o) upto += x;
  }
  if ((t & 63) == 63) wave_bulk[t >> 6] = upto;
  __syncthreads();
  int pos = next[c_bulk] + upto - bulk;
  for (int w = 0; w < (t >> 6); ++w) pos += wave_bulk[w];
#pragma unroll
  for (int i = 0; i < MAX; ++i) {
    if (cls[i] >= c_bulk) order[pos++] = t * per + i;
    else if (cls[i] >= 0) order[atomicAdd(&next[cls[i]], 1)] = t * per + i;
  }
}

__global__ void zero_word_kernel(int* __restrict__ word) {
  if (threadIdx.x == 0) *word = 0;
}

// Token blocks.  The sequence is two segments, tokens [0, n_first) and [n_first, n_tokens), each cut
// into blocks of its own (Sec. 4.2 keeps the patch tokens and the special tokens in separate blocks);
// nbq1 / nbk1 = number of query / key blocks of the first segment.  n_first = n_tokens is the plain
// single-segment blocking.
struct Segments {
  int n_first, nbq1, nbk1;
};

// A key tile of B keys in LDS.  With key blocks of B keys it is one listed block (a); with key blocks
// of B/2 keys it is two consecutive entries of the row's list, one per half (b < 0: the list ended,
// the second half is empty).
struct Tile {
  int a, b;
  unsigned oa, ob;  // byte offsets of the blocks' first keys inside the head (filled in by fix())
};

// Launches of few long rows (STREAM, see shares_rows() for which).  With one workgroup per row such a launch
// leaves much of the chip idle: 100 rows keep 100 CUs busy, and 688 rows of unequal length end with a few long
// ones.  Instead the key tiles of all rows, in order, are cut into equal pieces, one per workgroup that the
// chip holds (at least kMinQuota tiles each), and a workgroup walks its piece: the end of one row, whole rows,
// the start of another.
// A row that several workgroups share is summed by the last of them to finish (weights have reference 0
// everywhere, so partial sums just add up): every one leaves its unnormalised output and row sums in the
// workspace and counts itself in; the one that completes the count reads them all, in piece order, so the
// result does not depend on who came last.  Nobody waits for anybody.
// Sharing costs parts and their sum, so the plan leaves the rows whole (quota 0) where lists of nearly equal length
// would lose by it, see worth_sharing(): there is then a workgroup to each.  (One workgroup for several whole rows stays the
// oldest of its CU and holds up the other: 980 equal rows 616 -> 714 us.)
// Workspace of a launch: the table below, then two partial results per workgroup.
constexpr int kStreamMaxPlaces = 1024;   // workgroups: 2 x 256 (blocks of 128 rows), 4 x 256 (blocks of 64)
template <int B>
constexpr int kStreamPlaces = B == 64 ? kStreamMaxPlaces : kStreamMaxPlaces / 2;
constexpr int kMinQuota = 4;
struct StreamTable {
  int quota, used, pad[14];          // tiles to a piece (0: rows stay whole), number of pieces
  int start_row[kStreamMaxPlaces];   // workgroup w starts at tile start_tile[w] of row start_row[w]
  int start_tile[kStreamMaxPlaces];
  int arrived[kStreamMaxRows];       // pieces of the row that are done
};
constexpr size_t kStreamPartialWords = 66 * 64;  // per 64 query rows: 64 accumulators and 2 row sums of 64 lanes
static_assert(kStreamBytes >= sizeof(StreamTable) + 2 * 1024 * kStreamPartialWords * sizeof(float), "workspace of a STREAM launch");

// Partial results go between XCDs within a launch, so they are stored through to and loaded from the level that
// the XCDs share (cache bit sc1, device scope).  A store is waited for before the counter tells of it.  (A
// fence of device scope instead writes back and drops the whole L2 for every wave: 43 -> 207 us for one
// frame; atomic loads, one waited for after the other: 142 us.)
constexpr int kDeviceScope = 1 << 4;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t partial_rsrc(float* p) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, kStreamPartialWords * sizeof(float), 0x00020000);
}

// Whether rows of blocks of 128 gain by being shared.  In tiles per CU: what whole rows lose is the idle part of the last
// round of 256 rows, three tenths of which shows in the time, and the end of the longest rows; what sharing costs
// is a 25th and seven tiles.  us, whole rows without a plan / always shared / by this rule: 688 rows of 344 tiles, a tenth,
// a quarter, a half kept in lists of one length 99 / 112 / 102, 232 / 243 / 236, 450 / 460 / 450; lengths uniform
// 603 / 460 / 459; 344 rows, nine tenths, a tenth kept 489 / 416 / 414, 60 / 67 / 64; 980 rows of 196, a tenth 80 / 97 / 84.
__device__ __forceinline__ bool worth_sharing(int rows, int total, int longest) {
  const float mean = static_cast<float>(total) / rows, per_cu = total * (1.f / 256.f);
  const float idle = static_cast<float>((256 - (rows & 255)) & 255) * (1.f / 256.f);
  return 0.3f * idle * mean + 0.75f * (longest - mean) > 0.04f * per_cu + 7.f;
}

// One workgroup, one thread per row: prefix sums of the rows' tiles, then each row writes the pieces that
// start in it.  An empty row counts one tile, so that somebody writes its zeros.
__global__ __launch_bounds__(kStreamMaxRows) void stream_plan_kernel(const int32_t* __restrict__ kv_cnt, int rows, int nbk,
                                                                     int per_tile, int places, bool always, StreamTable* __restrict__ tab) {
  __shared__ int wave_sum[kStreamMaxRows / 64], wave_top[kStreamMaxRows / 64];
  const int t = threadIdx.x;
  const int lane = t & 63;
  int tiles = 0;
  if (t < rows) {
    const int cnt = kv_cnt != nullptr ? min(max(kv_cnt[t], 0), nbk) : nbk;
    tiles = max(1, (cnt + per_tile - 1) / per_tile);
    tab->arrived[t] = 0;
  }
  int end = tiles;
  for (int o = 1; o < 64; o <<= 1) {
    const int x = __shfl_up(end, o);
    if (lane >= o) end += x;
  }
  int top = tiles;
  for (int o = 1; o < 64; o <<= 1) top = max(top, __shfl_xor(top, o));
  if (lane == 63) {
    wave_sum[t >> 6] = end;
    wave_top[t >> 6] = top;
  }
  __syncthreads();
  int total = 0;
  for (int w = 0; w < kStreamMaxRows / 64; ++w) {
    end += w < (t >> 6) ? wave_sum[w] : 0;
    total += wave_sum[w];
    top = max(top, wave_top[w]);
  }
  if (!always && !worth_sharing(rows, total, top)) {  // the same in every thread
    if (t == 0) tab->quota = tab->used = 0;
    return;
  }
  const int quota = max(kMinQuota, (total + places - 1) / places);
  const int begin = end - tiles;
  for (int w = (begin + quota - 1) / quota; w * quota < end; ++w) {
    tab->start_row[w] = t;
    tab->start_tile[w] = w * quota - begin;
  }
  if (t == 0) {
    tab->quota = quota;
    tab->used = (total + quota - 1) / quota;
  }
}

// B: query rows per workgroup = keys per LDS tile.  KB: size of the key blocks the index list refers
// to, B or B/2.  STREAM: rows are shared out by tiles, see above.
//
// PAIR: the workgroup's 128 query rows are two blocks of 64 with a list each (KB = 64).  Tiles of two key
// blocks that both lists name go through the pipelined loop of the 128-row kernel, which a workgroup of one
// block of 64 cannot use (half the products per key loaded, and as many barriers and loads per tile); then a
// tile holds one key block of the first list alone and one of the second alone, and each wave takes
// half the keys of its own.  The two lists are sorted into these three in LDS (bit sets, then a scan), so they
// may come in any order; kPairMaxBlocks key blocks fit beside the tiles with two workgroups to a CU.
// 2,752 rows of 172 blocks, nine tenths kept: 515 -> 434 us; 5,504 of 344 1,910 -> 1,590.
// While the rest of the longer list runs, the waves of the other block idle.  A pair whose lists differ in length by
// more than what they share (and a dozen steps, about what another row's start and merge cost) is therefore taken
// row by row, four waves to each (ONE: its list dealt to the two halves in turn), and so is the odd block at the end of a head.  Lists of
// nine tenths
// and a twentieth in turn, 5,504 rows of 344: 1,080 us with two waves to a row, 1,500 in pairs only, 1,115 so.
//
// DUO: eight waves, one workgroup to a CU, take two neighbouring blocks of 128 rows (four waves to each, as above).  The part lowers its
// clock under large launches, and with no tiles moved at all the kernel is 10 % faster, half of that by a higher clock (loads left out
// after the first two tiles, 62.5 -> 56.2 ms, 1.60 -> 1.69 GHz).  Tiles that both rows need are loaded once for all eight
// waves, which halves the L2 -> LDS traffic: dense, 16 heads x 137,400 tokens 60.8 -> 58.0 ms, 43,968 6.35 -> 6.12 (by 0.4 to 4 % over
// cards).  The lists are sorted into common and own blocks as for PAIR (below a kept fraction of 0.3
// they stay as they are); own tiles follow, each group of four waves on its own, but with barriers for all eight.  That is no
// slower than two separate workgroups (dense without any sharing 60.8 -> 59.5: the groups stay in step, so what one loads the other
// finds in the L1); four buffers and a barrier for two tiles are (58.0 -> 58.8).
// A pair whose lists differ in length is taken row by row (`deal`), a row's tiles dealt to the two groups in turn.
// Nothing runs beside the start and the end of a pair, 13 us: Q is loaded while the lists are sorted, the first own tiles
// under the common ones, and every wave finishes 32 rows.
enum { kDone = -1, kByOne = -2 };  // what a workgroup of a pair has left to do
template <int B, int KB, bool STREAM, bool PAIR, bool DUO>
__global__ __launch_bounds__(DUO ? 512 : 2 * B, 2) void attn_bf16_kernel(
    const unsigned char* __restrict__ q, const unsigned char* __restrict__ k, const unsigned char* __restrict__ v,
    unsigned short* __restrict__ out, float* __restrict__ lse, const int32_t* __restrict__ kv_idx,
    const int32_t* __restrict__ kv_cnt, const int32_t* __restrict__ order, int idx_stride, int64_t n_tokens, int nb,
    int nbk, float scale_log2, Segments seg, int heads, int64_t n_static, int64_t n_pairs, int* __restrict__ next_row,
    const int32_t* choice, StreamTable* __restrict__ tab) {
  static_assert(KB == B || (2 * KB == B && B == 128), "key blocks are whole tiles or half tiles of 128");
  static_assert(!PAIR || (B == 128 && KB == 64 && !STREAM), "pairs of blocks of 64");
  static_assert(!DUO || (B == 128 && !STREAM && !PAIR), "pairs of blocks of 128");
  constexpr int NT = DUO ? 512 : 2 * B;   // threads
  constexpr int QB = PAIR ? 64 : B;       // query block size
  constexpr bool HALF = KB != B;          // two listed key blocks per tile
  constexpr int WQ = B / 64;              // waves along queries (64 rows each)
  constexpr int KW = B / 2;               // keys per wave per tile
  constexpr int NH = KW / 32;             // 32-key sub-tiles per wave per tile
  constexpr int NW = B / 32;              // waves that share a tile (DUO: of one of the two blocks)
  constexpr int TILE_BYTES = B * 128;     // one K or V tile
  // LDS layout: K buffers 0, 1, then V buffers 0, 1.  DUO: four buffer pairs, each K then V, see take_part.
  constexpr int V_BASE = DUO ? TILE_BYTES : 2 * TILE_BYTES;
  constexpr int BUF_BYTES = DUO ? 2 * TILE_BYTES : TILE_BYTES;  // from one buffer of a tensor to the other
  extern __shared__ __align__(16) unsigned char smem[];
  if (choice != nullptr && (*choice != 0) != DUO) return;  // see read_choice

  const int tid0 = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  const int gw = DUO ? wave & 3 : wave;  // number of the wave among those of its block ...
  const int gb = DUO ? wave >> 2 : 0;    // ... and which of the two blocks that is
  const int qi = gw % WQ;
  const int kh = gw / WQ;

  // One row (or pair of rows), or (STREAM) its tiles [tile0, tile1); the row's tiles are those of workgroups w0 .. w1, of which
  // this is number `me`.  ONE: the row is a single block of 64 that all four waves share, one of a
  // pair that is taken row by row; listed >= 0: its list is in LDS already, with that many blocks.
  // A pair: listed >= 0 means block `listed` of the two alone.  Returns kDone, or, with nothing done, kByOne if the row
  // or rows are to be run by ONE, or the length of the list that it has sorted into LDS for one row.
  // (Everything up to the dispatch at the end; not indented.)
  // DUO: `deal` means block `row` alone, its tiles dealt to the two groups of waves in turn.
  auto run = [&](auto onec, int64_t row, int tile0, int tile1, int w0, int w1, int me, int listed, bool deal) -> int {
  const int lane = DUO ? fresh_lane() : tid0 & 63;  // fresh: what follows from the lane is not kept from call to call
  const int tid = DUO ? wave * 64 + lane : tid0;
  const int n = lane & 31;
  const int g = lane >> 5;
  constexpr bool ONE = decltype(onec)::value;
  constexpr bool TWO = PAIR && !ONE;              // two blocks with a list each
  const int units = TWO || (DUO && !deal) ? (nb + 1) >> 1 : nb;  // rows, or pairs of rows, per head
  const int h = static_cast<int>(min(max(row / units, int64_t(0)), int64_t(heads - 1)));
  const int u_in_head = static_cast<int>(min(max(row - int64_t(h) * units, int64_t(0)), int64_t(units - 1)));
  const int I = TWO ? min(2 * u_in_head + qi, nb - 1) : DUO && !deal ? min(2 * u_in_head + gb, nb - 1) : u_in_head;  // this wave's query block
  const bool no_block = TWO && 2 * u_in_head + qi >= nb;            // the last pair of a head may be one block
  const int64_t head_bytes = int64_t(h) * n_tokens * 128;
  const int64_t rowid = int64_t(h) * nb + I;
  // this query block: first token and number of tokens (a block never crosses the segment boundary)
  const int n_tok = static_cast<int>(n_tokens);
  const int q_start = I < seg.nbq1 ? I * QB : seg.n_first + (I - seg.nbq1) * QB;
  const int q_valid = no_block ? 0 : min(QB, (I < seg.nbq1 ? seg.n_first : n_tok) - q_start);
  const int q_off = PAIR ? 0 : qi * 64;  // this wave's first row in the block
  // raw buffer views of this head's K and V (byte-addressed, bounds-checked by the hardware)
  const unsigned head_size = static_cast<unsigned>(n_tokens * 128);
  const i32x4 krsrc = make_rsrc(k + head_bytes, head_size);
  const i32x4 vrsrc = make_rsrc(v + head_bytes, head_size);
  const unsigned smem_addr =
      static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) unsigned char*)smem));

  // ---- Q fragments (B operand of S^T = K Q^T), pre-scaled: [query half][16-dim chunk]; lane (n, g)
  // holds dims 16c + 8g .. +7 of query row 32 b + n of the wave's 64 (rows past q_valid are computed, not stored).
  // A row with lists to sort asks for them first, so that both are on their way together.
  u32x4 q_raw[2][4];
  auto load_q = [&]() {
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2) {
      const int64_t row = min(int64_t(q_start) + q_off + b2 * 32 + n, n_tokens - 1);
#pragma unroll
      for (int c = 0; c < 4; ++c) q_raw[b2][c] = *reinterpret_cast<const u32x4*>(q + head_bytes + row * 128 + (2 * c + g) * 16);
    }
  };

  // ---- per-lane constants -------------------------------------------------------------------------
  // direct-to-LDS loads: wave-load j covers LDS bytes [1024 j, 1024 j + 1024) of a tile; this wave
  // issues j = wave + NW*i, i = 0..3, for the K tile and for the V tile.  Lane -> LDS position
  // p = 64 j + lane -> (row p/8, chunk position p%8) -> global chunk (p%8) ^ swz(row).  Row r_i is
  // r_0 + 8 NW i with r_0 < 8 NW, so swz_k(r_i) = swz_k(r_0) ^ swz_k(8 NW i) and swz_v(r_i) =
  // swz_v(r_0): the K offsets repeat with period KN in i up to a multiple of 1024 NW (which goes
  // into the wave-uniform offset), the V offsets differ by that multiple only.
  constexpr int KN = (B == 128) ? 2 : 4;
  const int dma_r0 = gw * 8 + (lane >> 3);
  const int dma_pc = lane & 7;
  unsigned koff[KN];
#pragma unroll
  for (int i = 0; i < KN; ++i) {
    const int r = dma_r0 + 8 * NW * i;
    koff[i] = r * 128 + ((dma_pc ^ swz_k(r)) << 4);
  }
  const unsigned voff = dma_r0 * 128 + ((dma_pc ^ swz_v(dma_r0)) << 4);
  // K operand reads (ds_read_b128) of the wave's sub-tile u: row r = kh*KW + 32u + n, logical chunk
  // 2c + g.  Since swz_k(r + 32) = swz_k(r) ^ 4, sub-tile 1 reads chunk c where sub-tile 0 reads c ^ 2.
  unsigned kaddr[4];
  {
    const int r = kh * KW + n;
#pragma unroll
    for (int c = 0; c < 4; ++c) kaddr[c] = r * 128 + (((2 * c + g) ^ swz_k(r)) << 4);
  }
  // V operand reads (transpose read, 8 bytes per lane): 16-lane group G = lane/16 covers dims
  // db*32 + 16*(G&1) .. +15 for key-slot half g = G/2; inside the group lane i names key
  // m = i/4 of the four and the dim quad j = i%4.  Key = kh*KW + 32u + 16cp + 8t + 4g + m.
  unsigned vaddr[2];
  {
    const int i16 = lane & 15, m = i16 >> 2, j = i16 & 3, G = lane >> 4;
    const int keyl = kh * KW + 4 * g + m;
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      const int cc = db * 4 + 2 * (G & 1) + (j >> 1);
      vaddr[db] = V_BASE + keyl * 128 + ((cc ^ swz_v(keyl)) << 4) + (j & 1) * 8;
    }
  }

  f32x16 o[2][2];  // O^T accumulators: [dim block][query half], this lane's query column
  float m_ref[2];  // SAFE pass: reference maximum per query column (log2 domain)
  float l_run[2];  // this lane's share of the row sums

  const bool dense = kv_idx == nullptr;
  constexpr int PER = HALF ? 2 : 1;  // list entries per tile
  const int count_row = no_block ? 0 : dense ? nbk : min(max(kv_cnt[rowid], 0), nbk);  // listed key blocks of the row
  // PAIR: blocks in both lists, then those of the first alone, at list[0 ..); those of the second alone at
  // list[nbk ..)
  unsigned short* const list = reinterpret_cast<unsigned short*>(smem + (DUO ? 2 : 1) * 4 * TILE_BYTES);
  int n_both = 0, n_alone[2] = {0, 0};
  constexpr bool LATE_Q = PAIR || DUO;
  if constexpr (!LATE_Q) load_q();
  if constexpr (ONE) {
    const int n_list = listed >= 0 ? listed : count_row;
    if (listed >= 0) load_q();
    if (listed < 0) {
      const int32_t* const idx0 = kv_idx + rowid * idx_stride;
      int j = idx0[min(tid, nbk - 1)];  // in one round of loads with the count, see below
      load_q();
      for (int e = tid; e < count_row; e += NT) {
        if (e != tid) j = idx0[e];
        list[(e & 1) * nbk + (e >> 1)] = static_cast<unsigned short>(min(max(j, 0), nbk - 1));
      }
    }
    n_alone[0] = (n_list + 1) >> 1;
    n_alone[1] = n_list >> 1;
    __syncthreads();
  } else if (DUO && dense) {
    load_q();
    n_both = nbk;  // also for the last pair of a head if it is one block: dense rows come out the same whatever their place
  } else if (DUO && deal) {
    const int32_t* const idx0 = kv_idx + rowid * idx_stride;
    int j = idx0[min(tid, nbk - 1)];
    load_q();
    for (int e = tid; e < count_row; e += NT) {
      if (e != tid) j = idx0[e];
      list[(e & 1) * nbk + (e >> 1)] = static_cast<unsigned short>(min(max(j, 0), nbk - 1));
    }
    n_alone[0] = (count_row + 1) >> 1;
    n_alone[1] = count_row >> 1;
    __syncthreads();
  } else if constexpr (PAIR || DUO) {
    unsigned char* const named = smem;  // per key block: in which of the two lists it is, kPairMaxBlocks each
    unsigned* const part = reinterpret_cast<unsigned*>(smem + 2 * kPairMaxBlocks);  // per 64 key blocks: two words of counts
    // counts and the first 256 entries of both lists in one round of loads: entries past a count are
    // whatever the buffer holds (idx_stride >= nbk) and are not used
    const int64_t id0 = int64_t(h) * nb + 2 * u_in_head + max(listed, 0);
    const bool two = listed < 0 && 2 * u_in_head + 1 < nb;
    const int32_t* const idx0 = kv_idx + id0 * idx_stride;
    const int32_t* const idx1 = two ? idx0 + idx_stride : idx0;
    if (DUO && !two) return kByOne;
    const int c0 = kv_cnt[id0], c1 = kv_cnt[two ? id0 + 1 : id0];
    int j0 = idx0[min(tid, nbk - 1)], j1 = idx1[min(tid, nbk - 1)];
    load_q();
    const int n0 = min(max(c0, 0), nbk), n1 = two ? min(max(c1, 0), nbk) : 0;
    auto enter = [&](int r, int J) { named[r * kPairMaxBlocks + min(max(J, 0), nbk - 1)] = 1; };
    auto uneven = [&](int both, int alone0, int alone1) {
      return __builtin_amdgcn_readfirstlane(DUO ? pair_differs(both, alone0, alone1, HALF ? 2 : 1) : abs(alone0 - alone1) > both + 12) != 0;
    };
    if (10 * (n0 + n1) < 6 * nbk) {
      if (!two || uneven(0, n0, n1)) return kByOne;
      // Short lists: of unrelated ones few blocks are in both, and sorting costs more than that saves.  5,504
      // rows of 344 tiles, a tenth kept: sorted 271 us, unsorted 249; a quarter 587, 567; half 1065 sorted.
      auto put = [&](int e, int a0, int a1) {
        if (e < n0) list[e] = static_cast<unsigned short>(min(max(a0, 0), nbk - 1));
        if (e < n1) list[nbk + e] = static_cast<unsigned short>(min(max(a1, 0), nbk - 1));
      };
      put(tid, j0, j1);
      for (int e = tid + NT; e < max(n0, n1); e += NT) put(e, idx0[e], idx1[e]);
      n_alone[0] = n0;
      n_alone[1] = n1;
      __syncthreads();
    } else {
      // A wave takes 64 key blocks at a time: two votes tell which list names them, and their counts, summed up over the
      // pieces before, where they go.  (One thread per 32 blocks, bit sets filled with atomics: 2 us more per pair.)
      const int pieces = (nbk + 63) >> 6;
      for (int i = tid; i < pieces * 4; i += NT) {
        reinterpret_cast<u32x4*>(named)[i] = u32x4{0u, 0u, 0u, 0u};
        reinterpret_cast<u32x4*>(named + kPairMaxBlocks)[i] = u32x4{0u, 0u, 0u, 0u};
      }
      __syncthreads();
      if (tid < n0) enter(0, j0);
      if (tid < n1) enter(1, j1);
      for (int e = tid + NT; e < max(n0, n1); e += NT) {
        j0 = idx0[e];
        j1 = idx1[e];
        if (e < n0) enter(0, j0);
        if (e < n1) enter(1, j1);
      }
      __syncthreads();
      auto votes = [&](int piece, unsigned long long (&set)[3]) {
        const unsigned long long b0 = __ballot(named[piece * 64 + lane] != 0), b1 = __ballot(named[kPairMaxBlocks + piece * 64 + lane] != 0);
        set[0] = b0 & b1;
        set[1] = b0 & ~b1;
        set[2] = b1 & ~b0;
      };
      unsigned long long set[3];
      for (int p = wave; p < pieces; p += NT / 64) {
        votes(p, set);
        if (lane == 0) {
          part[2 * p] = __popcll(set[0]) | (__popcll(set[1]) << 16);
          part[2 * p + 1] = __popcll(set[2]);
        }
      }
      __syncthreads();
      // the three counts (each at most 4096) in two words, summed over the pieces up to this lane's
      unsigned lo = lane < pieces ? part[2 * lane] : 0u, hi = lane < pieces ? part[2 * lane + 1] : 0u;
      auto add_from = [&](auto ctrl, auto rows) {  // adds the value of the lane that the DPP control names, 0 if there is none
        constexpr int C = decltype(ctrl)::value, R = decltype(rows)::value;
        lo += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), C, R, 0xf, false));
        hi += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(hi), C, R, 0xf, false));
      };
      add_from(Int<0x111>{}, Int<0xf>{});  // 1, 2, 4, 8 lanes before, within a row of 16
      add_from(Int<0x112>{}, Int<0xf>{});
      add_from(Int<0x114>{}, Int<0xf>{});
      add_from(Int<0x118>{}, Int<0xf>{});
      add_from(Int<0x142>{}, Int<0xa>{});  // last lane of rows 0 and 2 into rows 1 and 3
      add_from(Int<0x143>{}, Int<0xc>{});  // lane 31 into rows 2 and 3
      const unsigned all = __builtin_amdgcn_readlane(lo, 63);
      n_both = static_cast<int>(all & 0xffff);
      n_alone[0] = static_cast<int>(all >> 16);
      n_alone[1] = static_cast<int>(__builtin_amdgcn_readlane(hi, 63));
      if (two && uneven(n_both, n_alone[0], n_alone[1])) return kByOne;
      const int at[3] = {0, n_both, nbk};
      for (int p = wave; p < pieces; p += NT / 64) {
        votes(p, set);
        const unsigned before_lo = p > 0 ? __builtin_amdgcn_readlane(lo, p - 1) : 0u, before_hi = p > 0 ? __builtin_amdgcn_readlane(hi, p - 1) : 0u;
        const int before[3] = {static_cast<int>(before_lo & 0xffff), static_cast<int>(before_lo >> 16), static_cast<int>(before_hi)};
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          const int pos = __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(set[x] >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(set[x]), at[x] + before[x]));
          if ((set[x] >> lane) & 1) list[two ? pos : (pos & 1) * nbk + (pos >> 1)] = static_cast<unsigned short>(p * 64 + lane);
        }
      }
      __syncthreads();  // the lists are complete; the tiles may overwrite the rest
      if (!two) return n_alone[0];
    }
  }
  bf16x8 qf[2][4];
#pragma unroll
  for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      u32x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = __uint_as_float(q_raw[b2][c][e] << 16) * scale_log2;
        const float hi = __uint_as_float(q_raw[b2][c][e] & 0xffff0000u) * scale_log2;
        y[e] = pack_bf16(lo, hi);
      }
      qf[b2][c] = __builtin_bit_cast(bf16x8, y);
    }
  int count = PAIR || DUO ? n_both : count_row;  // of them, those of the tiles this workgroup takes,
  int ntiles = HALF ? (count + 1) >> 1 : count;  // the number of these tiles
  int first = 0;                                // and the first one
  auto take_tiles = [&](int t0, int t1) {
    first = t0;
    ntiles = min(t1, (count_row + PER - 1) / PER) - t0;
    count = min(count_row - t0 * PER, ntiles * PER);
  };
  if constexpr (STREAM) take_tiles(tile0, tile1);
  int lbase = 0;  // DUO: where in `list` these are
  // DUO: on to the blocks in both lists, or to those of this wave's block alone.  Buffer pairs in the LDS, 32 KB each:
  //   first block's own tile 0 | shared tile 0, first block's own tile 1 | shared tile 1, second block's own tile 1 | its own tile 0
  // so the first of the own tiles can be loaded before the shared ones are through.  Of two neighbouring pairs, `flip` says
  // whether even tiles go to the upper.
  int flip = 0;
  auto take_part = [&](bool both) {
    count = both ? n_both : gb ? n_alone[1] : n_alone[0];
    ntiles = HALF ? (count + 1) >> 1 : count;
    lbase = both ? 0 : gb ? nbk : n_both;
    flip = both ? 0 : gb;
  };
  // key block J: first token and number of tokens.  Blocks of the first segment (J < nbk1) tile
  // tokens [0, n_first), the others tokens [n_first, n_tokens); the last block of each may be ragged.
  auto key_start = [&](int J) { return J < seg.nbk1 ? J * KB : seg.n_first + (J - seg.nbk1) * KB; };
  auto key_count = [&](int J) { return min(KB, (J < seg.nbk1 ? seg.n_first : n_tok) - key_start(J)); };

  // The row's key-block list is the same for the whole workgroup, so its entries are fetched with
  // scalar loads (the list is read through a constant-address-space pointer: it is never written
  // while the kernel runs), which do not count as vector memory operations: the waits on the
  // direct-to-LDS loads (vmcnt) stay exact.  raw_at(it) only issues the loads of tile `it` (any it;
  // past the end it repeats the last tile) and hands back the unchecked entries; the caller keeps
  // them for a tile before fix() turns them into block numbers, so nothing waits for the load.
  typedef const int32_t __attribute__((address_space(4))) * const_idx_ptr;
  const const_idx_ptr cidx = dense ? (const_idx_ptr) nullptr : (const_idx_ptr)(kv_idx + rowid * idx_stride);
  auto raw_at = [&](int it) -> Tile {
    if constexpr (PAIR) {
      const int e = min(it, ntiles - 1) * 2;
      return Tile{list[e], list[min(e + 1, count - 1)], 0u, 0u};
    } else if constexpr (DUO) {
      if (dense) return Tile{min(it, nbk - 1), -1, 0u, 0u};
      const int e = min(it, ntiles - 1) * PER;
      Tile t{list[lbase + e], -1, 0u, 0u};
      if constexpr (HALF) t.b = list[lbase + min(e + 1, count - 1)];
      return t;
    } else if constexpr (STREAM) {
      if (dense) return Tile{min(first + it, nbk - 1), -1, 0u, 0u};
      const int e = first * PER + min(it, ntiles - 1) * PER;
      Tile t{cidx[e], -1, 0u, 0u};
      if constexpr (HALF) t.b = cidx[min(e + 1, first * PER + count - 1)];
      return t;
    } else {
      if (dense) return Tile{min(it, nbk - 1), -1, 0u, 0u};
      const int e = min(it, ntiles - 1) * PER;
      Tile t{cidx[e], -1, 0u, 0u};
      if constexpr (HALF) t.b = cidx[min(e + 1, count - 1)];
      return t;
    }
  };
  // An absent second half gets an offset past the end of the head's buffer: the bounds check of
  // the loads then zero-fills it.
  auto fix = [&](const Tile& r, int it) -> Tile {  // r = raw_at(it)
    Tile t{r.a, -1, 0u, head_size};
    if constexpr (PAIR || DUO) {  // dense too: uniform already
      t.a = __builtin_amdgcn_readfirstlane(r.a);
      if (HALF && min(it, ntiles - 1) * 2 + 1 < count) t.b = __builtin_amdgcn_readfirstlane(r.b);
    } else if (!dense) {
      t.a = min(max(r.a, 0), nbk - 1);
      if constexpr (HALF) {
        if (min(it, ntiles - 1) * 2 + 1 < count) t.b = min(max(r.b, 0), nbk - 1);
      }
    }
    t.oa = static_cast<unsigned>(key_start(t.a)) * 128u;
    if constexpr (HALF) {
      if (t.b >= 0) t.ob = static_cast<unsigned>(key_start(t.b)) * 128u;
    }
    return t;
  };
  auto block_at = [&](int it) -> Tile { return fix(raw_at(it), it); };
  // The offsets are operands of scalar type in the load instructions.  A tile description that has
  // been carried around a loop may live in vector registers (the same value in every lane): this
  // moves the offsets back.
  auto scalar = [&](Tile t) -> Tile {
    t.oa = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(t.oa)));
    t.ob = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(t.ob)));
    return t;
  };
  // This wave's keys of a tile are the tile rows [kh*KW, (kh+1)*KW).  wave_limit(t) is the first of
  // them that is not a key of the listed block (a ragged block, or an absent second half): rows at
  // or past it hold zeros or tokens of another block, and their scores are masked before they are
  // exponentiated.  A full tile gives (kh+1)*KW.
  auto wave_limit = [&](const Tile& t) {
    const int J = (HALF && kh == 1) ? t.b : t.a;
    const int cnt = J < 0 ? 0 : key_count(J);
    return HALF ? kh * KW + cnt : min(cnt, (kh + 1) * KW);
  };
  // scores of a 32-key sub-tile: keys at or past `limit` (tile row numbers) get weight 0
  // (register i of the lane is tile row row0 + 8(i/4) + 4g + i%4).  Runs for the few ragged
  // tiles only; the lane number is taken afresh through an opaque instruction, so that nothing of
  // this is computed ahead and kept in registers across the tile loops.
  auto mask_keys = [&](f32x16& sc, int row0, int limit) {  // row0: tile row of the sub-tile's first key
    const int l = fresh_lane();
    const int t = limit - row0 - ((l >> 5) << 2);  // row 8(i/4) + i%4 is masked iff it is >= t
#pragma unroll
    for (int i = 0; i < 16; ++i) sc[i] = (8 * (i >> 2) + (i & 3) >= t) ? -INFINITY : sc[i];
  };
  // Does the tile hold rows that are not keys of its listed block(s)?  The same answer in every wave
  // of the workgroup (the pipelined loop below leaves such tiles to the plain tile code, and all
  // waves must agree on that).  Only the last block of each segment can be short.
  const int short_a = (seg.n_first % KB) != 0 ? seg.nbk1 - 1 : -1;
  const int short_b = ((n_tok - seg.n_first) % KB) != 0 ? nbk - 1 : -1;
  auto tile_ragged = [&](const Tile& t) {
    bool r = t.a == short_a || t.a == short_b;
    if constexpr (HALF) r = r || t.b < 0 || t.b == short_a || t.b == short_b;
    return r;
  };
  // Direct-to-LDS load number i2 (0..7) of key tile J into buffer pair `buf`: even i2 moves 1 KB of
  // the K tile, odd i2 1 KB of the V tile.  Rows that lie past the end of the head's buffer fail
  // the hardware bounds check, which makes the load write zeros for them (so V rows past the end
  // are finite; rows past a ragged block inside the sequence hold the following tokens).
  // With half-tile key blocks, loads i = 0, 1 fill tile rows 0..63 from block a and i = 2, 3 rows
  // 64..127 from block b (an absent b: zero-filled, see fix()).
  // `both` (DUO): the eight waves load the tile together, four parts each: wave-load j = wave + 8 i, of which rows r_0 + 64 i.
  const unsigned dma_base = smem_addr + gw * 1024 + (DUO ? gb * 2 * BUF_BYTES : 0);  // this wave's 1 KB slice of every 4 KB (2 KB) group
  auto issue_part = [&](auto bothc, const Tile& J, auto bufc, auto i2c) {
    constexpr int buf = decltype(bufc)::value, i2 = decltype(i2c)::value;
    if constexpr (decltype(bothc)::value) {
      constexpr int i = i2 >> 1;
      if constexpr (i < 2) {
        constexpr unsigned dst = 2 * NW * i * 1024 + ((i2 & 1) ? V_BASE : 0) + buf * BUF_BYTES;
        const unsigned at = smem_addr + BUF_BYTES + wave * 1024, soff = HALF && i ? J.ob : J.oa + (HALF ? 0 : i * 2 * NW * 1024);
        if ((i2 & 1) != 0) dma16<dst>(vrsrc, voff + gb * 4096, soff, at);
        else dma16<dst>(krsrc, gb ? koff[1 % KN] : koff[0], soff, at);
      }
      return;
    } else {
    constexpr int i = i2 >> 1;
    constexpr bool is_v = (i2 & 1) != 0;
    constexpr unsigned dst = NW * i * 1024 + (is_v ? V_BASE : 0) + buf * BUF_BYTES;
    if constexpr (HALF) {
      const unsigned soff = (i >> 1) ? J.ob : J.oa;
      if (is_v) {
        dma16<dst>(vrsrc, voff, soff + (i & 1) * NW * 1024, dma_base);
      } else {
        dma16<dst>(krsrc, koff[i % KN], soff, dma_base);
      }
    } else {
      const unsigned soff = J.oa;
      if (is_v) {
        dma16<dst>(vrsrc, voff, soff + i * NW * 1024, dma_base);
      } else {
        dma16<dst>(krsrc, koff[i % KN], soff + (i / KN) * KN * NW * 1024, dma_base);
      }
    }
    }
  };
  auto issue = [&](auto both, const Tile& J, auto bufc) {
    issue_part(both, J, bufc, Int<0>{}); issue_part(both, J, bufc, Int<1>{}); issue_part(both, J, bufc, Int<2>{}); issue_part(both, J, bufc, Int<3>{});
    issue_part(both, J, bufc, Int<4>{}); issue_part(both, J, bufc, Int<5>{}); issue_part(both, J, bufc, Int<6>{}); issue_part(both, J, bufc, Int<7>{});
  };
  auto issue_rt = [&](auto both, const Tile& J, int buf) {  // buffer known at run time only
    if (buf) issue(both, J, Int<1>{});
    else issue(both, J, Int<0>{});
  };

  // K operands (A of S^T = K Q^T) of the wave's 32-key sub-tile u; boff = byte offset of the buffer
  auto read_k_at = [&](const unsigned (&at)[4], bf16x8 (&ka)[4], unsigned boff, int u) {
#pragma unroll
    for (int c = 0; c < 4; ++c) ka[c] = *LDS_PTR(bf16x8, smem + boff + at[(u & 1) ? (c ^ 2) : c] + u * 4096);
  };
  auto read_k = [&](bf16x8 (&ka)[4], unsigned boff, int u) { read_k_at(kaddr, ka, boff, u); };
  // V^T operands (A of O^T += V^T P^T) of sub-tile u: [dim block][16-key chunk]
  auto read_v_at = [&](const unsigned (&at)[2], bf16x8 (&va)[2][2], unsigned boff, int u) {
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int cp = 0; cp < 2; ++cp) {
        const unsigned char* p = smem + boff + at[db] + (32 * u + 16 * cp) * 128;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
        const s16x4 hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + 8 * 128));
        const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
        const u32x4 av = {lo2[0], lo2[1], hi2[0], hi2[1]};
        va[db][cp] = __builtin_bit_cast(bf16x8, av);
      }
  };
  auto read_v = [&](bf16x8 (&va)[2][2], unsigned boff, int u) { read_v_at(vaddr, va, boff, u); };

  // weights of key pair j (registers 2j, 2j+1) of a score block: exp2, add to the row sum, round to
  // bf16, store as word j of the two B operands.  The row sum takes the fp32 weights with two plain
  // adds: on this part a dot2 of the packed pair costs four times as much as an add and, unlike the
  // exp2 and the adds, does not run beside the matrix pipe.
  auto weigh_pair = [&](const f32x16& sc, u32x4 (&w)[2], float& lsum, int j) {
    const float e0 = __builtin_amdgcn_exp2f(sc[2 * j]), e1 = __builtin_amdgcn_exp2f(sc[2 * j + 1]);
    lsum += e0 + e1;
    w[j >> 2][j & 3] = pack_bf16(e0, e1);
  };

  // ---------------------------------------------------------------------------------------------
  // One tile, plain form: per (32-key sub-tile, query half) scores (4 MFMAs) -> weights -> O update
  // (4 MFMAs), from the tile buffers at byte offset boff.  `limit` = wave_limit of the tile.
  //   SAFE = true: online softmax.  The accumulator of the score MFMA starts at -m_ref, so the MFMA
  //   result is already relative to the reference, and m_ref is raised only when a sub-tile exceeds
  //   it by more than 2^kRaise.
  //   SAFE = false: reference 0, no maximum.
  // In both forms the scores of tile rows that are not keys of the listed block are masked.
  // after_reads() runs once every LDS read of the tile has been consumed.
  // ka, va, sc, w: working registers (the pipelined loop lends its own, which are free between runs).
  // row0, nh: the wave's first tile row and number of 32-key sub-tiles; kat, vat: its operand addresses there.
  auto compute_rows = [&](auto safec, auto nhc, int row0, const unsigned (&kat)[4], const unsigned (&vat)[2], unsigned boff,
                          int limit, auto&& after_reads, bf16x8 (&ka)[4], bf16x8 (&va)[2][2], f32x16 (&sc)[2],
                          u32x4 (&w)[2][2]) {
    constexpr bool SAFE = decltype(safec)::value;
    constexpr int nh = decltype(nhc)::value;
    const bool ragged = limit < row0 + 32 * nh;
#pragma unroll
    for (int u = 0; u < nh; ++u) {
      read_k_at(kat, ka, boff, u);
      read_v_at(vat, va, boff, u);
      // the scores of both query halves first (eight MFMAs in a row), so that the weights of the
      // first half are computed while the matrix pipe still works on the second, and the O update
      // of the first half runs under the weights of the second
      float base[2];
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        base[b2] = (SAFE && m_ref[b2] != -INFINITY) ? m_ref[b2] : 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) sc[b2][i] = -base[b2];
#pragma unroll
        for (int c = 0; c < 4; ++c) sc[b2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[c], qf[b2][c], sc[b2], 0, 0, 0);
      }
      if (ragged) {
        mask_keys(sc[0], row0 + 32 * u, limit);
        mask_keys(sc[1], row0 + 32 * u, limit);
      }
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        if constexpr (SAFE) {
          float tmax = -INFINITY;
#pragma unroll
          for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, sc[b2][i]);
          tmax = fmaxf(tmax, xor32(tmax));
          const bool unset = m_ref[b2] == -INFINITY;
          const bool raise = unset ? (tmax > -INFINITY) : (tmax > kRaise);
          if (__any(raise)) {  // rare after the first tile
            const float shift = raise ? tmax : 0.f;
            const float alpha = unset ? 1.f : exp2f(-shift);  // nothing accumulated yet while unset
            if (raise) m_ref[b2] = base[b2] + shift;
            l_run[b2] *= alpha;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
              for (int i = 0; i < 16; ++i) o[db][b2][i] *= alpha;
#pragma unroll
            for (int i = 0; i < 16; ++i) sc[b2][i] -= shift;
          }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) weigh_pair(sc[b2], w[b2], l_run[b2], j);
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
          for (int cp = 0; cp < 2; ++cp)
            o[db][b2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[db][cp], __builtin_bit_cast(bf16x8, w[b2][cp]),
                                                                o[db][b2], 0, 0, 0);
      }
      if (u == nh - 1) after_reads();
    }
  };
  auto compute_tile = [&](auto safec, unsigned boff, int limit, auto&& after_reads, bf16x8 (&ka)[4],
                          bf16x8 (&va)[2][2], f32x16 (&sc)[2], u32x4 (&w)[2][2]) {
    compute_rows(safec, Int<NH>{}, kh * KW, kaddr, vaddr, boff, limit, after_reads, ka, va, sc, w);
  };

  // Plain tile loop: compute_tile per tile, one barrier per tile, the next tile's loads in flight
  // meanwhile.  Used for the SAFE pass and by workgroups of one block of 64 rows and two waves.
  // DUO: `steps` tiles take the workgroup's barriers, ntiles of them (or none) are this wave's.
  auto plain_loop = [&](auto safec, auto both, int steps) {
    if (steps <= 0) return;
    Tile J_cur{0, -1, 0u, 0u};
    if (!DUO || ntiles > 0) {
      J_cur = block_at(0);
      if (!DUO || decltype(both)::value) issue(both, scalar(J_cur), Int<0>{});
    }
    Tile J_pre = raw_at(1);  // list entries are fetched a tile before they are used
    bf16x8 ka[4], va[2][2];
    f32x16 sc[2];
    u32x4 w[2][2];
    for (int it = 0; it < steps; ++it) {
      const int buf = (it + flip) & 1;
      const Tile J_next = (it + 1 < ntiles) ? fix(J_pre, it + 1) : Tile{0, -1, 0u, 0u};
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share of tile `it` has landed
      __syncthreads();                     // ... and so has everyone else's; buffer buf^1 is free
      if (DUO && it >= ntiles) continue;
      if (it + 1 < ntiles) issue_rt(both, scalar(J_next), buf ^ 1);
      // The list entries of the tile after next.  Scalar loads return out of order with LDS reads, so
      // a wait for LDS data would also wait for them: they are issued where every LDS read of the
      // tile has been consumed, and used at the top of the next tile.
      compute_tile(safec, buf * BUF_BYTES, wave_limit(J_cur), [&]() { J_pre = raw_at(it + 2); }, ka, va, sc, w);
      J_cur = J_next;
    }
  };

  // PAIR: the key blocks that one list alone names.  Tile rows 0..63 hold one of the first block's, rows
  // 64..127 one of the second's; wave (qi, kh) takes keys 32 kh .. 32 kh + 31 of its own.
  auto alone_loop = [&](auto safec) {
    const int steps = max(n_alone[0], n_alone[1]);
    if (steps <= 0) return;
    const int row0 = qi * 64 + kh * 32;
    unsigned kat[4], vat[2];
    {
      const int l = fresh_lane();  // so that the addresses are not kept in registers across the other loop
      const int r = row0 + (l & 31);
#pragma unroll
      for (int c = 0; c < 4; ++c) kat[c] = r * 128 + (((2 * c + (l >> 5)) ^ swz_k(r)) << 4);
      const int i16 = l & 15, m = i16 >> 2, j = i16 & 3, G = l >> 4;
      const int keyl = row0 + 4 * (l >> 5) + m;
#pragma unroll
      for (int db = 0; db < 2; ++db)
        vat[db] = V_BASE + keyl * 128 + (((db * 4 + 2 * (G & 1) + (j >> 1)) ^ swz_v(keyl)) << 4) + (j & 1) * 8;
    }
    auto raw = [&](int it) { return Tile{list[n_both + min(it, n_alone[0])], list[nbk + min(it, max(n_alone[1] - 1, 0))], 0u, 0u}; };
    auto made = [&](const Tile& r, int it) {
      Tile t{-1, -1, head_size, head_size};
      if (it < n_alone[0]) t.a = __builtin_amdgcn_readfirstlane(r.a);
      if (it < n_alone[1]) t.b = __builtin_amdgcn_readfirstlane(r.b);
      if (t.a >= 0) t.oa = static_cast<unsigned>(key_start(t.a)) * 128u;
      if (t.b >= 0) t.ob = static_cast<unsigned>(key_start(t.b)) * 128u;
      return t;
    };
    Tile cur = made(raw(0), 0);
    issue(std::false_type{}, scalar(cur), Int<0>{});
    Tile pre = raw(1);
    bf16x8 ka[4], va[2][2];
    f32x16 sc[2];
    u32x4 w[2][2];
    for (int it = 0; it < steps; ++it) {
      const Tile nxt = made(pre, it + 1);
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share of tile `it` has landed
      __syncthreads();                     // ... and so has everyone else's; the other buffer is free
      if (it + 1 < steps) issue_rt(std::false_type{}, scalar(nxt), (it & 1) ^ 1);
      pre = raw(it + 2);
      const int J = qi ? cur.b : cur.a;
      const int limit = qi * 64 + (J < 0 ? 0 : key_count(J));
      if (limit > row0) compute_rows(safec, Int<1>{}, row0, kat, vat, (it & 1) * TILE_BYTES, limit, []() {}, ka, va, sc, w);
      cur = nxt;
    }
  };

  // ---------------------------------------------------------------------------------------------
  // Fast pass for block 128: the same arithmetic as compute_tile<SAFE = false>, software pipelined
  // inside the wave.  A unit is (32-key sub-tile u, query half b): scores QK (4 MFMAs into 16
  // registers), weights W (16 exp2, 8 packs, 16 adds), O update PV (4 MFMAs).  A tile has four units
  // n = 0..3 = (u0,b0), (u0,b1), (u1,b0), (u1,b1).  While the VALU works on W(n) the matrix pipe gets
  // QK(n+1) and PV(n-1), one MFMA per four VALU instructions, so the wave's VALU and MFMA streams
  // overlap instead of waiting for each other.  K operands of a sub-tile serve two units, V operands
  // likewise; they are fetched from LDS at least half a unit ahead of their first use.  By the end
  // of unit 1 every LDS read of the tile has been issued, so at the start of unit 2 the workgroup
  // synchronises once: the next tile is known to have landed (its first K operands are read right
  // after the last score MFMA of this tile) and the current buffers are free, so the eight loads of
  // the tile after next are issued into them, one after each of the following MFMAs.
  //
  // The pipelined code has no masking in it (a conditional in the slot sequence costs 5 %): it runs
  // over the row's leading full tiles.  From the first tile with rows that are not keys (a short
  // block, an absent half) the remaining tiles go through compute_tile, which masks.  With ascending
  // lists that is the row's last tile, or, for a split sequence with the short first segment's
  // blocks listed last but a few, the last few tiles.  Either way a tile costs every wave exactly
  // one barrier, and the loads stay two tiles ahead.
  auto fast_loop = [&](auto both, int steps) {  // as plain_loop
    constexpr bool BOTH = decltype(both)::value;
    if (steps <= 0) return;
    f32x16 sc[2];        // scores: [query half]
    u32x4 pw[2][2];      // weights as packed bf16 pairs: [query half][16-key chunk]
    bf16x8 ka[4];        // K operands of the sub-tile whose scores are computed next
    bf16x8 va[2][2][2];  // V^T operands: [sub-tile][dim block][16-key chunk]
    float ex[2][2];      // exponentiated scores of the key pair that is packed in the next slot
    // Row sums on the matrix pipe.  In v_mfma_f32_16x16x32_bf16 lane l supplies, as B operand, eight
    // bf16 values B[k][j] of column j = l%16 with k = 8(l/16) .. 8(l/16)+7, supplies row l%16 of A for
    // the same eight k, and receives D[4(l/16) + r][l%16] in accumulator register r = 0..3.  With
    //   A_h[i][k] = 1 if i%4 == h and k/8 == i/4, else 0
    // the product D = A_h B puts, in register h of every lane, the sum of that lane's own eight B
    // values, and nothing in the other registers.  The B operand is the very register tuple of packed
    // weights that the O update multiplies with V, so two such instructions per unit (h = the query
    // half) sum the sixteen weights a lane holds: they replace sixteen fp32 adds per unit (64 cycles
    // of vector issue in a loop whose vector and matrix pipes are both saturated) by 32 cycles of
    // matrix pipe, and the sums are over the bf16 weights, exactly the values that multiply V.
    // Not for pairs of blocks of 64 (SUM32): their other tiles, and launches of few rows, sum fp32 weights, and a
    // row's lse must not depend on which way its blocks went.  The sixteen adds cost a hundredth:
    // 2,752 rows of 172 blocks, nine tenths kept, 428 us with the MFMAs, 433 with the adds.
    constexpr bool SUM32 = PAIR;
    f32x4 lacc = {0.f, 0.f, 0.f, 0.f};
    bf16x8 row_sel[2];
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      const bool on = (lane & 3) == h2 && (lane >> 4) == ((lane & 15) >> 2);
      const unsigned w1 = on ? 0x3F803F80u : 0u;  // two bf16 ones
      row_sel[h2] = __builtin_bit_cast(bf16x8, u32x4{w1, w1, w1, w1});
    }
    auto add_weights = [&](auto hc, const u32x4& words) {
      lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(row_sel[decltype(hc)::value], __builtin_bit_cast(bf16x8, words), lacc, 0,
                                                      0, 0);
    };

    // one unit N = (sub-tile N/2, query half N%2).  Slots 0..3: MFMA of QK(N+1) + one weight pair;
    // slots 4..7: MFMA of PV(N-1) + one weight pair.  mid(slot) places LDS reads, the barrier and
    // loads after that slot's MFMA.
    auto unit = [&](auto nc, auto&& mid) {
      constexpr int N = decltype(nc)::value;
      constexpr int BQ = N & 1;                 // query half whose weights are computed
      constexpr int BN = (N + 1) & 1;           // query half of QK(N+1)
      constexpr int BP = (N + 3) & 1;           // query half of PV(N-1)
      constexpr int UP = ((N + 3) & 3) >> 1;    // sub-tile of PV(N-1)
#define BSGA_SLOT(S_)                                                                                          \
  {                                                                                                            \
    if constexpr ((S_) < 4) {                                                                                  \
      if constexpr ((S_) == 0) {                                                                               \
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};   \
        sc[BN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[0], qf[BN][0], zero, 0, 0, 0);                     \
      } else {                                                                                                 \
        sc[BN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[(S_) & 3], qf[BN][(S_) & 3], sc[BN], 0, 0, 0);      \
      }                                                                                                        \
    } else {                                                                                                   \
      /* the two dim blocks alternate: consecutive MFMAs are independent and share the weights  */         \
      o[(S_) & 1][BP] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                                               \
          va[UP][(S_) & 1][((S_) >> 1) & 1], __builtin_bit_cast(bf16x8, pw[BP][((S_) >> 1) & 1]), o[(S_) & 1][BP], 0, \
          0, 0);                                                                                               \
    }                                                                                                          \
    /* weights, staggered by one slot so that no instruction waits for the one just before it:   */          \
    /* pack pair S_ (exponentiated in the previous slot), with SUM32 sum it (two fp32 adds), then */          \
    /* exponentiate the next pair.                                                               */          \
    {                                                                                                          \
      const unsigned pk = pack_bf16(ex[(S_) & 1][0], ex[(S_) & 1][1]);                                         \
      if constexpr (SUM32) { /* pinned: summed up later, all of a unit's weights would stay alive */           \
        l_run[BQ] += ex[(S_) & 1][0] + ex[(S_) & 1][1];                                                        \
        asm volatile("" : "+v"(l_run[BQ]));                                                                    \
      }                                                                                                        \
      if constexpr ((S_) < 7) {                                                                                \
        ex[((S_) + 1) & 1][0] = __builtin_amdgcn_exp2f(sc[BQ][2 * (S_) + 2]);                                  \
        ex[((S_) + 1) & 1][1] = __builtin_amdgcn_exp2f(sc[BQ][2 * (S_) + 3]);                                  \
      } else {                                                                                                 \
        ex[0][0] = __builtin_amdgcn_exp2f(sc[BN][0]);                                                          \
        ex[0][1] = __builtin_amdgcn_exp2f(sc[BN][1]);                                                          \
      }                                                                                                        \
      __builtin_amdgcn_sched_barrier(0);                                                                       \
      /* row sums: the previous unit's second group of weights in slot 1, this unit's first in slot 5 */    \
      if constexpr (!SUM32 && (S_) == 1) add_weights(Int<BP>{}, pw[BP][1]);                                    \
      if constexpr (!SUM32 && (S_) == 5) add_weights(Int<BQ>{}, pw[BQ][0]);                                    \
      pw[BQ][(S_) >> 2][(S_) & 3] = pk;                                                                        \
    }                                                                                                          \
    mid(Int<(S_)>{});                                                                                          \
    __builtin_amdgcn_sched_barrier(0);                                                                         \
  }
      BSGA_SLOT(0) BSGA_SLOT(1) BSGA_SLOT(2) BSGA_SLOT(3) BSGA_SLOT(4) BSGA_SLOT(5) BSGA_SLOT(6) BSGA_SLOT(7)
#undef BSGA_SLOT
    };

    // a whole (full) tile in buffer pair `buf` (byte offset boff; the other pair is at boff ^ BUF_BYTES).
    // On entry: sc[0] = QK(0) of this tile, ka = K operands of sub-tile 0, pw[1] / va[1] = weights /
    // V operands of the previous tile's unit 3 (zeros at the start of a run).  What it prepares for
    // the following tile (K operands and first scores from the other buffer) goes unused when the run
    // ends here.
    auto tile = [&](const Tile& J_next2, auto bufc) {
      constexpr int buf = decltype(bufc)::value;
      constexpr unsigned boff = buf * BUF_BYTES;
      unit(Int<0>{}, [&](auto slot) {  // QK(1); K(u1); PV(previous 3); V(u0)
        constexpr int S = decltype(slot)::value;
        if constexpr (S == 0) read_v(va[0], boff, 0);
        if constexpr (S == 3) read_k(ka, boff, 1);
      });
      unit(Int<1>{}, [&](auto slot) {  // QK(2); PV(0); V(u1)
        constexpr int S = decltype(slot)::value;
        if constexpr (S == 0) read_v(va[1], boff, 1);
      });
      unit(Int<2>{}, [&](auto slot) {  // synchronise; QK(3); K(next tile u0); PV(1) + loads 0..3
        constexpr int S = decltype(slot)::value;
        if constexpr (S == 0) {
          __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share of the next tile has landed
          __syncthreads();                     // every read of this tile is complete in every wave
        }
        if constexpr (S == 3) read_k(ka, boff ^ BUF_BYTES, 0);
        if constexpr (S >= 4) issue_part(both, J_next2, bufc, Int<S - 4>{});
      });
      unit(Int<3>{}, [&](auto slot) {  // QK(next tile's unit 0); PV(2) + loads 4..7
        constexpr int S = decltype(slot)::value;
        if constexpr (S >= 4 && !BOTH) issue_part(both, J_next2, bufc, slot);
      });
    };

    // ---- tiles 0 and 1 on their way ----------------------------------------------------------------
    Tile J_cur{0, -1, 0u, 0u};
    if (!DUO || ntiles > 0) {
      J_cur = block_at(0);
      if (!DUO || BOTH) issue(both, scalar(J_cur), Int<0>{});  // own tiles of DUO: under way already
    }
    Tile J_nxt = J_cur;
    if (ntiles > 1) {
      J_nxt = block_at(1);
      if constexpr (DUO && !BOTH) issue_rt(both, scalar(J_nxt), flip ^ 1);
      else issue(both, scalar(J_nxt), Int<1>{});
    }
    Tile J_pre = raw_at(2);  // fetched one tile before it becomes "the tile after next"
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    // Invariant at the top of the loop: tile T lies in buffer T&1 and every wave knows it; the loads
    // of tile T+1 into the other buffer have been issued; J_cur / J_nxt are tiles T / T+1 and J_pre
    // holds the raw list entries of tile T+2.
    int T = 0;
    if ((!DUO || ntiles > 0) && !tile_ragged(J_cur)) {
      // ---- the run of full tiles: K operands of sub-tile 0, QK(0), nothing pending for the O update --
      if (DUO && flip) read_k(ka, BUF_BYTES, 0);
      else read_k(ka, 0u, 0);
#pragma unroll
      for (int cp = 0; cp < 2; ++cp) {
        pw[1][cp] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int db = 0; db < 2; ++db) va[1][db][cp] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
      }
      {
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        sc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[0], qf[0][0], zero, 0, 0, 0);
#pragma unroll
        for (int c = 1; c < 4; ++c) sc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[c], qf[0][c], sc[0], 0, 0, 0);
      }
      ex[0][0] = __builtin_amdgcn_exp2f(sc[0][0]);
      ex[0][1] = __builtin_amdgcn_exp2f(sc[0][1]);
      __builtin_amdgcn_sched_barrier(0);
      // two tiles per round, so that every LDS address is a constant of the code (even tiles lie in
      // buffer pair 0, odd ones in pair 1)
      auto step = [&](auto bufc) {
        // the tile after next; at the end of the list one more (harmless) load of a valid tile
        const Tile J2 = scalar((T + 2 < ntiles) ? fix(J_pre, T + 2) : J_cur);
        J_pre = raw_at(T + 3);
        tile(J2, bufc);
        J_cur = J_nxt;
        J_nxt = J2;
        ++T;
        return T < ntiles && !tile_ragged(J_cur);
      };
      // The place of the loop in the code matters, the same every 32 bytes and not for all lists alike, and changes with the code before
      // it.  Dense, 43,968 tokens, nine tenths of as many, of 137,400 and, with key blocks of 64, of 43,968: here 6,196, 5,723, 55,695 and
      // 5,985 us, on a multiple of 32 6,192, 5,761, 56,185 and 5,973 (a scene of 100 frames 2.7 % slower), 8 past one 6,280, 5,737, 55,698,
      // 5,966, 16 past one 6,192, 5,733, 55,829, 6,034.
      if constexpr (DUO && BOTH) asm volatile(".p2align 6\n\ts_nop 0");
      for (bool odd = DUO && !BOTH && flip != 0; odd || step(Int<0>{}); odd = false)
        if (!step(Int<1>{})) break;
      // ---- the O update and the last row-sum step of the run's last unit ------------------------------
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int cp = 0; cp < 2; ++cp)
          o[db][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[1][db][cp], __builtin_bit_cast(bf16x8, pw[1][cp]),
                                                             o[db][1], 0, 0, 0);
      if constexpr (!SUM32) {
        add_weights(Int<1>{}, pw[1][1]);
        l_run[0] += lacc[0];
        l_run[1] += lacc[1];
      }
    }
    // ---- from the first ragged tile on: plain tiles (the same buffers and the same one barrier per
    // tile; the loads stay two tiles ahead) ------------------------------------------------------------
    for (; T < ntiles; ++T) {
      compute_tile(std::false_type{}, ((T + flip) & 1) * BUF_BYTES, wave_limit(J_cur), []() {}, ka, va[0], sc, pw);
      const Tile J2 = scalar((T + 2 < ntiles) ? fix(J_pre, T + 2) : J_cur);
      J_pre = raw_at(T + 3);
      __builtin_amdgcn_s_waitcnt(0x0F70);  // this wave's share of tile T+1 has landed
      __syncthreads();                     // ... everyone's has, and nobody still reads tile T
      issue_rt(both, J2, (T + flip) & 1);
      J_cur = J_nxt;
      J_nxt = J2;
    }
    if constexpr (DUO && !BOTH) {
      for (; T < steps; ++T) __syncthreads();  // the other block's tiles
    }
  };

  // DUO: the end of a pass, as below.  Of the two waves that hold the key halves of 64 query rows each finishes 32, and
  // leaves the other its share of the other 32; then (deal) the second four waves theirs to the first four.
  auto end_duo = [&](auto safec) -> bool {
    constexpr bool SAFE = decltype(safec)::value;
    constexpr int WORDS = 34 * 64;  // 32 accumulators, reference maximum and row sum of 64 lanes
    const int lane = fresh_lane(), n = lane & 31, g = lane >> 5;
    float* const parked = reinterpret_cast<float*>(smem) + 16;
    volatile int* flag = reinterpret_cast<volatile int*>(smem);
    auto leave = [&](float* at, const f32x16& x0, const f32x16& x1, float m, float l) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        at[i * 64 + lane] = x0[i];
        at[(16 + i) * 64 + lane] = x1[i];
      }
      at[32 * 64 + lane] = m;
      at[33 * 64 + lane] = l;
    };
    f32x16 x[2];
    float m, l;
    if (kh == 0) {
      leave(parked + wave * WORDS, o[0][1], o[1][1], m_ref[1], l_run[1]);
      x[0] = o[0][0];
      x[1] = o[1][0];
      m = m_ref[0];
      l = l_run[0];
    } else {
      leave(parked + wave * WORDS, o[0][0], o[1][0], m_ref[0], l_run[0]);
      x[0] = o[0][1];
      x[1] = o[1][1];
      m = m_ref[1];
      l = l_run[1];
    }
    if (wave == 0 && lane == 0) *flag = 0;
    auto take = [&](const float* at) {
      float a0 = 1.f, a1 = 1.f;
      if constexpr (SAFE) {
        const float m1 = at[32 * 64 + lane], top = fmaxf(m, m1);
        const float mu = (top == -INFINITY) ? 0.f : top;
        a0 = exp2f(m - mu);  // exp2f(-inf) = 0 for a half that saw nothing
        a1 = exp2f(m1 - mu);
        m = top;
      }
      l = l * a0 + at[33 * 64 + lane] * a1;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        x[0][i] = x[0][i] * a0 + at[i * 64 + lane] * a1;
        x[1][i] = x[1][i] * a0 + at[(16 + i) * 64 + lane] * a1;
      }
    };
    __syncthreads();
    take(parked + (wave ^ 2) * WORDS);
    l += xor32(l);
    if (deal) {
      if (gb == 1) leave(parked + (8 + gw) * WORDS, x[0], x[1], m, l);
      __syncthreads();
      if (gb == 0) take(parked + (8 + gw) * WORDS);
    }
    const bool writes = !(deal && gb == 1);
    if constexpr (!SAFE) {
      bool bad = false;
      if (writes && count_row > 0) {  // an empty row is zeros by definition, not a range problem
        bad = !(l >= 0x1p-80f && l <= 0x1p100f);
#pragma unroll
        for (int i = 0; i < 16; ++i) bad = bad || !(fabsf(x[0][i]) < INFINITY) || !(fabsf(x[1][i]) < INFINITY);
      }
      if (bad) *flag = 1;
      __syncthreads();
      const bool any_bad = *flag != 0;
      __syncthreads();
      if (any_bad) return true;
    }
    const int lrow = q_off + kh * 32 + n;
    if (writes && lrow < q_valid) {
      const int64_t row = int64_t(q_start) + lrow;
      const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const int i = 4 * r4;
          const u32x2 w = {pack_bf16(x[db][i] * inv, x[db][i + 1] * inv), pack_bf16(x[db][i + 2] * inv, x[db][i + 3] * inv)};
          *reinterpret_cast<u32x2*>(out + (int64_t(h) * n_tokens + row) * kD + db * 32 + 8 * r4 + 4 * g) = w;
        }
      if (lse != nullptr && g == 0) lse[int64_t(h) * n_tokens + row] = l > 0.f ? ((SAFE ? m : 0.f) + log2f(l)) * kLn2 : -INFINITY;
    }
    return false;
  };

  // A whole pass over the row's key tiles, then the merge of the two key halves (wave (qi, 1) parks
  // its state in LDS as [qi][68 values][64 lanes] and wave (qi, 0) folds it in) and the output.
  // Returns true (to every thread of the workgroup) if the fast pass must be repeated in SAFE mode
  // because a row sum or an output left the range in which reference-free weights are trustworthy:
  // a weight 2^s overflows for s >= 128 (the row sum then exceeds the upper limit, or O is not
  // finite), and weights below 2^-126 flush to zero, which is harmless as long as the row sum is at
  // least 2^-80 (at most 2^24 keys x 2^-126 lost: a relative error under 2^-22).
  auto pass = [&](auto safec) -> bool {
    constexpr bool SAFE = decltype(safec)::value;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][b2][i] = 0.f;
    m_ref[0] = m_ref[1] = -INFINITY;
    l_run[0] = l_run[1] = 0.f;
    if constexpr (DUO) {
      auto shift = [&](unsigned by) {
#pragma unroll
        for (int c = 0; c < 4; ++c) kaddr[c] += by;
        vaddr[0] += by;
        vaddr[1] += by;
      };
      const int most = max(n_alone[0], n_alone[1]);
      take_part(false);
      if (ntiles > 0) issue_rt(std::false_type{}, scalar(block_at(0)), flip);
      if (n_both > 0) {
        take_part(true);
        shift(BUF_BYTES);
        if constexpr (SAFE) plain_loop(safec, std::true_type{}, ntiles);
        else fast_loop(std::true_type{}, ntiles);
        shift(0u - BUF_BYTES);
        take_part(false);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // no load may still be on its way into the buffers ...
        __syncthreads();                     // ... nor anyone read them
      }
      if (most > 0) {
        shift(gb * 2 * BUF_BYTES);
        const int steps = HALF ? (most + 1) >> 1 : most;
        if constexpr (SAFE) plain_loop(safec, std::false_type{}, steps);
        else fast_loop(std::false_type{}, steps);
        shift(0u - gb * 2 * BUF_BYTES);
      }
    } else if constexpr (!SAFE && B == 128) fast_loop(std::false_type{}, ntiles);
    else plain_loop(safec, std::false_type{}, ntiles);
    if constexpr (PAIR) {
      __builtin_amdgcn_s_waitcnt(0x0F70);  // no load may still be on its way into the buffers ...
      __syncthreads();                     // ... nor anyone read them
      alone_loop(safec);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // no direct-to-LDS load may still be in flight
    __syncthreads();                     // ... in any wave: LDS can be reused

    if constexpr (DUO) return end_duo(safec);
    float* park = reinterpret_cast<float*>(smem) + 16 + qi * 68 * 64;
    if (kh == 1) {
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
          for (int i = 0; i < 16; ++i) park[((db * 2 + b2) * 16 + i) * 64 + lane] = o[db][b2][i];
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        park[(64 + b2) * 64 + lane] = m_ref[b2];
        park[(66 + b2) * 64 + lane] = l_run[b2];
      }
    }
    volatile int* flag = reinterpret_cast<volatile int*>(smem);  // workgroup-wide OR of `bad`
    if (tid == 0) *flag = 0;
    __syncthreads();
    bool bad = false;
    float lt[2], mt[2];
    if (kh == 0) {
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        const float l1 = park[(66 + b2) * 64 + lane];
        float a0 = 1.f, a1 = 1.f;
        mt[b2] = 0.f;
        if constexpr (SAFE) {
          const float m1 = park[(64 + b2) * 64 + lane];
          const float m0 = m_ref[b2];
          mt[b2] = fmaxf(m0, m1);
          const float mu = (mt[b2] == -INFINITY) ? 0.f : mt[b2];
          a0 = exp2f(m0 - mu);  // exp2f(-inf) = 0 for a half that saw nothing
          a1 = exp2f(m1 - mu);
        }
        float l = l_run[b2] * a0 + l1 * a1;
        l += xor32(l);
        lt[b2] = l;
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            o[db][b2][i] = o[db][b2][i] * a0 + park[((db * 2 + b2) * 16 + i) * 64 + lane] * a1;
            if constexpr (!SAFE && !STREAM && !ONE) bad = bad || !(fabsf(o[db][b2][i]) < INFINITY);
          }
        if constexpr (!SAFE && !STREAM && !ONE) bad = bad || !(l >= 0x1p-80f && l <= 0x1p100f);
      }
    }
    if constexpr (ONE) {  // the states of the two halves of the list, like those of the two halves of a tile
      float* const mid = reinterpret_cast<float*>(smem) + 16;
      __syncthreads();
      if (kh == 0 && qi == 1) {
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2) {
#pragma unroll
          for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) mid[((db * 2 + b2) * 16 + i) * 64 + lane] = o[db][b2][i];
          mid[(64 + b2) * 64 + lane] = mt[b2];
          mid[(66 + b2) * 64 + lane] = lt[b2];
        }
      }
      __syncthreads();
      if (kh == 0 && qi == 0) {
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2) {
          float a0 = 1.f, a1 = 1.f;
          if constexpr (SAFE) {
            const float m0 = mt[b2], m1 = mid[(64 + b2) * 64 + lane];
            mt[b2] = fmaxf(m0, m1);
            const float mu = (mt[b2] == -INFINITY) ? 0.f : mt[b2];
            a0 = exp2f(m0 - mu);
            a1 = exp2f(m1 - mu);
          }
          lt[b2] = lt[b2] * a0 + mid[(66 + b2) * 64 + lane] * a1;
#pragma unroll
          for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              o[db][b2][i] = o[db][b2][i] * a0 + mid[((db * 2 + b2) * 16 + i) * 64 + lane] * a1;
        }
      }
    }
    const bool writes = kh == 0 && !(ONE && qi != 0);  // this wave holds the finished rows
    if constexpr (STREAM && !SAFE) {
      if (w1 > w0) {  // uniform: a row of several workgroups
        float* const partials = reinterpret_cast<float*>(tab + 1);
        // a workgroup has at most two parts of rows: the end of one and the start of another
        // per 64 query rows: accumulators four to a lane, [16][64 lanes][4], then the row sums [2][64 lanes]
        auto slot = [&](int w) { return partial_rsrc(partials + ((2 * int64_t(w) + (w == w0)) * WQ + qi) * kStreamPartialWords); };
        if (kh == 0) {
          const auto dst = slot(me);
#pragma unroll
          for (int b2 = 0; b2 < 2; ++b2) {
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
              for (int r4 = 0; r4 < 4; ++r4) {
                const f32x16& x = o[db][b2];
                const f32x4 y = {x[4 * r4], x[4 * r4 + 1], x[4 * r4 + 2], x[4 * r4 + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, y), dst, lane * 16,
                                                       ((db * 2 + b2) * 4 + r4) * 1024, kDeviceScope);
              }
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(lt[b2]), dst, lane * 4, 16384 + b2 * 256, kDeviceScope);
          }
        }
        __builtin_amdgcn_s_waitcnt(0);  // this part has arrived where every XCD sees it ...
        __syncthreads();                // ... before it is counted
        if (tid == 0) *flag = atomicAdd(&tab->arrived[row], 1);
        __syncthreads();
        const int before = __builtin_amdgcn_readfirstlane(*flag);
        __syncthreads();
        if (before != w1 - w0) return false;  // somebody is still at it
        if (tid == 0) *flag = 0;
        if (kh == 0) {
#pragma unroll
          for (int b2 = 0; b2 < 2; ++b2) {
            lt[b2] = 0.f;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
              for (int i = 0; i < 16; ++i) o[db][b2][i] = 0.f;
          }
          for (int w = w0; w <= w1; ++w) {
            const auto src = slot(w);
            f32x4 y[2][2][4];
            float ly[2];
#pragma unroll
            for (int b2 = 0; b2 < 2; ++b2) {
#pragma unroll
              for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4)
                  y[db][b2][r4] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                                src, lane * 16, ((db * 2 + b2) * 4 + r4) * 1024, kDeviceScope));
              ly[b2] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(src, lane * 4, 16384 + b2 * 256, kDeviceScope));
            }
            __builtin_amdgcn_sched_barrier(0);  // all of them in flight before the first is added
#pragma unroll
            for (int b2 = 0; b2 < 2; ++b2) {
#pragma unroll
              for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][b2][i] += y[db][b2][i >> 2][i & 3];
              lt[b2] += ly[b2];
            }
          }
        }
        __syncthreads();  // the cleared flag
      }
    }
    if constexpr (!SAFE) {
      if ((STREAM || ONE) && writes) {  // otherwise checked as it was merged
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2) {
          bad = bad || !(lt[b2] >= 0x1p-80f && lt[b2] <= 0x1p100f);
#pragma unroll
          for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) bad = bad || !(fabsf(o[db][b2][i]) < INFINITY);
        }
      }
      if (count_row <= 0) bad = false;  // an empty row is zeros by definition, not a range problem
      if (bad) *flag = 1;
      __syncthreads();
      const bool any_bad = *flag != 0;
      __syncthreads();
      if (any_bad) return true;
    }
    if (writes) {
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        const float inv = lt[b2] > 0.f ? 1.f / lt[b2] : 0.f;
        const int lrow = q_off + b2 * 32 + n;
        const int64_t row = int64_t(q_start) + lrow;
        if (lrow < q_valid) {
#pragma unroll
          for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
              const f32x16& x = o[db][b2];
              const int i = 4 * r4;
              const u32x2 w = {pack_bf16(x[i] * inv, x[i + 1] * inv), pack_bf16(x[i + 2] * inv, x[i + 3] * inv)};
              *reinterpret_cast<u32x2*>(out + (int64_t(h) * n_tokens + row) * kD + db * 32 + 8 * r4 + 4 * g) = w;
            }
          if (lse != nullptr && g == 0)
            lse[int64_t(h) * n_tokens + row] = lt[b2] > 0.f ? (mt[b2] + log2f(lt[b2])) * kLn2 : -INFINITY;
        }
      }
    }
    return false;
  };

  if (pass(std::false_type{})) {
    if constexpr (STREAM) take_tiles(0, 1 << 30);  // the whole row, whoever had its parts
    pass(std::true_type{});
  }
  return kDone;
  };  // run

  if constexpr (STREAM) {
    // consecutive pieces to one XCD (workgroup w runs on XCD w % 8), as for whole rows below
    constexpr int places = kStreamPlaces<B>;
    const int w = static_cast<int>(blockIdx.x);
    const int rows = heads * nb;
    const int me = (w & 7) * (places >> 3) + ((w & (places - 1)) >> 3);
    const int quota = __builtin_amdgcn_readfirstlane(tab->quota), used = __builtin_amdgcn_readfirstlane(tab->used);
    int row = __builtin_amdgcn_readfirstlane(tab->start_row[me]);
    int tile = __builtin_amdgcn_readfirstlane(tab->start_tile[me]);
    int done = 0, most = quota;
    if (quota == 0) {
      row = (w | 511) < rows ? (w & ~511) + (w & 7) * 64 + ((w & 511) >> 3) : w;
      tile = 0;
      most = 1;
    } else if (w >= places || me >= used) {
      return;  // the whole workgroup, before any barrier
    }
    while (done < most && row < rows) {
      int take = 1 << 30, w0 = 0, w1 = 0;
      if (quota != 0) {
        const int cnt = kv_cnt != nullptr ? min(max(kv_cnt[row], 0), nbk) : nbk;
        const int tiles = __builtin_amdgcn_readfirstlane(max(1, HALF ? (cnt + 1) >> 1 : cnt));
        take = min(quota - done, tiles - tile);
        const int begin = me * quota + done - tile;  // the row's first tile, counted over all rows
        w0 = begin / quota;
        w1 = (begin + tiles - 1) / quota;
      }
      run(std::false_type{}, row, tile, tile + take, w0, w1, me, -1, false);
      done += take;
      tile = 0;
      ++row;
      __syncthreads();  // the next row's loads overwrite what the end of this one reads
    }
    return;
  }
  // Which (head, query block) row this workgroup computes.  Workgroup number w of the grid runs on
  // XCD w % 8, whatever the XCDs' speeds, and the chip holds 512 workgroups at a time, 64 per XCD.
  //  - The first n_static workgroups take positions of the launch order by their number.  Inside each
  //    full group of 512 consecutive workgroups the positions are dealt out so that an XCD gets 64
  //    consecutive ones: rows that are neighbours in the order, whose lists tend to overlap, then
  //    share one L2 instead of being spread over all eight.
  //  - The other workgroups (there are more of them than rows left) take the remaining positions
  //    first come, first served, through one atomic counter, and leave at once when none is left.
  //    Under load the XCDs of a part run at clocks that differ by several per cent; an XCD that is
  //    through with its static share early thus takes more of the remaining rows than a slow one.
  const int units = PAIR || DUO ? (nb + 1) >> 1 : nb;  // workgroups' worth of rows per head
  const int64_t total = int64_t(heads) * units;
  const int64_t w = int64_t(blockIdx.y) * units + blockIdx.x;
  int64_t pos;
  if (w < n_static) {
    constexpr int PLACES = DUO ? 256 : 512;  // workgroups that the chip holds
    const int r = static_cast<int>(w & (PLACES - 1));
    pos = (w - r) + PLACES <= n_static ? (w - r) + (r & 7) * (PLACES / 8) + (r >> 3) : w;
  } else {
    if (next_row == nullptr) return;  // the grid is rounded up to whole heads
    int* slot = reinterpret_cast<int*>(smem);
    if (tid0 == 0) *slot = atomicAdd(next_row, 1);
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(*slot);
    __syncthreads();  // the slot lies where the first K tile goes
    if (t >= (PAIR ? 2 * total - n_pairs : total) - n_static) return;  // the whole workgroup leaves, before any other barrier
    pos = n_static + t;
  }
  int64_t row = order != nullptr ? int64_t(__builtin_amdgcn_readfirstlane(order[pos])) : pos;
  if constexpr (PAIR || DUO) {
    int which = -1;
    if constexpr (PAIR) row = pair_of(row, n_pairs, which);
    const int64_t h = min(max(row / units, int64_t(0)), int64_t(heads - 1));
    const int I = 2 * static_cast<int>(min(max(row - h * units, int64_t(0)), int64_t(units - 1)));
    const int first = which < 0 ? I : I + which, last = min(which < 0 ? I + 2 : first + 1, nb);
    if (first >= nb) return;
    if constexpr (DUO) {
      for (int next = -1;;) {  // -1: the pair
        const bool deal = next >= 0;
        const int left = run(std::false_type{}, deal ? h * nb + next : row, 0, 0, 0, 0, 0, -1, deal);
        if (!deal && left == kDone) return;
        next = deal ? next + 1 : first;
        if (next >= last) return;
        __syncthreads();  // whatever the end of the row before still reads
      }
    }
    const int listed = run(std::false_type{}, row, 0, 0, 0, 0, 0, which, false);
    if (listed == kDone) return;
#pragma unroll 1
    for (int i = first; i < last; ++i) {
      __syncthreads();  // whatever the end of the row before still reads
      run(std::true_type{}, h * nb + i, 0, 0, 0, 0, 0, listed, false);
    }
  } else {
    run(std::false_type{}, row, 0, 0, 0, 0, 0, -1, false);
  }
}

}  // namespace

int launch_attn_bf16(const void* q, const void* k, const void* v, int heads, int64_t n_tokens, int64_t n_first,
                     int block, int block_k, float softmax_scale, const int32_t* kv_idx, const int32_t* kv_cnt,
                     int idx_stride, void* out, float* lse, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  const int nb = static_cast<int>(split_blocks(n_tokens, n_first, block));     // query blocks
  const int nbk = static_cast<int>(split_blocks(n_tokens, n_first, block_k));  // key blocks the lists refer to
  const Segments seg = {static_cast<int>(n_first), static_cast<int>(ceil_div(n_first, block)),
                        static_cast<int>(ceil_div(n_first, block_k))};
  const int32_t* order = nullptr;
  const int32_t* choice = nullptr;
  const size_t order_bytes = attn_order_bytes(heads, n_tokens);
  const bool duo = block == 128 && kv_idx == nullptr && dense_pairs(heads, nb);  // every row is the same: no need to choose
  // few long rows, shared between workgroups (a launch of 1024 rows or more is never one of these)
  const bool share = !(duo && int64_t(heads) * nb > 512) && workspace != nullptr && attn_stream_shape(heads, n_tokens) &&
                     shares_rows(int64_t(heads) * nb, block, ceil_div(nbk, block / block_k), kv_idx == nullptr) &&
                     workspace_bytes >= order_bytes + kStreamBytes + 256;
  const bool choose = block == 128 && kv_idx != nullptr && workspace != nullptr && chooses_pairs(heads, nb, nbk);
  const bool pair = pairs_rows(block, heads, nb, nbk) || (duo && !share);

  // How the units (rows, or pairs of rows) of a kernel go to its workgroups; see the end of the kernel.
  struct Spread {
    dim3 grid;
    int64_t n_static;  // units taken by workgroup number
    int64_t n_pairs;   // units that are pairs, see pair_of
    int singly;        // pairs after them that go row by row
    bool big;          // the other units are handed out at run time
  };
  auto spread = [&](bool two, bool eight_waves) {
    const int nu = two ? (nb + 1) >> 1 : nb;
    const int64_t rows = int64_t(heads) * nu;
    // Pairs of blocks of 64: the last `singly` ones go row by row.  How many depends on the shape alone, not on the lists nor on whether
    // there is a launch order, for a row that is taken by itself is summed in another order than one that is taken in a pair.
    int64_t singly = 0;
    if (two && !eight_waves && heads + ceil_div(128, nu) <= 65535) {
      const int64_t rest = rows - 512;
      // The chip holds 512 workgroups.  Up to 128 pairs that are left after the first 512 go row by row, a CU to each:
      // 1,064 rows of 532 blocks, nine tenths, a quarter kept, a band: 655 -> 610, 252 -> 204, 216 -> 179 us.  Where more
      // are left the last 64 do, which evens out the end: 1,600 rows of 100 blocks 176 -> 164, 69 -> 61, 62 -> 60 us.  With
      // 400 and more there is no room for them: 1,840 rows of 115 205 -> 207 us, 2,032 of 127 242 -> 261.
      if (rows < 1024) singly = rest <= 128 ? rest : rest < 400 ? 64 : 0;
      // Of larger launches up to half as many pairs as CUs that are left over after whole rounds of one per CU, so that a CU has half
      // a pair more to do than another and not a whole one; with more left over there is a pair for most CUs anyway.  In the launch order they
      // are units like the others.  us, in pairs only / so, nine tenths kept (half, a quarter, a tenth, lengths uniform): 1,040 pairs 283 / 269
      // (202 / 182, 127 / 111, 71 / 65, 229 / 222), 1,152, of which 128 are left over, 322 / 318 (228 / 214, 146 / 133, 79 / 76, 269 / 254), 1,376
      // 444 / 436 (307 / 285, 188 / 180, 98 / 93, 361 / 349), 1,552 562 / 544 (384 / 366, 230 / 221, 114 / 112, 446 / 436).
      else if (rows % 256 <= 128 && rows + rows % 256 <= kOrderOneMax) singly = rows % 256;
    }
    const int64_t n_pairs = rows - singly, items = rows + singly;
    int64_t n_static = items;  // without a workspace every unit is taken by workgroup number
    int64_t extra = singly;    // workgroups beyond one per row or pair
    // ordering and balancing matter only when the grid does not fit the chip at once
    // (and only while the extra workgroups fit the grid's second dimension)
    const bool big = workspace != nullptr && rows >= 1024 && rows < (int64_t(1) << 30) &&
                     heads + ceil_div(rows / 16 + 1024, nu) <= 65535;
    if (big) {
      // The last eighth of the rows is handed out at run time; half as many workgroups again as that
      // are launched for it, so that an XCD can take up to 1.5 times its even share of those rows.
      const int64_t dynamic = rows / 8;
      n_static = (rows - dynamic) / 512 * 512;
      extra = singly + (rows - n_static) / 2 + 512;
    }
    return Spread{dim3(nu, heads + static_cast<int>(ceil_div(extra, nu))), n_static, n_pairs, static_cast<int>(singly), big};
  };
  const Spread plan = spread(pair, block == 128);
  int* next_row = nullptr;
  if (plan.big && kv_idx == nullptr) {
    // dense: the workspace holds the counter only
    next_row = static_cast<int*>(workspace);
    hipLaunchKernelGGL(zero_word_kernel, dim3(1), dim3(64), 0, stream, next_row);
  }
  if (plan.big && kv_idx != nullptr) {
    // workspace: launch order of the units, then the [classes][heads] table, the number of the merged
    // class, the counter of the rows handed out at run time (cleared by order_one_kernel or order_merge_kernel) and, where
    // pairs are thought of, the choice and the pairs' table (there is room: it is sized for blocks of 64, and has nb - 2 words a head left)
    const int nu = static_cast<int>(plan.grid.x);
    const int64_t rows = int64_t(heads) * nu;
    int32_t* ord = static_cast<int32_t*>(workspace);
    int32_t* table = ord + rows + plan.singly;
    next_row = table + int64_t(kOrderClasses) * heads + 1;
    const int per_tile = block_k == block ? 1 : 2;
    int32_t* const chosen = choose ? table + int64_t(kOrderClasses) * heads + 2 : nullptr;
    choice = chosen;
    if (rows <= kOrderOneMax) {
      hipLaunchKernelGGL(order_one_kernel, dim3(1), dim3(1024), 0, stream, kv_cnt, nb, nu, pair, nbk, heads, plan.singly, per_tile,
                         chosen, ord, next_row);
    } else {
      int32_t* const pairs = choose ? chosen + 1 : nullptr;
      hipLaunchKernelGGL(order_hist_kernel, dim3(heads), dim3(256), 0, stream, kv_cnt, nb, nu, pair, nbk, heads, table, pairs);
      hipLaunchKernelGGL(order_merge_kernel, dim3(1), dim3(256), 0, stream, table, heads, pairs, nb, nbk, per_tile);
      hipLaunchKernelGGL(order_scan_kernel, dim3(1), dim3(1024), 0, stream, table, int64_t(kOrderClasses) * heads);
      hipLaunchKernelGGL(order_place_kernel, dim3(heads), dim3(256), 0, stream, kv_cnt, nb, nu, pair, nbk, heads, choice, table, ord);
    }
    if (int rc = check_hip(hipGetLastError(), "bsga bf16 attention (launch order)")) return rc;
    order = ord;
  }
  const float scale_log2 = softmax_scale * kLog2e;
  if (!share && !pair && few_rows(block, int64_t(heads) * nb))
    return launch_attn_few(q, k, v, heads, n_tokens, n_first, scale_log2, kv_idx, kv_cnt, idx_stride, out, lse, stream);
  const unsigned char* qp = static_cast<const unsigned char*>(q);
  const unsigned char* kp = static_cast<const unsigned char*>(k);
  const unsigned char* vp = static_cast<const unsigned char*>(v);
  unsigned short* op = static_cast<unsigned short*>(out);
  // LDS: two K and two V tile buffers (64 KB for block 128); block 64 also needs room for the
  // parked accumulators of the end merge (17 KB + 64 B), which 32 KB covers
  const size_t lds64 = 4 * 64 * 128, lds128 = 4 * 128 * 128;
  if (getenv("BSGA_DEBUG") != nullptr) {
    int n64 = -1, n128 = -1;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&n64, attn_bf16_kernel<64, 64, false, false, false>, 128, lds64);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&n128, attn_bf16_kernel<128, 128, false, false, false>, 256, lds128);
    fprintf(stderr, "[bsga] attention occupancy (workgroups per CU): block 64 -> %d, block 128 -> %d\n", n64, n128);
  }
  auto launch = [&](auto kernel, const Spread& to, int threads, size_t lds, StreamTable* tab) {
    hipLaunchKernelGGL(kernel, to.grid, dim3(threads), lds, stream, qp, kp, vp, op, lse, kv_idx, kv_cnt, order, idx_stride,
                       n_tokens, nb, nbk, scale_log2, seg, heads, to.n_static, to.n_pairs, next_row, choice, tab);
  };
  if (share) {
    const uintptr_t at = reinterpret_cast<uintptr_t>(workspace) + order_bytes;
    StreamTable* tab = reinterpret_cast<StreamTable*>((at + 255) & ~uintptr_t(255));
    const int places = block == 64 ? kStreamPlaces<64> : kStreamPlaces<128>;
    const Spread all = {dim3(max(places, heads * nb)), 0, 0, 0, false};
    hipLaunchKernelGGL(stream_plan_kernel, dim3(1), dim3(kStreamMaxRows), 0, stream, kv_cnt, heads * nb, nbk,
                       block_k == block ? 1 : 2, places, block == 64 || kv_idx == nullptr, tab);
    if (int rc = check_hip(hipGetLastError(), "bsga bf16 attention (plan)")) return rc;
    if (block == 64) launch(attn_bf16_kernel<64, 64, true, false, false>, all, 128, lds64, tab);
    else if (block_k == 128) launch(attn_bf16_kernel<128, 128, true, false, false>, all, 256, lds128, tab);
    else launch(attn_bf16_kernel<128, 64, true, false, false>, all, 256, lds128, tab);
    return check_hip(hipGetLastError(), "bsga bf16 attention launch");
  }
  if (duo || choice != nullptr) {
    const Spread pairs = spread(true, true);
    const size_t lds = 2 * lds128 + (kv_idx != nullptr ? 4 * size_t(nbk) : 0);
    if (block_k == 128) launch(attn_bf16_kernel<128, 128, false, false, true>, pairs, 512, lds, nullptr);
    else launch(attn_bf16_kernel<128, 64, false, false, true>, pairs, 512, lds, nullptr);
    if (int rc = check_hip(hipGetLastError(), "bsga bf16 attention launch")) return rc;
    if (duo) return BSGA_OK;
  }
  if (pair) launch(attn_bf16_kernel<128, 64, false, true, false>, plan, 256, lds128 + 4 * size_t(nbk), nullptr);
  else if (block == 64) launch(attn_bf16_kernel<64, 64, false, false, false>, plan, 128, lds64, nullptr);
  else if (block_k == 128) launch(attn_bf16_kernel<128, 128, false, false, false>, plan, 256, lds128, nullptr);
  else launch(attn_bf16_kernel<128, 64, false, false, false>, plan, 256, lds128, nullptr);
  return check_hip(hipGetLastError(), "bsga bf16 attention launch");
}

}  // namespace bsga
