// fp32 attention over kept key blocks (Sec. 4.1, Eq. (2); Eq. (1) when no index list is given), online softmax in fp32.
// Two kernels: attn_fp32_split_kernel for launches of more than 128 units of 64 query rows, attn_fp32_kernel for the rest.
//
// attn_fp32_split_kernel: both products on the bf16 matrix instructions, every fp32 operand split in three.
//   x = x1 + x2 + x3, eight bits each, and nothing is left over (almost: see kCutOff).  Of the nine products of two such sums
//   the six of the order of 2^-18 and above are taken (11, 12, 21, 22, 13, 31), the small ones first, accumulated in fp32.
//   A bf16 product is exact in fp32 and 16 of them are summed per instruction, so a sum has fewer roundings than
//   on v_mfma_f32_32x32x2; the output products of a tile are summed apart and added to the output with one more.  Error of the output
//   against float64 (2-norms): 2,748 tokens of a scene 2.0e-7, on the fp32 instructions 4.7e-7; 5,496 2.5e-7 and 6.5e-7; logits
//   a hundred times as large 3.1e-6 and 4.4e-6; the row sums' logarithm as before.
//   Six instructions of 32 cycles stand for eight of 64: 1,540 cycles of matrix products per tile and wave.  What bounds the kernel is
//   the chain of steps that a tile is for a wave (about 5,000 cycles alone), so what counts is how many workgroups a CU holds.
//   A workgroup of four waves owns 64 query rows of one block; wave (qi, kh) takes 32 of them and 32 keys of every
//   tile of 64, and the two key halves have softmax states of their own, merged at the end.
//   PRE: split_kv_kernel has left the parts of K and V in the call's workspace, and tiles go from there straight to the LDS (48 KB),
//   K under the output products of the tile before, V under the scores of its own.  No tile passes through registers, which leaves
//   room for three workgroups to a CU: 5,496 tokens 794 -> 664 us, 2,748 221 -> 178 (both with the split), 50 % of the
//   matrix pipe before.  With two workgroups and the parts through registers 774 and 219.
//   Otherwise the four waves load a tile, split it together and leave the parts in the LDS, two workgroups to a CU.  Two accumulators in
//   turn keep the matrix pipe from waiting for itself: 827 -> 802 us (with three workgroups there is no room for that in the output
//   products, and no need).  Rows are 128 bytes, chunks of 16 bytes permuted as in the bf16 kernel, whose operand
//   layouts these are: S^T = K Q^T leaves the weights where they are the B operand of O^T = V^T P^T, and V^T comes by
//   transposing LDS reads.
//   Values the split cannot hold (infinities, NaN, very small ones, see below) make a row sum or an output something else
//   than a finite number.  The unit then starts over on fp32 instructions (unit_fp32).  16 heads of 2,748 tokens, dense, with the workspace /
//   without, 181 / 224 us: one NaN in a head 300 / 369, NaN in every tile 338 / 367, an infinity in the last token of each head, which is met
//   at the end, 478 / 548, all values of 1e-36 344 / 368.  On the fp32 instructions throughout 290.
//   16 heads, dense, 32 rows or 64 on the fp32 instructions / so: 700 tokens 33 / 28 us, 1,374 109 / 70, 2,748 288 / 219, 5,496
//   1,074 / 664 (186 TFLOP/s; a library fp32 GEMM reaches 154).
//   Measured and not taken: the next tile's split and the weights interleaved with the products in one wave (820 us: what
//   one wave can issue in a row then bounds it); three workgroups to a CU that split for themselves (168 registers spill: 868).
//
// attn_fp32_kernel: both products on v_mfma_f32_32x32x2.  A workgroup of four waves owns 32 query rows; its waves take the
//   32-key pieces of the row's key blocks in turn, each with a softmax state of its own, merged through LDS at the end.  Twice
//   as many workgroups, and four times the waves to a key: a head of 1,374 tokens 33 us, split 51; two of 2,748 65 and 96.
//   A piece of 32 keys is 64 MFMAs of 64 cycles per wave.  K and V come straight from global memory into operand registers, without LDS or
//   barriers: V of a piece is loaded under its score products, K of the next one under its output products.
//   S^T = K Q^T: lane (n = lane%32, g = lane/32) holds dims 8c + 4g .. +3, c = 0..7, of key n as A operand and
//   of query n as B operand (the contraction takes the dims in that order); accumulator register i of the lane
//   is key 8(i/4) + 4g + i%4 of query n.
//   O^T += V^T P^T: step i multiplies keys 8(i/4) + 4g + i%4, so the weights are used where they are; the lane
//   supplies dims 2n and 2n + 1 of that key, one for each of the two accumulators.
//
// In both, consecutive units run on one XCD (workgroup w runs on XCD w % 8), so that an L2 holds the keys of two heads and
// not of all of them.
#include <type_traits>

#include "bf16_tile.h"
#include "bsga_internal.h"

namespace bsga {
namespace {

constexpr int kD = 64;
constexpr int kTile = 64;                       // keys
constexpr int kPiece = 32;                      // keys a wave takes at a time on the fp32 instructions
constexpr int kPlane = kTile * kD * 2;          // one of the three parts of a K or V tile, bytes
constexpr int kRowWords = 18 * 64;              // what a wave leaves for its neighbour: 16 accumulators, maximum, sum of 64 lanes

// the three parts of a and b, packed in pairs.  The first is rounded to nearest, so that the rest has either sign; the others
// are cut off, which is a byte permutation instead of a conversion of twice the time.  `left`: what the third parts are cut from, ORed.
__device__ __forceinline__ void split_pair(float a, float b, unsigned& p1, unsigned& p2, unsigned& p3, unsigned& left) {
  p1 = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
  a -= __uint_as_float(p1 << 16);
  b -= __uint_as_float(p1 & 0xffff0000u);
  p2 = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
  a -= __uint_as_float(__float_as_uint(a) & 0xffff0000u);
  b -= __uint_as_float(__float_as_uint(b) & 0xffff0000u);
  p3 = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
  left |= __float_as_uint(a) | __float_as_uint(b);
}

// the three parts of eight values; returns `left` of all of them
__device__ __forceinline__ unsigned split_chunk(f32x4 x0, f32x4 x1, u32x4 (&y)[3]) {
  unsigned left = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    unsigned p1, p2, p3;
    split_pair(e < 2 ? x0[2 * e] : x1[2 * e - 4], e < 2 ? x0[2 * e + 1] : x1[2 * e - 3], p1, p2, p3, left);
    y[0][e] = p1;
    y[1][e] = p2;
    y[2][e] = p3;
  }
  return left;
}

// Three times eight bits are a whole fp32 number, down to about 2^-110: bf16 ends 16 bits above fp32 (the matrix
// instructions keep subnormal numbers of both), and what is cut off there, up to 2^-133, is 1e-4 of 2^-120.
//  - A value counts to its own size.  One that the parts do not hold whole is reported by the unit that splits it, or written as a NaN
//    beforehand, and so come the outputs of all who list its key.
//  - Keys and queries count by what they do to a logit, which is nothing (64 products of 2^96 and 2^-133) as long as the key is whole
//    or the query below 2^96, and the other way round.  It is queries that are looked at: those below 2^-110 or from 2^96 on become NaN.
//  - A weight of less than 2^-110 of its row's largest is off by up to 2^-133 of that one.  Nothing is done about it.
// The unit then starts over on fp32 instructions, see unit_fp32.
constexpr unsigned kCutOff = 0xffffu;  // bits of `left` that the third parts have no room for
__device__ __forceinline__ void mark(u32x4 (&y)[3]) { y[2][0] |= 0x7fffu; }

// c + x y of two split operands, the small products first
__device__ __forceinline__ f32x16 products(const bf16x8 (&x)[3], const bf16x8 (&y)[3], f32x16 c) {
  constexpr int X[6] = {2, 0, 1, 1, 0, 0}, Y[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int i = 0; i < 6; ++i) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[X[i]], y[Y[i]], c, 0, 0, 0);
  return c;
}

// the same; two such sums in turn, since an instruction that waits for the one before
// it leaves the matrix pipe idle
__device__ __forceinline__ void products(const bf16x8 (&x0)[3], const bf16x8 (&y0)[3], f32x16& c0, const bf16x8 (&x1)[3],
                                         const bf16x8 (&y1)[3], f32x16& c1) {
  constexpr int X[6] = {2, 0, 1, 1, 0, 0}, Y[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x0[X[i]], y0[Y[i]], c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x1[X[i]], y1[Y[i]], c1, 0, 0, 0);
  }
}

// K and V split beforehand: token t of head h has kPartRow bytes at (h n_tokens + t) kPartRow, the three parts of its key, then
// those of its value.  A thread splits eight dims of one of the two.
static_assert(kPartRow == 6 * kD * 2, "three parts of a key and of a value");
__global__ __launch_bounds__(256) void split_kv_kernel(const float* __restrict__ k, const float* __restrict__ v, int64_t chunks,
                                                       unsigned char* __restrict__ parts) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (t >= chunks) return;
  const float* const src = (blockIdx.y ? v : k) + t * 8;
  const f32x4 x0 = *reinterpret_cast<const f32x4*>(src), x1 = *reinterpret_cast<const f32x4*>(src + 4);
  u32x4 y[3];
  if ((split_chunk(x0, x1, y) & kCutOff) != 0u && blockIdx.y) mark(y);
  unsigned char* const dst = parts + (t >> 3) * kPartRow + blockIdx.y * 3 * 128 + (t & 7) * 16;
#pragma unroll
  for (int x = 0; x < 3; ++x) *reinterpret_cast<u32x4*>(dst + x * 128) = y[x];
}

// What a workgroup of attn_fp32_split_kernel works on: 64 rows of a query block and the key blocks of its list.
template <int B>
struct Unit {
  int64_t n_tokens, n_first, head_off, row0;
  const int32_t* list;  // null: all blocks
  int nb1, nb, h, rows, count;
  // blocks 0 .. nb1-1 tile tokens [0, n_first), the others tokens [n_first, n_tokens)
  __device__ __forceinline__ int64_t block_start(int J) const { return J < nb1 ? int64_t(J) * B : n_first + int64_t(J - nb1) * B; }
  __device__ __forceinline__ int block_count(int J) const {
    return static_cast<int>(min<int64_t>(B, (J < nb1 ? n_first : n_tokens) - block_start(J)));
  }
  static constexpr int PIECES = B / kTile;  // tiles per key block
  __device__ __forceinline__ int pieces() const { return count * PIECES; }
  // the first tile from `piece` on that holds a key at all: a short block may end before its later tiles
  __device__ __forceinline__ int next_piece(int piece, int64_t& key0, int& valid) const {
    for (; piece < pieces(); ++piece) {
      const int it = piece / PIECES;
      // through the scalar cache: a vector load's wait would be for the tiles on their way too
      const int J = list == nullptr ? it : min(max(((const int32_t __attribute__((address_space(4)))*)list)[it], 0), nb - 1);
      key0 = block_start(J) + (piece % PIECES) * kTile;
      valid = block_count(J) - (piece % PIECES) * kTile;
      if (valid > 0) break;
    }
    return piece;
  }
};

// State of a wave's softmax over 32 rows: O^T: [dim block], the lane's query
struct Softmax {
  f32x16 o[2];
  float m, l;
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < 16; ++i) o[0][i] = o[1][i] = 0.f;
    m = -INFINITY;
    l = 0.f;
  }
  // scores of 32 keys, of which those from `valid` on do not count -> weights; maximum and sum follow.  Returns what the
  // output so far is to be multiplied by.
  __device__ __forceinline__ float weigh(f32x16& s, int valid, int g) {
    if (valid < 32) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = (8 * (i >> 2) + 4 * g + (i & 3) >= valid) ? -INFINITY : s[i];
    }
    float top = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) top = fmaxf(top, s[i]);
    top = fmaxf(top, __shfl_xor(top, 32));
    float a = 1.f;
    if (__any(top > m)) {
      const float m_new = fmaxf(m, top);
      a = m == m_new ? 1.f : __builtin_amdgcn_exp2f(m - m_new);  // 0 on the first tile
      m = m_new;
    }
    const float ref = m == -INFINITY ? 0.f : m;  // a wave that has seen nothing but weights of zero (scores of -inf) has no maximum
    float part[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = __builtin_amdgcn_exp2f(s[i] - ref);
      part[i & 1] += s[i];
    }
    l = fmaf(l, a, part[0] + part[1]);
    return a;
  }
  // The end of a pass: wave (qi, kh) finishes dims 32 kh .. 32 kh + 31 of its 32 rows, with what wave (qi, 1 - kh) leaves.  `bad` (or
  // null): set, and nothing is stored, if a sum or an output is no finite number.  Returns whether it is set, to every thread.
  template <int B>
  __device__ __forceinline__ bool finish(const Unit<B>& un, int wave, int lane, float* park, int* bad, float* out, float* lse) const {
    const int qi = wave & 1, kh = wave >> 1, n = lane & 31, g = lane >> 5;
#pragma unroll
    for (int i = 0; i < 16; ++i) park[wave * kRowWords + i * 64 + lane] = kh ? o[0][i] : o[1][i];
    park[wave * kRowWords + 16 * 64 + lane] = m;
    park[wave * kRowWords + 17 * 64 + lane] = l;
    __syncthreads();
    const float* other = park + (wave ^ 2) * kRowWords;
    const float m1 = other[16 * 64 + lane], top = fmaxf(m, m1);
    const float mu = top == -INFINITY ? 0.f : top;
    const float a0 = __builtin_amdgcn_exp2f(m - mu), a1 = __builtin_amdgcn_exp2f(m1 - mu);  // 0 for a wave that saw no key
    float sum = l * a0 + other[17 * 64 + lane] * a1;
    sum += __shfl_xor(sum, 32);
    f32x16 x;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = (kh ? o[1][i] : o[0][i]) * a0 + other[i * 64 + lane] * a1;
    if (bad != nullptr) {
      bool b = un.count > 0 && !(sum > 0.f && sum < INFINITY);
#pragma unroll
      for (int i = 0; i < 16; ++i) b = b || !(fabsf(x[i]) < INFINITY);
      if (b) *bad = 1;
      __syncthreads();
      if (*bad != 0) return true;
    }
    const int r = 32 * qi + n;
    if (r < un.rows) {
      // listed keys, but none with a weight: the softmax is 0 / 0
      const float inv = sum > 0.f ? 1.f / sum : un.count > 0 ? NAN : 0.f;
      float* dst = out + un.head_off + (un.row0 + r) * kD + 32 * kh + 4 * g;
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        *reinterpret_cast<f32x4*>(dst + 8 * r4) = f32x4{x[4 * r4] * inv, x[4 * r4 + 1] * inv, x[4 * r4 + 2] * inv, x[4 * r4 + 3] * inv};
      if (lse != nullptr && kh == 0 && g == 0)
        lse[int64_t(un.h) * un.n_tokens + un.row0 + r] = sum > 0.f ? (top + log2f(sum)) * 0.6931471805599453f : -INFINITY;
    }
    return false;
  }
};

// A unit in fp32 instructions, where it has numbers that the parts do not hold.  Tiles go through registers to the LDS, the next one on
// its way meanwhile; the chunks of Q and K are permuted.  Step d multiplies dims 8(d/4) + 4g + d%4, step i keys 8(i/4) + 4g + i%4 of the wave's.
template <int B>
__device__ __forceinline__ void unit_fp32(const Unit<B>& un, int wave, const float* __restrict__ q, const float* __restrict__ k,
                                          const float* __restrict__ v, float scale_log2, float* smem, float* out, float* lse) {
  const int lane = fresh_lane();  // so that nothing of this is kept in registers beside the split operands
  const int tid = wave * 64 + lane, qi = wave & 1, kh = wave >> 1, n = lane & 31, g = lane >> 5;
  float* const kt = smem;
  float* const vt = smem + kTile * kD;
  float* const qt = vt + kTile * kD;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (tid >> 4) + 16 * i, c = tid & 15;
    *reinterpret_cast<f32x4*>(qt + r * kD + ((c ^ (r & 15)) << 2)) =
        *reinterpret_cast<const f32x4*>(q + un.head_off + (un.row0 + min(r, un.rows - 1)) * kD + 4 * c) * scale_log2;
  }
  f32x4 raw[2][4];  // [K, V]: chunk (four dims) tid % 16 of tile rows tid / 16 + 16 i
  auto load = [&](int64_t key0, int valid) {  // keys past `valid` repeat the last one; they are masked, and their values are zeros
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (tid >> 4) + 16 * i;
      const int64_t at = un.head_off + (key0 + min(r, valid - 1)) * kD + 4 * (tid & 15);
      raw[0][i] = *reinterpret_cast<const f32x4*>(k + at);
      raw[1][i] = *reinterpret_cast<const f32x4*>(v + at);
      if (r >= valid) raw[1][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  Softmax st;
  st.clear();
  int64_t key0 = 0;
  int valid = 0;
  int piece = un.next_piece(0, key0, valid);
  if (piece < un.pieces()) load(key0, valid);
  while (piece < un.pieces()) {
    __syncthreads();  // whatever is still read
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (tid >> 4) + 16 * i, c = tid & 15;
      *reinterpret_cast<f32x4*>(kt + r * kD + ((c ^ (r & 15)) << 2)) = raw[0][i];
      *reinterpret_cast<f32x4*>(vt + r * kD + 4 * c) = raw[1][i];
    }
    __syncthreads();
    const int mine = valid - 32 * kh;  // keys of this wave
    piece = un.next_piece(piece + 1, key0, valid);
    if (piece < un.pieces()) load(key0, valid);
    if (mine <= 0) continue;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 s = zero;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int at = ((2 * c + g) ^ (n & 15)) << 2;
      const f32x4 x = *reinterpret_cast<const f32x4*>(kt + (32 * kh + n) * kD + at), y = *reinterpret_cast<const f32x4*>(qt + (32 * qi + n) * kD + at);
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], s, 0, 0, 0);
    }
    const float a = st.weigh(s, mine, g);
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      f32x16 t = zero;  // apart, as the split products are
#pragma unroll
      for (int i = 0; i < 16; ++i)
        t = __builtin_amdgcn_mfma_f32_32x32x2f32(vt[(32 * kh + 8 * (i >> 2) + 4 * g + (i & 3)) * kD + 32 * db + n], s[i], t, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i) st.o[db][i] = fmaf(st.o[db][i], a, t[i]);
    }
  }
  __syncthreads();
  st.finish(un, wave, lane, smem, nullptr, out, lse);
}

template <int B, bool PRE>
__global__ __launch_bounds__(256, PRE ? 3 : 2) void attn_fp32_split_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                           const float* __restrict__ v, const unsigned char* __restrict__ parts,
                                                           int64_t n_tokens, int64_t n_first,
                                                           int nb1, int nb, float scale_log2,
                                                           const int32_t* __restrict__ kv_idx,
                                                           const int32_t* __restrict__ kv_cnt, int idx_stride,
                                                           float* __restrict__ out, float* __restrict__ lse) {
  constexpr int UNITS = B / 64;  // workgroups per query block
  __shared__ __align__(16) unsigned char smem[6 * kPlane];  // K parts 1, 2, 3, V parts 1, 2, 3
  __shared__ int bad_s;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qi = wave & 1;
  const int kh = wave >> 1;
  const int n = lane & 31;
  const int g = lane >> 5;
  // unit of this workgroup: XCD x takes the x-th eighth of all units
  const int64_t total = int64_t(gridDim.x) * gridDim.y;
  const int64_t w = int64_t(blockIdx.y) * gridDim.x + blockIdx.x;
  const int64_t xcd = w & 7, per = total >> 3, rest = total & 7;
  const int64_t unit = xcd * per + min(xcd, rest) + (w >> 3);
  const int h = static_cast<int>(unit / gridDim.x);
  const int u = static_cast<int>(unit - int64_t(h) * gridDim.x);
  const int I = u / UNITS;
  const int64_t row = int64_t(h) * nb + I;
  Unit<B> un{n_tokens, n_first, int64_t(h) * n_tokens * kD, 0, kv_idx == nullptr ? nullptr : kv_idx + row * idx_stride, nb1, nb, h, 0, 0};
  un.rows = un.block_count(I) - (u % UNITS) * 64;  // query rows from this unit's first on
  if (un.rows <= 0) return;                        // the whole workgroup, before any barrier
  un.row0 = un.block_start(I) + (u % UNITS) * 64;
  un.count = kv_idx == nullptr ? nb : min(max(kv_cnt[row], 0), nb);
  const int pieces = un.pieces();
  const int64_t head_off = un.head_off;
  auto next_piece = [&](int piece, int64_t& key0, int& valid) { return un.next_piece(piece, key0, valid); };
  if (tid == 0) bad_s = 0;
  const float* const q_row = q + head_off + (un.row0 + min(32 * qi + n, un.rows - 1)) * kD;  // rows past the end are not stored
  Softmax st;
  st.clear();

  // ---- the products in split operands ---------------------------------------------------------------
  // returns true, to every thread, if a row sum or an output is not finite already
  auto tiles = [&]() -> bool {
    bf16x8 qf[4][3];  // [16-dim chunk][part]: dims 16c + 8g .. +7 of query n
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(q_row + 16 * c + 8 * g), x1 = *reinterpret_cast<const f32x4*>(q_row + 16 * c + 8 * g + 4);
      u32x4 y[3];
      split_chunk(x0 * scale_log2, x1 * scale_log2, y);
      float top = 0.f;
      unsigned low = ~0u;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = (e < 4 ? x0[e] : x1[e - 4]) * scale_log2;
        top = fmaxf(top, fabsf(x));
        low = min(low, 2u * __float_as_uint(x) - 1u);  // without its sign; a zero is the largest
      }
      if (top >= 0x1p96f || low < 2u * 0x08800000u - 1u) mark(y);  // 2^-110
#pragma unroll
      for (int x = 0; x < 3; ++x) qf[c][x] = __builtin_bit_cast(bf16x8, y[x]);
    }
    unsigned kaddr[4], vaddr[2];  // operand addresses in a part, see attn_bf16.hip
    {
      const int r = kh * 32 + n;
#pragma unroll
      for (int c = 0; c < 4; ++c) kaddr[c] = r * 128 + (((2 * c + g) ^ swz_k(r)) << 4);
      const int i16 = lane & 15, mm = i16 >> 2, j = i16 & 3, G = lane >> 4;
      const int key = kh * 32 + 4 * g + mm;
#pragma unroll
      for (int db = 0; db < 2; ++db)
        vaddr[db] = 3 * kPlane + key * 128 + (((db * 4 + 2 * (G & 1) + (j >> 1)) ^ swz_v(key)) << 4) + (j & 1) * 8;
    }
    bf16x8 pf[2][3];
    // scores and weights of the K tile in the LDS; returns what weigh() does
    auto scores = [&](int valid) -> float {
      f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, s2 = s;  // dims 0 .. 31 and 32 .. 63
      auto read_k = [&](int c, bf16x8 (&kf)[3]) {
#pragma unroll
        for (int x = 0; x < 3; ++x) kf[x] = *reinterpret_cast<const bf16x8*>(smem + x * kPlane + kaddr[c]);
      };
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bf16x8 kf[2][3];
        read_k(c, kf[0]);
        read_k(c + 2, kf[1]);
        products(kf[0], qf[c], s, kf[1], qf[c + 2], s2);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] += s2[i];
      const float a = st.weigh(s, valid - 32 * kh, g);
#pragma unroll
      for (int cp = 0; cp < 2; ++cp) {
        u32x4 y[3];
        split_chunk(f32x4{s[8 * cp], s[8 * cp + 1], s[8 * cp + 2], s[8 * cp + 3]}, f32x4{s[8 * cp + 4], s[8 * cp + 5], s[8 * cp + 6], s[8 * cp + 7]}, y);
#pragma unroll
        for (int x = 0; x < 3; ++x) pf[cp][x] = __builtin_bit_cast(bf16x8, y[x]);
      }
      return a;
    };
    // output products of the V tile.  Summed up apart and added with one fp32 rounding: the matrix instructions round a sum that has
    // grown large worse.
    auto outputs = [&](float a) {
      auto read_v = [&](int db, int cp, bf16x8 (&vf)[3]) {
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          const unsigned char* p = smem + x * kPlane + vaddr[db] + 16 * cp * 128;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + 8 * 128));
          const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
          vf[x] = __builtin_bit_cast(bf16x8, u32x4{lo2[0], lo2[1], hi2[0], hi2[1]});
        }
      };
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if constexpr (PRE) {  // one after the other: the registers are three workgroups'
#pragma unroll
        for (int db = 0; db < 2; ++db) {
          f32x16 t = zero;
#pragma unroll
          for (int cp = 0; cp < 2; ++cp) {
            bf16x8 vf[3];
            read_v(db, cp, vf);
            t = products(vf, pf[cp], t);
          }
#pragma unroll
          for (int i = 0; i < 16; ++i) st.o[db][i] = fmaf(st.o[db][i], a, t[i]);
        }
      } else {
        f32x16 t[2] = {zero, zero};
#pragma unroll
        for (int cp = 0; cp < 2; ++cp) {
          bf16x8 vf[2][3];
          read_v(0, cp, vf[0]);
          read_v(1, cp, vf[1]);
          products(vf[0], pf[cp], t[0], vf[1], pf[cp], t[1]);
        }
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) st.o[db][i] = fmaf(st.o[db][i], a, t[db][i]);
      }
    };
    // Whether a row sum or an output is not finite, which it then stays, or a number was not whole: looked at every eight tiles, before a
    // barrier, and known to all after it.
    unsigned left = 0;
    auto look = [&]() {
      float top = st.l;
#pragma unroll
      for (int i = 0; i < 16; ++i)  // three operands to an instruction, and NaN if one is
        top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(top, fabsf(st.o[0][i])), fabsf(st.o[1][i]));
      if (!(top < INFINITY) || (left & kCutOff) != 0u) bad_s = 1;
    };
    auto given_up = [&]() { return __builtin_amdgcn_readfirstlane(*const_cast<volatile int*>(&bad_s)) != 0; };
    int64_t key0 = 0;
    int valid = 0, done = 0;
    int piece = next_piece(0, key0, valid);
    if constexpr (PRE) {
      // Direct to the LDS: load i of a wave covers rows 8 j .. 8 j + 7, j = wave + 4 (i / 3), of part i % 3; lane -> row 8 j + lane / 8
      // and, at chunk position lane % 8, the chunk that belongs there.  Rows past the end of the head come as zeros, those past the end of
      // a key block are the tokens that follow: their weight is 0 (and where they are not finite, see Softmax::finish).
      const i32x4 rsrc = make_rsrc(parts + int64_t(h) * n_tokens * kPartRow, static_cast<unsigned>(n_tokens * kPartRow));
      const unsigned lds = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) unsigned char*)smem)) + wave * 1024;
      unsigned off[2][2];  // [K, V][row]
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r = (wave + 4 * i) * 8 + (lane >> 3), c = lane & 7;
        off[0][i] = r * kPartRow + ((c ^ swz_k(r)) << 4);
        off[1][i] = r * kPartRow + 3 * 128 + ((c ^ swz_v(r)) << 4);
      }
      auto fetch = [&](auto tc, int64_t key0) {
        constexpr int T = decltype(tc)::value;
        const unsigned at = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(key0) * kPartRow);
        const unsigned base = __builtin_amdgcn_readfirstlane(lds);
        dma16<(3 * T + 0) * kPlane>(rsrc, off[T][0], at, base);
        dma16<(3 * T + 1) * kPlane>(rsrc, off[T][0], at + 128, base);
        dma16<(3 * T + 2) * kPlane>(rsrc, off[T][0], at + 256, base);
        dma16<(3 * T + 0) * kPlane + 4096>(rsrc, off[T][1], at, base);
        dma16<(3 * T + 1) * kPlane + 4096>(rsrc, off[T][1], at + 128, base);
        dma16<(3 * T + 2) * kPlane + 4096>(rsrc, off[T][1], at + 256, base);
      };
      // K of the next tile is loaded under the output products, V under the scores of its own; each has one place in the LDS, which
      // is free from the barrier on that ends the products with it.
      auto arrived = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0), lgkmcnt(0): this wave's share has landed, and it has read what it had to
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      };
      if (piece < pieces) fetch(std::integral_constant<int, 0>{}, key0);
      while (piece < pieces) {
        const bool ask = (++done & 7) == 0;
        if (ask) look();
        asm volatile("" ::: "memory");
        arrived();
        if (ask && given_up()) return true;
        fetch(std::integral_constant<int, 1>{}, key0);
        const int here = valid;
        piece = next_piece(piece + 1, key0, valid);
        const float a = scores(here);
        asm volatile("" ::: "memory");
        arrived();
        if (piece < pieces) fetch(std::integral_constant<int, 0>{}, key0);
        outputs(a);
      }
      asm volatile("" ::: "memory");
      arrived();
    } else {
      // this thread's share of a tile: chunk (eight dims) tid % 8 of tile rows tid / 8 and 32 + tid / 8, of K and of V
      const int lr = tid >> 3, lc = tid & 7;
      f32x4 raw[2][2][2];  // [K, V][row][half of the chunk]
      auto load = [&](int64_t key0, int valid) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int r = lr + 32 * i;
          // keys past `valid` repeat the last one; they are masked
          const int64_t at = head_off + (key0 + min(r, valid - 1)) * kD + 8 * lc;
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            raw[0][i][x] = *reinterpret_cast<const f32x4*>(k + at + 4 * x);
            raw[1][i][x] = *reinterpret_cast<const f32x4*>(v + at + 4 * x);
          }
        }
      };
      auto store = [&](int valid) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int r = lr + 32 * i;
            if (t == 1 && r >= valid) raw[t][i][0] = raw[t][i][1] = f32x4{0.f, 0.f, 0.f, 0.f};  // their weight is 0, and the last one may be infinite
            u32x4 y[3];
            const unsigned rest = split_chunk(raw[t][i][0], raw[t][i][1], y);
            if (t == 1) left |= rest;
            unsigned char* at = smem + t * 3 * kPlane + r * 128 + ((lc ^ (t ? swz_v(r) : swz_k(r))) << 4);
#pragma unroll
            for (int x = 0; x < 3; ++x) *reinterpret_cast<u32x4*>(at + x * kPlane) = y[x];
          }
      };
      if (piece < pieces) load(key0, valid);
      while (piece < pieces) {
        const int here = valid;
        store(here);
        const bool ask = (++done & 7) == 0;
        if (ask) look();
        __syncthreads();
        if (ask && given_up()) return true;
        piece = next_piece(piece + 1, key0, valid);
        if (piece < pieces) load(key0, valid);
        const float a = scores(here);
        outputs(a);
        __syncthreads();
      }
      if ((left & kCutOff) != 0u) bad_s = 1;  // finish() asks for it after a barrier
    }
    return false;
  };

  bool given_up = tiles();
  if (!given_up) given_up = st.finish(un, wave, lane, reinterpret_cast<float*>(smem), &bad_s, out, lse);
  if (given_up) unit_fp32(un, wave, q, k, v, scale_log2, reinterpret_cast<float*>(smem), out, lse);
}

template <int B>
__global__ __launch_bounds__(256, 2) void attn_fp32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                           const float* __restrict__ v, int64_t n_tokens, int64_t n_first,
                                                           int nb1, int nb, float scale_log2,
                                                           const int32_t* __restrict__ kv_idx,
                                                           const int32_t* __restrict__ kv_cnt, int idx_stride,
                                                           float* __restrict__ out, float* __restrict__ lse) {
  constexpr int ROWS = 32;            // query rows of a workgroup
  constexpr int UNITS = B / ROWS;     // workgroups per query block
  constexpr int PIECES = B / kPiece;  // pieces per key block
  __shared__ float park[4][34][64];  // per wave and lane: 32 output accumulators, reference maximum, row sum
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31;
  const int g = lane >> 5;
  // unit of this workgroup: XCD x takes the x-th eighth of all units
  const int64_t total = int64_t(gridDim.x) * gridDim.y;
  const int64_t w = int64_t(blockIdx.y) * gridDim.x + blockIdx.x;
  const int64_t xcd = w & 7, per = total >> 3, rest = total & 7;
  const int64_t unit = xcd * per + min(xcd, rest) + (w >> 3);
  const int h = static_cast<int>(unit / gridDim.x);
  const int u = static_cast<int>(unit - int64_t(h) * gridDim.x);
  const int I = u / UNITS;
  const int64_t head_off = int64_t(h) * n_tokens * kD;
  // blocks 0 .. nb1-1 tile tokens [0, n_first), the others tokens [n_first, n_tokens)
  auto block_start = [&](int J) { return J < nb1 ? int64_t(J) * B : n_first + int64_t(J - nb1) * B; };
  auto block_count = [&](int J) {
    return static_cast<int>(min<int64_t>(B, (J < nb1 ? n_first : n_tokens) - block_start(J)));
  };
  const int rows = block_count(I) - (u % UNITS) * ROWS;  // query rows from this unit's first on
  if (rows <= 0) return;                                  // the whole workgroup, before any barrier
  const int64_t row0 = block_start(I) + (u % UNITS) * ROWS;

  float qr[32];
  const float* src = q + head_off + (row0 + min(n, rows - 1)) * kD + 4 * g;  // rows past the end are not stored
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(src + 8 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e) qr[4 * c + e] = x[e] * scale_log2;
  }
  f32x16 o[2];
  float m, l;
#pragma unroll
  for (int i = 0; i < 16; ++i) o[0][i] = o[1][i] = 0.f;
  m = -INFINITY;
  l = 0.f;

  const bool dense = kv_idx == nullptr;
  const int64_t row = int64_t(h) * nb + I;
  const int count = dense ? nb : min(max(kv_cnt[row], 0), nb);
  const int pieces = count * PIECES;
  auto key_block = [&](int piece) {
    const int it = piece / PIECES;
    return dense ? it : min(max(kv_idx[row * idx_stride + it], 0), nb - 1);
  };
  float kr[32];
  auto load_k = [&](int64_t key0, int valid) {  // keys past `valid` repeat the last one; they are masked
    const float* src = (k + head_off + key0 * kD) + static_cast<unsigned>(min(n, valid - 1) * kD + 4 * g);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(src + 8 * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) kr[4 * c + e] = x[e];
    }
  };

  // pieces of this wave that hold a key at all: a short block may end before its later pieces
  auto next_piece = [&](int piece, int& J, int& valid) {
    for (; piece < pieces; piece += 4) {
      J = key_block(piece);
      valid = block_count(J) - (piece % PIECES) * kPiece;
      if (valid > 0) break;
    }
    return piece;
  };
  int J = 0, valid = 0;
  int piece = next_piece(wave, J, valid);
  int64_t key0 = 0;
  if (piece < pieces) {
    key0 = block_start(J) + (piece % PIECES) * kPiece;
    load_k(key0, valid);
  }
  while (piece < pieces) {
    f32x2 vr[16];
    {
      const float* base = v + head_off + key0 * kD;  // the same in every lane
      if (valid >= kPiece) {
        const unsigned at = 4 * g * kD + 2 * n;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          vr[i] = *reinterpret_cast<const f32x2*>((base + (i >> 3) * 16 * kD) + at + (8 * ((i >> 2) & 1) + (i & 3)) * kD);
      } else {  // keys past `valid` are zeros (the last one is read in their place, and may be infinite); their weight is 0
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = 8 * (i >> 2) + 4 * g + (i & 3);
          vr[i] = *reinterpret_cast<const f32x2*>(base + static_cast<unsigned>(min(key, valid - 1) * kD + 2 * n));
          if (key >= valid) vr[i] = f32x2{0.f, 0.f};
        }
      }
    }
    f32x16 s;
    s = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < 32; ++d) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kr[d], qr[d], s, 0, 0, 0);
    if (valid < kPiece) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = (8 * (i >> 2) + 4 * g + (i & 3) >= valid) ? -INFINITY : s[i];
    }
    {
      float top = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) top = fmaxf(top, s[i]);
      top = fmaxf(top, __shfl_xor(top, 32));
      if (__any(top > m)) {
        const float m_new = fmaxf(m, top);
        const float a = m == m_new ? 1.f : __builtin_amdgcn_exp2f(m - m_new);  // 0 on the first piece
        l *= a;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          o[0][i] *= a;
          o[1][i] *= a;
        }
        m = m_new;
      }
    }
    float part[2] = {}, ref;  // a wave that has seen nothing but weights of zero (scores of -inf) has no maximum
    ref = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i == 8) {  // the first half of V is used up: its registers take the next piece's keys
        __builtin_amdgcn_sched_barrier(0);
        piece = next_piece(piece + 4, J, valid);
        if (piece < pieces) {
          key0 = block_start(J) + (piece % PIECES) * kPiece;
          load_k(key0, valid);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      const float p = __builtin_amdgcn_exp2f(s[i] - ref);
      part[i & 1] += p;
      o[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i][0], p, o[0], 0, 0, 0);
      o[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i][1], p, o[1], 0, 0, 0);
    }
    l += part[0] + part[1];
  }

  // ---- merge: wave w finishes accumulator registers 4w .. 4w+3, i.e. dims 16w + 8g .. +7 ------------
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    park[wave][2 * i][lane] = o[0][i];
    park[wave][2 * i + 1][lane] = o[1][i];
  }
  park[wave][32][lane] = m;
  park[wave][33][lane] = l;
  __syncthreads();
  float mw[4], top = -INFINITY;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    mw[x] = park[x][32][lane];
    top = fmaxf(top, mw[x]);
  }
  const float mu = top == -INFINITY ? 0.f : top;
  float sum = 0.f, acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const float a = __builtin_amdgcn_exp2f(mw[x] - mu);  // 0 for a wave that saw no key
    sum += park[x][33][lane] * a;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] += park[x][8 * wave + j][lane] * a;
  }
  sum += __shfl_xor(sum, 32);
  if (n < rows) {
    // listed keys, but none with a weight: the softmax is 0 / 0
    const float inv = sum > 0.f ? 1.f / sum : count > 0 ? NAN : 0.f;
    float* dst = out + head_off + (row0 + n) * kD + 16 * wave + 8 * g;
    *reinterpret_cast<f32x4*>(dst) = f32x4{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
    *reinterpret_cast<f32x4*>(dst + 4) = f32x4{acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv};
    if (lse != nullptr && wave == 0 && g == 0)
      lse[int64_t(h) * n_tokens + row0 + n] = sum > 0.f ? (top + log2f(sum)) * 0.6931471805599453f : -INFINITY;
  }
}


}  // namespace

int launch_attn_fp32(const float* q, const float* k, const float* v, int heads, int64_t n_tokens, int64_t n_first,
                     int block, float softmax_scale, const int32_t* kv_idx, const int32_t* kv_cnt, int idx_stride, float* out,
                     float* lse, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  const int nb = static_cast<int>(split_blocks(n_tokens, n_first, block));
  const int nb1 = static_cast<int>(ceil_div(n_first, block));
  const float scale_log2 = softmax_scale * 1.4426950408889634f;
  const dim3 grid(nb * (block / 64), heads), grid32(nb * (block / 32), heads);
  unsigned char* parts = nullptr;
  auto launch_split = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, q, k, v, parts, n_tokens, n_first, nb1, nb, scale_log2, kv_idx, kv_cnt,
                       idx_stride, out, lse);
  };
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid32, dim3(256), 0, stream, q, k, v, n_tokens, n_first, nb1, nb, scale_log2, kv_idx, kv_cnt, idx_stride,
                       out, lse);
  };
  // A unit of 64 rows to a workgroup where that keeps half of the CUs busy.  Dense, 32 rows on the fp32 instructions / 64 split: 86
  // units 65 / 96 us, 96 12 / 17, 172 201 / 188, 176 33 / 28, 272 69 / 54.
  if (int64_t(heads) * nb * (block / 64) <= kFp32FewUnits) {
    if (block == 64) launch(attn_fp32_kernel<64>);
    else launch(attn_fp32_kernel<128>);
    return check_hip(hipGetLastError(), "bsga fp32 attention launch");
  }
  const size_t need = static_cast<size_t>(heads) * static_cast<size_t>(n_tokens) * kPartRow;
  if (need <= kPartsMaxBytes && workspace != nullptr && workspace_bytes >= need && (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0) {
    parts = static_cast<unsigned char*>(workspace);
    const int64_t chunks = int64_t(heads) * n_tokens * (kD / 8);
    hipLaunchKernelGGL(split_kv_kernel, dim3(static_cast<unsigned>(ceil_div(chunks, 256)), 2), dim3(256), 0, stream, k, v, chunks, parts);
    if (int rc = check_hip(hipGetLastError(), "bsga fp32 attention (operand split)")) return rc;
    if (block == 64) launch_split(attn_fp32_split_kernel<64, true>);
    else launch_split(attn_fp32_split_kernel<128, true>);
  } else {
    if (block == 64) launch_split(attn_fp32_split_kernel<64, false>);
    else launch_split(attn_fp32_split_kernel<128, false>);
  }
  return check_hip(hipGetLastError(), "bsga fp32 attention launch");
}

}  // namespace bsga
