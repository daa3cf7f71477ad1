// fp32 attention over kept key blocks (Sec. 4.1, Eq. (2); Eq. (1) when no index list is given), both
// products on v_mfma_f32_32x32x2 (fp32 operands, fp32 accumulation), online softmax in fp32.
//
// Work split.  A workgroup of four waves owns 64 (or, where that leaves CUs idle, 32) query rows of one block;
// its waves take the 32-key pieces of the row's key blocks in turn, each with a softmax state of its own,
// and the four states are merged through LDS at the end.  Consecutive units run on one XCD (workgroup w runs
// on XCD w % 8), so that an L2 holds the keys of two heads and not of all of them.
//
// Bound by the matrix pipe: a piece of 32 keys is 128 MFMAs of 64 cycles per wave against 32 exponentials and
// 24 loads.  K and V therefore come straight from global memory into operand registers, without LDS or
// barriers: V of a piece is loaded under its score products, K of the next one under its output products.
// Each loaded operand feeds two MFMAs with 64 rows; with 32 rows the loads cost a third of the time.
//   S^T = K Q^T: lane (n = lane%32, g = lane/32) holds dims 8c + 4g .. +3, c = 0..7, of key n as A operand and
//   of query n as B operand (the contraction takes the dims in that order); accumulator register i of the lane
//   is key 8(i/4) + 4g + i%4 of query n.
//   O^T += V^T P^T: step i multiplies keys 8(i/4) + 4g + i%4, so the weights are used where they are; the lane
//   supplies dims 2n and 2n + 1 of that key, one for each of the two accumulators.
// 16 heads x 2,748 tokens, dense (30.9 GFLOP): 0.32 ms, 96 TFLOP/s, 5,496 tokens 108, of 154 that a library
// fp32 GEMM reaches here; one thread per row with scalar FMAs took 1.95 ms (16 TFLOP/s).
#include "bsga_internal.h"

namespace bsga {
namespace {

constexpr int kD = 64;
constexpr int kPiece = 32;  // keys a wave takes at a time

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

template <int B, int NQ>
__global__ __launch_bounds__(256, 2) void attn_fp32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                           const float* __restrict__ v, int64_t n_tokens, int64_t n_first,
                                                           int nb1, int nb, float scale_log2,
                                                           const int32_t* __restrict__ kv_idx,
                                                           const int32_t* __restrict__ kv_cnt, int idx_stride,
                                                           float* __restrict__ out, float* __restrict__ lse) {
  constexpr int ROWS = 32 * NQ;       // query rows of a workgroup
  constexpr int UNITS = B / ROWS;     // workgroups per query block
  constexpr int PIECES = B / kPiece;  // pieces per key block
  __shared__ float park[4][34 * NQ][64];  // per wave and lane: 32 NQ output accumulators, NQ reference maxima, NQ row sums
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

  float qr[NQ][32];
#pragma unroll
  for (int b = 0; b < NQ; ++b) {
    const float* src = q + head_off + (row0 + min(32 * b + n, rows - 1)) * kD + 4 * g;  // rows past the end are not stored
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(src + 8 * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) qr[b][4 * c + e] = x[e] * scale_log2;
    }
  }
  f32x16 o[NQ][2];
  float m[NQ], l[NQ];
#pragma unroll
  for (int b = 0; b < NQ; ++b) {
#pragma unroll
    for (int i = 0; i < 16; ++i) o[b][0][i] = o[b][1][i] = 0.f;
    m[b] = -INFINITY;
    l[b] = 0.f;
  }

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
    f32x16 s[NQ];
#pragma unroll
    for (int b = 0; b < NQ; ++b) s[b] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < 32; ++d)
#pragma unroll
      for (int b = 0; b < NQ; ++b) s[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(kr[d], qr[b][d], s[b], 0, 0, 0);
    if (valid < kPiece) {
#pragma unroll
      for (int b = 0; b < NQ; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[b][i] = (8 * (i >> 2) + 4 * g + (i & 3) >= valid) ? -INFINITY : s[b][i];
    }
#pragma unroll
    for (int b = 0; b < NQ; ++b) {
      float top = s[b][0];
#pragma unroll
      for (int i = 1; i < 16; ++i) top = fmaxf(top, s[b][i]);
      top = fmaxf(top, __shfl_xor(top, 32));
      if (__any(top > m[b])) {
        const float m_new = fmaxf(m[b], top);
        const float a = m[b] == m_new ? 1.f : __builtin_amdgcn_exp2f(m[b] - m_new);  // 0 on the first piece
        l[b] *= a;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          o[b][0][i] *= a;
          o[b][1][i] *= a;
        }
        m[b] = m_new;
      }
    }
    float part[NQ][2] = {}, ref[NQ];  // a wave that has seen nothing but weights of zero (scores of -inf) has no maximum
#pragma unroll
    for (int b = 0; b < NQ; ++b) ref[b] = m[b] == -INFINITY ? 0.f : m[b];
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
#pragma unroll
      for (int b = 0; b < NQ; ++b) {
        const float p = __builtin_amdgcn_exp2f(s[b][i] - ref[b]);
        part[b][i & 1] += p;
        o[b][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i][0], p, o[b][0], 0, 0, 0);
        o[b][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i][1], p, o[b][1], 0, 0, 0);
      }
    }
#pragma unroll
    for (int b = 0; b < NQ; ++b) l[b] += part[b][0] + part[b][1];
  }

  // ---- merge: wave w finishes accumulator registers 4w .. 4w+3, i.e. dims 16w + 8g .. +7 ------------
#pragma unroll
  for (int b = 0; b < NQ; ++b) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      park[wave][32 * b + 2 * i][lane] = o[b][0][i];
      park[wave][32 * b + 2 * i + 1][lane] = o[b][1][i];
    }
    park[wave][32 * NQ + b][lane] = m[b];
    park[wave][33 * NQ + b][lane] = l[b];
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < NQ; ++b) {
    float mw[4], top = -INFINITY;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      mw[x] = park[x][32 * NQ + b][lane];
      top = fmaxf(top, mw[x]);
    }
    const float mu = top == -INFINITY ? 0.f : top;
    float sum = 0.f, acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const float a = __builtin_amdgcn_exp2f(mw[x] - mu);  // 0 for a wave that saw no key
      sum += park[x][33 * NQ + b][lane] * a;
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += park[x][32 * b + 8 * wave + j][lane] * a;
    }
    sum += __shfl_xor(sum, 32);
    if (32 * b + n < rows) {
      // listed keys, but none with a weight: the softmax is 0 / 0
      const float inv = sum > 0.f ? 1.f / sum : count > 0 ? NAN : 0.f;
      float* dst = out + head_off + (row0 + 32 * b + n) * kD + 16 * wave + 8 * g;
      *reinterpret_cast<f32x4*>(dst) = f32x4{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
      *reinterpret_cast<f32x4*>(dst + 4) = f32x4{acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv};
      if (lse != nullptr && wave == 0 && g == 0)
        lse[int64_t(h) * n_tokens + row0 + 32 * b + n] = sum > 0.f ? (top + log2f(sum)) * 0.6931471805599453f : -INFINITY;
    }
  }
}

}  // namespace

int launch_attn_fp32(const float* q, const float* k, const float* v, int heads, int64_t n_tokens, int64_t n_first,
                     int block, float softmax_scale, const int32_t* kv_idx, const int32_t* kv_cnt, int idx_stride, float* out,
                     float* lse, hipStream_t stream) {
  const int nb = static_cast<int>(split_blocks(n_tokens, n_first, block));
  const int nb1 = static_cast<int>(ceil_div(n_first, block));
  const float scale_log2 = softmax_scale * 1.4426950408889634f;
  auto launch = [&](auto kernel, int rows) {
    hipLaunchKernelGGL(kernel, dim3(nb * (block / rows), heads), dim3(256), 0, stream, q, k, v, n_tokens, n_first, nb1, nb,
                       scale_log2, kv_idx, kv_cnt, idx_stride, out, lse);
  };
  // 64 rows per workgroup load half as much per product (0.88 of the time per row when both fill the card), 32
  // rows spread a short layer better: compare the longest CU, 256 CUs, in units of 32 rows.  Dense, 16 heads,
  // 32 / 64 rows: 340 tokens 12.3 / 19.7 us, 700 40 / 34, 1040 76 / 90, 1374 120 / 119, 2000 193 / 172,
  // 2748 366 / 322, 5496 1214 / 1147; two heads, 2748 tokens 62 / 103, 4122 179 / 157.
  const int64_t units = int64_t(heads) * nb * (block / 64);
  const bool wide = 0.88 * static_cast<double>(2 * ceil_div(units, 256)) <= static_cast<double>(ceil_div(2 * units, 256));
  if (block == 64) {
    if (wide) launch(attn_fp32_kernel<64, 2>, 64);
    else launch(attn_fp32_kernel<64, 1>, 32);
  } else {
    if (wide) launch(attn_fp32_kernel<128, 2>, 64);
    else launch(attn_fp32_kernel<128, 1>, 32);
  }
  return check_hip(hipGetLastError(), "bsga fp32 attention launch");
}

}  // namespace bsga
