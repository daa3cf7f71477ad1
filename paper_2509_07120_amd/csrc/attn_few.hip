// bf16 attention over kept key blocks for launches of few short rows: fewer than 1024 blocks of 64 queries, of which the chip holds 512 at once.
// Products, operand layouts, softmax and range check are those of attn_bf16.hip; what differs is the split.
//
// Such a launch is a chain of latencies: a workgroup has one row of a few key blocks.  With tiles that all four waves share
// (two key blocks at a time, double buffered, a barrier for each) a step took 1.5 to 2 us, of which the products are 0.25.
// Here the four waves of a row are independent until the end: each takes pieces of 32 keys in turn, 64 queries x 32 keys at a
// time, moves them into LDS of its own with direct-to-LDS loads two pieces ahead (reissued as soon as a piece's operands are
// in registers) and waits for nobody.  Then the waves' states are summed through the same LDS, a quarter of the row by each.
// Rows go to the XCDs in consecutive parts, so that an L2 holds the keys of few heads.
// A step is now 0.6 us with one workgroup to a CU and 1.1 us with two (57 steps a wave, 128 rows of 115 of 128 blocks 37.5 us, 512 rows 68): its products
// and exponentials, one after the other.  The attention of
// one frame (352 rows of 20 of 22 blocks) 21.7 -> 16.7 us, of which 0.8 by asking for the next piece under the products and not before
// them (128 rows of 115 of 128 blocks 39.1 -> 37.5).  Tried: the products of one half of the queries between the exponentials
// of the other, within a piece 17.7 us, across pieces with three buffers of K 18.2 to 19.0; K of the next piece read under the last
// products 17.4.
#include <type_traits>

#include "bf16_tile.h"
#include "bsga_internal.h"

namespace bsga {
namespace {

constexpr int kD = 64;
constexpr int kPiece = 32;                      // keys of a wave's step
constexpr int kBuf = 2 * kPiece * 128;          // K, then V
constexpr int kWaveLds = 2 * kBuf;              // also the wave's parked output: 64 registers of 64 lanes
static_assert(kWaveLds == 64 * 64 * 4, "the parked output takes the place of the buffers");
constexpr float kRaise = 8.0f;                  // second pass: the reference maximum follows when exceeded by 2^8
constexpr float kLn2 = 0.6931471805599453f;

__global__ __launch_bounds__(256, 2) void attn_few_kernel(const unsigned char* __restrict__ q, const unsigned char* __restrict__ k,
                                                          const unsigned char* __restrict__ v, unsigned short* __restrict__ out,
                                                          float* __restrict__ lse, const int32_t* __restrict__ kv_idx,
                                                          const int32_t* __restrict__ kv_cnt, int idx_stride, int n_tokens, int n_first,
                                                          int nb1, int nb, float scale_log2, int rows) {
  __shared__ __align__(16) unsigned char smem[4 * kWaveLds];
  __shared__ float sums[4][2][2][64];  // [wave][row sum, reference][query half][lane]
  __shared__ int flag;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, g = lane >> 5;
  const int per_xcd = static_cast<int>(gridDim.x) >> 3;  // workgroup w runs on XCD w % 8
  const int row = static_cast<int>(blockIdx.x & 7) * per_xcd + static_cast<int>(blockIdx.x >> 3);
  if (row >= rows) return;  // the whole workgroup, before any barrier
  const int h = row / nb, I = row - h * nb;
  const int64_t head_bytes = int64_t(h) * n_tokens * 128;
  // block I (of queries or keys): first token and number of tokens; the sequence's two parts are blocked apart
  auto block_start = [&](int b) { return b < nb1 ? b * 64 : n_first + (b - nb1) * 64; };
  auto block_count = [&](int b) { return min(64, (b < nb1 ? n_first : n_tokens) - block_start(b)); };
  const int q_start = block_start(I), q_valid = block_count(I);

  // the wave's pieces: step j is half wave % 2 of list entry 2 j + wave / 2; lane l keeps the entry of step 64 * i + l
  const int half = wave & 1, first = wave >> 1;
  const int32_t* const idx = kv_idx + int64_t(row) * idx_stride;
  auto fetch = [&](int j0) { return idx[min(2 * (j0 + lane) + first, nb - 1)]; };
  int mine = fetch(0);
  const int cnt = __builtin_amdgcn_readfirstlane(min(max(kv_cnt[row], 0), nb));
  const int steps = (cnt - first + 1) >> 1;

  const unsigned head_size = static_cast<unsigned>(n_tokens) * 128u;
  const i32x4 krsrc = make_rsrc(k + head_bytes, head_size), vrsrc = make_rsrc(v + head_bytes, head_size);
  const unsigned wave_lds = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) unsigned char*)smem)) + wave * kWaveLds;
  // wave-load i of a piece covers its rows 8 i .. 8 i + 7; swz_k(r + 8 i) = swz_k(r) ^ i there, swz_v(r + 8 i) = swz_v(r)
  const int r0 = lane >> 3, pos = lane & 7;
  unsigned koff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) koff[i] = r0 * 128 + ((pos ^ r0 ^ i) << 4) + i * 1024;
  const unsigned voff = r0 * 128 + ((pos ^ swz_v(r0)) << 4);
  int limits[2];  // keys of the pieces in flight, by buffer
  auto issue = [&](int j, int b) {
    if (j > 0 && (j & 63) == 0) mine = fetch(j);
    const int J = min(max(__builtin_amdgcn_readlane(mine, j & 63), 0), nb - 1);
    const int start = block_start(J), left = block_count(J) - kPiece * half;
    limits[b] = left;
    const unsigned soff = static_cast<unsigned>(start + (left > 0 ? kPiece * half : 0)) * 128u;  // of a piece with no keys, the block's first
    const unsigned lds = wave_lds + b * kBuf;
    dma16<0>(krsrc, koff[0], soff, lds);
    dma16<1024>(krsrc, koff[1], soff, lds);
    dma16<2048>(krsrc, koff[2], soff, lds);
    dma16<3072>(krsrc, koff[3], soff, lds);
    dma16<kPiece * 128>(vrsrc, voff, soff, lds);
    dma16<kPiece * 128 + 1024>(vrsrc, voff, soff + 1024, lds);
    dma16<kPiece * 128 + 2048>(vrsrc, voff, soff + 2048, lds);
    dma16<kPiece * 128 + 3072>(vrsrc, voff, soff + 3072, lds);
  };
  auto begin = [&]() {
    if (steps > 0) issue(0, 0);
    if (steps > 1) issue(1, 1);
  };
  begin();

  u32x4 q_raw[2][4];
#pragma unroll
  for (int b2 = 0; b2 < 2; ++b2) {
    const int64_t at = min(q_start + b2 * 32 + n, n_tokens - 1);  // rows past the block are computed, not stored
#pragma unroll
    for (int c = 0; c < 4; ++c) q_raw[b2][c] = *reinterpret_cast<const u32x4*>(q + head_bytes + at * 128 + (2 * c + g) * 16);
  }

  int kaddr[4], vaddr[2];
#pragma unroll
  for (int c = 0; c < 4; ++c) kaddr[c] = wave * kWaveLds + n * 128 + (((2 * c + g) ^ swz_k(n)) << 4);
  {
    const int i16 = lane & 15, m = i16 >> 2, j = i16 & 3, G = lane >> 4;
    const int key = 4 * g + m;
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      const int cc = db * 4 + 2 * (G & 1) + (j >> 1);
      vaddr[db] = wave * kWaveLds + kPiece * 128 + key * 128 + ((cc ^ swz_v(key)) << 4) + (j & 1) * 8;
    }
  }

  bf16x8 qf[2][4];
#pragma unroll
  for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      u32x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        y[e] = pack_bf16(__uint_as_float(q_raw[b2][c][e] << 16) * scale_log2, __uint_as_float(q_raw[b2][c][e] & 0xffff0000u) * scale_log2);
      qf[b2][c] = __builtin_bit_cast(bf16x8, y);
    }

  // Returns true (to the whole workgroup) if the row has to be repeated with a running maximum, see attn_bf16.hip.
  auto pass = [&](auto safec) -> bool {
    constexpr bool SAFE = decltype(safec)::value;
    f32x16 o[2][2];  // [dim block][query half]
    float m_ref[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][b2][i] = 0.f;
    if constexpr (SAFE) {
      if (steps > 64) mine = fetch(0);
      begin();
    }
    auto step = [&](int j, auto bufc) {
      constexpr int b = decltype(bufc)::value;
      if (j + 1 < steps) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // the next piece's eight loads may be on their way
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      bf16x8 ka[4], va[2][2];
#pragma unroll
      for (int c = 0; c < 4; ++c) ka[c] = *LDS_PTR(bf16x8, smem + kaddr[c] + b * kBuf);
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int cp = 0; cp < 2; ++cp) {
          const unsigned char* p = smem + vaddr[db] + b * kBuf + 16 * cp * 128;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + 8 * 128));
          const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
          va[db][cp] = __builtin_bit_cast(bf16x8, u32x4{lo2[0], lo2[1], hi2[0], hi2[1]});
        }
      const int limit = limits[b];
      f32x16 sc[2];
      float base[2];
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        base[b2] = (SAFE && m_ref[b2] != -INFINITY) ? m_ref[b2] : 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) sc[b2][i] = -base[b2];
#pragma unroll
        for (int c = 0; c < 4; ++c) sc[b2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[c], qf[b2][c], sc[b2], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the operands are in registers: the buffer is free.  Its
      // loads go out under the products
      if (j + 2 < steps) issue(j + 2, b);
      __builtin_amdgcn_sched_barrier(0);
      if (limit < kPiece) {
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
          for (int i = 0; i < 16; ++i) sc[b2][i] = 8 * (i >> 2) + 4 * g + (i & 3) >= limit ? -INFINITY : sc[b2][i];
      }
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        if constexpr (SAFE) {
          float tmax = -INFINITY;
#pragma unroll
          for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, sc[b2][i]);
          tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
          const bool unset = m_ref[b2] == -INFINITY;
          const bool raise = unset ? (tmax > -INFINITY) : (tmax > kRaise);
          if (__any(raise)) {
            const float shift = raise ? tmax : 0.f;
            const float alpha = unset ? 1.f : exp2f(-shift);
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
        u32x4 w[2];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float e0 = __builtin_amdgcn_exp2f(sc[b2][2 * e]), e1 = __builtin_amdgcn_exp2f(sc[b2][2 * e + 1]);
          l_run[b2] += e0 + e1;
          w[e >> 2][e & 3] = pack_bf16(e0, e1);
        }
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
          for (int cp = 0; cp < 2; ++cp)
            o[db][b2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[db][cp], __builtin_bit_cast(bf16x8, w[cp]), o[db][b2], 0, 0, 0);
      }
    };
    int j = 0;
    for (; j + 1 < steps; j += 2) {
      step(j, std::integral_constant<int, 0>{});
      step(j + 1, std::integral_constant<int, 1>{});
    }
    if (j < steps) step(j, std::integral_constant<int, 0>{});

    // ---- the four states together: each wave leaves its own in four quarters (dim block, query half), [4][64 lanes][4], and
    // wave w sums quarter w.  None of its loads are on their way any more, and the LDS is its own.
    if (threadIdx.x == 0) flag = 0;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x16& x = o[db][b2];
          *reinterpret_cast<f32x4*>(smem + wave * kWaveLds + (((db * 2 + b2) * 4 + r4) * 64 + lane) * 16) =
              f32x4{x[4 * r4], x[4 * r4 + 1], x[4 * r4 + 2], x[4 * r4 + 3]};
        }
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2) {
      sums[wave][0][b2][lane] = l_run[b2];
      sums[wave][1][b2][lane] = m_ref[b2];
    }
    __syncthreads();
    const int db = wave >> 1, b2 = wave & 1;
    float mt = 0.f, lt = 0.f, a[4] = {1.f, 1.f, 1.f, 1.f};
    if constexpr (SAFE) {
      mt = fmaxf(fmaxf(sums[0][1][b2][lane], sums[1][1][b2][lane]), fmaxf(sums[2][1][b2][lane], sums[3][1][b2][lane]));
      const float mu = mt == -INFINITY ? 0.f : mt;
#pragma unroll
      for (int w = 0; w < 4; ++w) a[w] = exp2f(sums[w][1][b2][lane] - mu);  // 0 for a wave that saw nothing
    }
    f32x16 x;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      lt += sums[w][0][b2][lane] * a[w];
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(smem + w * kWaveLds + (((db * 2 + b2) * 4 + r4) * 64 + lane) * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[4 * r4 + r] += y[r] * a[w];
      }
    }
    lt += __shfl_xor(lt, 32);
    if constexpr (!SAFE) {
      bool bad = !(lt >= 0x1p-80f && lt <= 0x1p100f);
#pragma unroll
      for (int i = 0; i < 16; ++i) bad = bad || !(fabsf(x[i]) < INFINITY);
      if (bad && cnt > 0) flag = 1;  // an empty row is zeros by definition, not a range problem
      __syncthreads();
      if (flag != 0) return true;
    }
    const int lrow = b2 * 32 + n;
    if (lrow < q_valid) {
      const int64_t at = int64_t(h) * n_tokens + q_start + lrow;
      const float inv = lt > 0.f ? 1.f / lt : 0.f;
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        *reinterpret_cast<u32x2*>(out + at * kD + db * 32 + 8 * r4 + 4 * g) =
            u32x2{pack_bf16(x[4 * r4] * inv, x[4 * r4 + 1] * inv), pack_bf16(x[4 * r4 + 2] * inv, x[4 * r4 + 3] * inv)};
      if (lse != nullptr && db == 0 && g == 0) lse[at] = lt > 0.f ? (mt + log2f(lt)) * kLn2 : -INFINITY;
    }
    return false;
  };

  if (pass(std::false_type{})) {
    __syncthreads();  // everybody has read the flag and the sums
    pass(std::true_type{});
  }
}

}  // namespace

int launch_attn_few(const void* q, const void* k, const void* v, int heads, int64_t n_tokens, int64_t n_first, float scale_log2,
                    const int32_t* kv_idx, const int32_t* kv_cnt, int idx_stride, void* out, float* lse, hipStream_t stream) {
  const int nb = static_cast<int>(split_blocks(n_tokens, n_first, 64)), rows = heads * nb;
  hipLaunchKernelGGL(attn_few_kernel, dim3(static_cast<unsigned>(8 * ceil_div(rows, 8))), dim3(256), 0, stream,
                     static_cast<const unsigned char*>(q), static_cast<const unsigned char*>(k), static_cast<const unsigned char*>(v),
                     static_cast<unsigned short*>(out), lse, kv_idx, kv_cnt, idx_stride, static_cast<int>(n_tokens), static_cast<int>(n_first),
                     static_cast<int>(ceil_div(n_first, 64)), nb, scale_log2, rows);
  return check_hip(hipGetLastError(), "bsga bf16 attention launch");
}

}  // namespace bsga
