// The parts of a transformer block around the attention (Sec. 3.1; the appendix "Theoretical FLOPs Reduction" for what
// they are): linear layers in bf16 with their neighbours folded in, and the layer norm.
//
// linear_kernel: y[i][f] = sum_k x[i][k] w[f][k] + b[f] on v_mfma_f32_32x32x16_bf16, fp32 accumulation, the sum started from the bias.
//
// Tile and split.  A workgroup of four waves, one to a SIMD, takes 64 FU features x 64 TU tokens; each wave a quarter, 32 FU x 32 TU,
// so an operand read from LDS feeds TU (FU) products: at 256 x 192 a step of 64 in k reads 112 KB of LDS and writes 56 KB, 1,350 cycles of
// its time, under 1,536 of matrix products.
// The features are the products' rows, so a lane holds one token and four consecutive features.
//
// Data movement.  Both operands go from global memory straight to LDS (direct-to-LDS loads, 16 bytes per lane), in steps of 64 in k,
// S buffers; rows of 128 bytes, chunks swizzled (swz_k) so that the operand reads are free of bank conflicts.
// Workgroups are persistent and take the steps of all their tiles as one sequence: the loads of the next tile's first steps are under
// way while the last step and the epilogue of this one run.  One barrier per step, a quarter step before its end: by then every
// wave has the operands of the last quarter in registers, so the buffer is free for the step S later, whose loads are
// issued over the next half step (over a quarter: 10,992 tokens, 1024 -> 3072 features 87 us and not 80, 4096 -> 1024 85 and not
// 80; over a whole step 83 and 88.  Steps of 32 in k with four buffers, rows of 64 bytes: 84 and 85).
// Few tiles are bound by the latency of a step's loads, 0.85 us with two buffers, and the smaller tiles have room for more: 128 x 64,
// five buffers instead of two, 800 tokens 4096 -> 1024 54 -> 22 us.
//
// x is [tokens][k], or (x_step = tokens * 128) [k / 64][tokens][64], as the attention leaves its heads: a step is then a head, and the
// heads need not be merged first.  The result is [tokens][features], row i optionally at row_index[i] and added to that row
// of `residual`, or [features / 64][tokens][64], as the attention wants them.
// The epilogue turns 32 tokens at a time through a piece of LDS of the wave's own, so that stores (and the residual's loads) are
// whole rows of up to 256 bytes.  LATER: with another tile to follow, the finished one waits in registers as bf16, and a piece of it is
// turned, and put through GELU, between the products of each of the next tile's first steps.  The stores of all CUs at once take 14 of
// 87 us (10,992 tokens, 1024 -> 3072), GELU another 25 of 126 (1024 -> 4096), with the matrix pipes idle; now 71 and 106.
#include <utility>

#include "bf16_tile.h"
#include "bsga_internal.h"

namespace bsga {
namespace {

// Token tiles that neighbouring workgroups take before the next feature tile, so that an XCD reads few rows of either operand.  4 / 8 / 16 / 32, us:
// 33,000 tokens 4096 -> 1024 266 / 262 / 265 / 272, 1024 -> 3072 195 / 192 / 194 / 205; 16,488 4096 -> 1024 135 / 135 / 138 / 162.
constexpr int kTokenGroup = 8;

struct LinearArgs {
  const unsigned char* x;
  const unsigned char* w;
  const unsigned char* bias;
  const unsigned char* residual;
  unsigned char* out;
  const int32_t* row_index;
  unsigned x_bytes, x_row, x_step;  // bytes of x, of a row, from one step of 64 in k to the next
  unsigned w_bytes, w_row, out_bytes;
  int n_tokens, features, steps;
  int token_tiles, feature_tiles;
  bool heads;  // result as [features / 64][tokens][64]
};

// x Phi(x) = max(x, 0) - |x| h(|x|) with h(a) = Phi(-a), and h = 2^Q, Q a polynomial of degree 7 fitted to log2 Phi(-a) over [0, 7.5] (minimax, by
// reweighted least squares): h is off by 2.2e-5 of itself there, a hundredth of the rounding to bf16 that follows; beyond, below 2^-43, Q goes
// on falling and h ends as 0.  One exponential and no reciprocal: GELU shares the cycles of the products (62 a value; 94 with h = t P(t) exp(-a^2 / 2),
// t = 1 / (1 + c a)).  Infinities and NaN come out as the product x Phi(x) does: -inf 0 is NaN, so that a sum
// that has overflowed stays to be seen (inf is kept by clamping x from above alone).
__device__ __forceinline__ float gelu(float x) {
  const float a = __builtin_fabsf(x);
  float q = -1.4221640e-6f;
  q = fmaf(q, a, 5.2221996e-5f);
  q = fmaf(q, a, -8.4678171e-4f);
  q = fmaf(q, a, 8.1363982e-3f);
  q = fmaf(q, a, -5.3110495e-2f);
  q = fmaf(q, a, -0.45939937f);
  q = fmaf(q, a, -1.1508543f);
  q = fmaf(q, a, -1.0000257f);
  return fmaf(-__builtin_fabsf(fminf(x, 30.f)), __builtin_amdgcn_exp2f(q), fmaxf(x, 0.f));
}

__device__ __forceinline__ float low_bf16(unsigned x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float high_bf16(unsigned x) { return __uint_as_float(x & 0xffff0000u); }

// LDS operations of one wave run in order; this keeps the compiler from moving them past each other
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int FU, int TU, int S, bool LATER>
constexpr int kLinearLds = S * (64 * FU + 64 * TU) * 128 + 4 * 32 * (LATER ? 2 : FU) * 64;
template <int FU, int TU, int S>
constexpr int kLinearPerCu = 2 * kLinearLds<FU, TU, S, false> <= 160 * 1024 ? 2 : 1;  // workgroups to a CU

template <typename Fn, int... I>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, Fn&& fn) {
  (fn(std::integral_constant<int, I>{}), ...);
}
template <int N, typename Fn>  // fn(0) .. fn(N - 1), the number as a constant
__device__ __forceinline__ void each(Fn&& fn) {
  each_of(std::make_integer_sequence<int, N>{}, fn);
}

template <int FU, int TU, int S, bool GELU, bool LATER>
__global__ __launch_bounds__(256, (kLinearPerCu<FU, TU, S>)) void linear_kernel(LinearArgs a) {
  constexpr int FT = 64 * FU, TT = 64 * TU;  // tile
  constexpr int STAGE = (FT + TT) * 128;
  constexpr int SPAN = 2 * FU;  // places in the code over which a step's loads are spread
  constexpr int LOADS = 2 * (FU + TU);  // of a wave for a step
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wf = wave & 1, wt = wave >> 1;
  const int n = lane & 31, g = lane >> 5;

  // which tiles: round r of this workgroup is tile r * gridDim.x + me; consecutive numbers to one XCD (workgroup w runs on XCD w % 8),
  // eight token tiles by four feature tiles there at a time
  const int grid = static_cast<int>(gridDim.x), w_id = static_cast<int>(blockIdx.x);
  const int me = (grid & 7) == 0 ? (w_id & 7) * (grid >> 3) + (w_id >> 3) : w_id;
  const int tiles = a.token_tiles * a.feature_tiles;
  auto place = [&](int tile, int& f0, int& t0) {
    const int per = kTokenGroup * a.feature_tiles;
    const int group = tile / per, rest = tile - group * per;
    const int wide = min(kTokenGroup, a.token_tiles - group * kTokenGroup);
    const int f = rest / wide;
    f0 = f * FT;
    t0 = (group * kTokenGroup + rest - f * wide) * TT;
  };

  // ---- loads: wave-load i of a tensor's tile covers rows 8 wave + 32 i .. +7 ----------------------------------------
  const unsigned smem_addr = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) unsigned char*)smem));
  const i32x4 wrsrc = make_rsrc(a.w, a.w_bytes), xrsrc = make_rsrc(a.x, a.x_bytes);
  unsigned w_off[2], x_off[2];
  {
    const int r0 = wave * 8 + (lane >> 3);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const unsigned chunk = ((lane & 7) ^ swz_k(r0 + 32 * p)) << 4;
      w_off[p] = r0 * a.w_row + chunk;
      x_off[p] = r0 * a.x_row + chunk;
    }
  }
  auto load = [&](auto ic, unsigned wsoff, unsigned xsoff, unsigned lds) {
    constexpr int i = decltype(ic)::value, j = i - 2 * FU;
    if constexpr (j < 0) dma16<i * 4096>(wrsrc, w_off[i & 1], wsoff + i * 32 * a.w_row, lds);
    else dma16<FT * 128 + j * 4096>(xrsrc, x_off[j & 1], xsoff + j * 32 * a.x_row, lds);
  };

  // ---- operand reads: row r0 + 32 u of the wave's, chunk 2c + g; swz_k(r + 32) = swz_k(r) ^ 4 ------------------------
  int f_addr[4], x_addr[4];
  {
    const int rf = wf * 32 * FU + n, rx = wt * 32 * TU + n;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      f_addr[c] = rf * 128 + (((2 * c + g) ^ swz_k(rf)) << 4);
      x_addr[c] = FT * 128 + rx * 128 + (((2 * c + g) ^ swz_k(rx)) << 4);
    }
  }
  auto read_f = [&](int buf, int c, int u) { return *LDS_PTR(bf16x8, smem + buf + f_addr[(u & 1) ? c ^ 2 : c] + u * 4096); };
  auto read_x = [&](int buf, int c, int u) { return *LDS_PTR(bf16x8, smem + buf + x_addr[(u & 1) ? c ^ 2 : c] + u * 4096); };

  f32x16 acc[FU][TU];
  bf16x8 fa[2][FU], fx[2][TU];

  // the steps of all tiles in a row; (lf, lt, ls): what is loaded next
  int tile = me;
  if (tile >= tiles) return;
  int load_tile = me, ls = 0;
  unsigned wsoff, xsoff;
  {
    int f0, t0;
    place(tile, f0, t0);
    wsoff = f0 * a.w_row;
    xsoff = t0 * a.x_row;
  }
  auto advance = [&]() {  // to the step after the one that was just loaded
    wsoff += 128;
    xsoff += a.x_step;
    if (++ls == a.steps) {
      ls = 0;
      load_tile += grid;
      int f0, t0;
      place(load_tile < tiles ? load_tile : me, f0, t0);  // past the end: loaded again and not used
      wsoff = f0 * a.w_row;
      xsoff = t0 * a.x_row;
    }
  };

  u32x2 bias_raw[FU][4];
  auto load_bias = [&](int f0) {
#pragma unroll
    for (int u = 0; u < FU; ++u)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        bias_raw[u][r4] = *reinterpret_cast<const u32x2*>(a.bias + 2 * min(f0 + wf * 32 * FU + 32 * u + 8 * r4 + 4 * g, a.features - 4));
  };
  auto start_sums = [&]() {
#pragma unroll
    for (int u = 0; u < FU; ++u)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
#pragma unroll
        for (int t = 0; t < TU; ++t) {
          acc[u][t][4 * r4] = low_bf16(bias_raw[u][r4].x);
          acc[u][t][4 * r4 + 1] = high_bf16(bias_raw[u][r4].x);
          acc[u][t][4 * r4 + 2] = low_bf16(bias_raw[u][r4].y);
          acc[u][t][4 * r4 + 3] = high_bf16(bias_raw[u][r4].y);
        }
  };

  const unsigned lds_wave = smem_addr + wave * 1024;
#pragma unroll
  for (int i = 0; i < S - 1; ++i) {
    each<LOADS>([&](auto l) { load(l, wsoff, xsoff, lds_wave + i * STAGE); });
    advance();
  }
  each<LOADS>([&](auto l) {
    if constexpr (decltype(l)::value * SPAN / LOADS < FU) load(l, wsoff, xsoff, lds_wave + (S - 1) * STAGE);
  });
  {
    int f0, t0;
    place(tile, f0, t0);
    load_bias(f0);
  }
  start_sums();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  int buf = 0, load_buf = (S - 1) * STAGE;
#pragma unroll
  for (int u = 0; u < FU; ++u) fa[0][u] = read_f(buf, 0, u);
#pragma unroll
  for (int t = 0; t < TU; ++t) fx[0][t] = read_x(buf, 0, t);

  // LATER: the finished tile waits in registers as bf16, piece by piece (32 tokens x 32 PU features), see above
  constexpr int PU = GELU ? 1 : 2, NP = TU * FU / PU, UN = NP % 4 == 0 ? 4 : NP % 3 == 0 ? 3 : 2;  // pieces; those that the code names
  constexpr int CH = 4 * PU, R = 64 / CH;  // chunks of 16 bytes of a piece's rows, rows that the wave reads back at a time
  u32x2 wait[LATER ? NP : 1][CH];
  u32x4 back[32 / R];
  float y[4];
  int wf0 = 0, wt0 = a.n_tokens;  // the waiting tile: none
  const auto orsrc = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, static_cast<int>(a.out_bytes), 0x00020000);
  unsigned char* const turn_piece = smem + S * STAGE + wave * (32 * PU * 64);
  auto piece_value = [&](auto ic, auto vc) {  // value v of a lane's 16 PU, into LDS by fours
    constexpr int i = decltype(ic)::value, v = decltype(vc)::value, k = v >> 2, r = v & 3;
    if constexpr (GELU) y[r] = gelu(r & 1 ? high_bf16(wait[i][k][r >> 1]) : low_bf16(wait[i][k][r >> 1]));
    if constexpr (r == 3) {
      u32x2 two = wait[i][k];
      if constexpr (GELU) two = u32x2{pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
      *reinterpret_cast<u32x2 __attribute__((address_space(3)))*>(
          (__attribute__((address_space(3))) unsigned char*)(turn_piece + n * (CH * 16) + ((k ^ (n & (CH - 1))) << 4) + 8 * g)) = two;
    }
  };
  auto piece_back = [&]() {
    wave_lds_fence();
#pragma unroll
    for (int p = 0; p < 32 / R; ++p) {
      const int r = p * R + lane / CH;
      back[p] = *LDS_PTR(u32x4, turn_piece + r * (CH * 16) + (((lane & (CH - 1)) ^ (r & (CH - 1))) << 4));
    }
    wave_lds_fence();
  };
  auto piece_store = [&](int piece) {
    const int t = piece / (FU / PU), f = wf0 + wf * 32 * FU + (piece - t * (FU / PU)) * 32 * PU + (lane & (CH - 1)) * 8;
#pragma unroll
    for (int p = 0; p < 32 / R; ++p) {
      const int i = wt0 + wt * 32 * TU + 32 * t + p * R + lane / CH;
      unsigned at = a.heads ? (static_cast<unsigned>(f >> 6) * a.n_tokens + i) * 128u + (f & 63) * 2 : (static_cast<unsigned>(i) * a.features + f) * 2u;
      if (i >= a.n_tokens || f >= a.features) at = 0xffffffffu;  // past the buffer's end: not stored
      __builtin_amdgcn_raw_buffer_store_b128(back[p], orsrc, at, 0, 0);
    }
  };
  auto pieces_move = [&]() {
#pragma unroll
    for (int i = 0; i + UN < (LATER ? NP : 0); ++i)
#pragma unroll
      for (int k = 0; k < CH; ++k) wait[i][k] = wait[i + UN][k];
  };

  // A step; with a piece of the waiting tile (piecec >= 0, number `piece`): its values between the products of the first three quarters, its
  // stores where the last loads have just arrived, so that the next wait for loads finds them a step old.
  auto step = [&](auto piecec, int piece) {
    constexpr int pi = decltype(piecec)::value;
    each<4>([&](auto cc) {
      constexpr int c = decltype(cc)::value, c1 = (c + 1) & 3;
      if constexpr (c == 3) {
        if constexpr (pi >= 0) piece_back();
        // the operands of this quarter are in registers and the next step's loads have arrived, everywhere after the barrier
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * LOADS) : "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        load_buf = buf;
        buf = buf == (S - 1) * STAGE ? 0 : buf + STAGE;
        advance();
        if constexpr (pi >= 0) piece_store(piece);
      }
      each<FU>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        fa[c1 & 1][u] = read_f(buf, c1, u);
#pragma unroll
        for (int t = u; t < TU; t += FU) fx[c1 & 1][t] = read_x(buf, c1, t);
        each<LOADS>([&](auto l) {
          constexpr int i = decltype(l)::value;
          if constexpr (i * SPAN / LOADS == c1 * FU + u) load(l, wsoff, xsoff, lds_wave + load_buf);
        });
#pragma unroll
        for (int t = 0; t < TU; ++t)
          acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[c & 1][u], fx[c & 1][t], acc[u][t], 0, 0, 0);
        if constexpr (pi >= 0 && c < 3)
          each<16 * PU>([&](auto v) {
            if constexpr (decltype(v)::value * 3 * FU / (16 * PU) == c * FU + u) piece_value(piecec, v);
          });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  constexpr std::integral_constant<int, -1> none;

  for (;;) {
    int s = 0;
    if constexpr (LATER)
      for (; s < NP; s += UN) {  // (the launcher sees to it that a tile has as many steps)
        each<UN>([&](auto i) { step(i, s + decltype(i)::value); });
        pieces_move();
      }
    for (; s < a.steps; ++s) step(none, 0);

    if constexpr (LATER) {
      place(tile, wf0, wt0);
      tile += grid;
      const bool last = tile >= tiles;
      int nf, nt;
      place(last ? me : tile, nf, nt);
      load_bias(nf);
#pragma unroll
      for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          const f32x16& x = acc[i % (FU / PU) * PU + (k >> 2)][i / (FU / PU)];
          const int e = 4 * (k & 3);
          wait[i][k] = u32x2{pack_bf16(x[e], x[e + 1]), pack_bf16(x[e + 2], x[e + 3])};
        }
      if (last) {
        for (int p = 0; p < NP; p += UN) {
          each<UN>([&](auto i) {
            each<16 * PU>([&](auto v) { piece_value(i, v); });
            piece_back();
            piece_store(p + decltype(i)::value);
          });
          pieces_move();
        }
        break;
      }
      start_sums();
      continue;
    }
    if constexpr (!LATER) {
    // ---- epilogue -----------------------------------------------------------------------------------------
    int f0, t0;
    place(tile, f0, t0);
    tile += grid;
    const bool last = tile >= tiles;
    {
      int nf, nt;
      place(last ? me : tile, nf, nt);
      load_bias(nf);
    }
    const auto rrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(a.residual), 0, static_cast<int>(a.out_bytes), 0x00020000);
    constexpr int ROW = FU * 64;  // bytes of a wave's features of one token
    constexpr int RC = ROW / 16;  // chunks of 16 bytes
    unsigned char* const turn = smem + S * STAGE + wave * (32 * ROW);
    const int fw = f0 + wf * 32 * FU, tw = t0 + wt * 32 * TU;
    constexpr int PASS = 64 / RC;       // tokens that the wave reads back at a time
    constexpr int PASSES = 32 / PASS;
    const int rc = lane % RC, rr = lane / RC;
    const int f = fw + rc * 8;  // the lane's eight features
// where the lane's rows go (past the buffer's end: not stored), all row numbers asked for at once; the residual's rows are asked
    // for before the 32 tokens are turned.  (Row numbers, then the
    // residual, after one another for each 32 tokens: 38.6 us and not 31.5 for 10,992 tokens, 1024 -> 1024 with both.)
    unsigned at[TU][PASSES];
    u32x4 res[PASSES];
#pragma unroll
    for (int t = 0; t < TU; ++t)
#pragma unroll
      for (int p = 0; p < PASSES; ++p) {
        const int i = tw + 32 * t + p * PASS + rr;
        const unsigned row = a.row_index != nullptr ? min(max(a.row_index[min(i, a.n_tokens - 1)], 0), a.n_tokens - 1) : i;
        at[t][p] = a.heads ? (static_cast<unsigned>(f >> 6) * a.n_tokens + i) * 128u + (f & 63) * 2 : (row * a.features + f) * 2u;
        if (i >= a.n_tokens || f >= a.features) at[t][p] = 0xffffffffu;
      }
    auto ask = [&](int t) {
      if (a.residual == nullptr) return;
#pragma unroll
      for (int p = 0; p < PASSES; ++p) res[p] = __builtin_amdgcn_raw_buffer_load_b128(rrsrc, at[t][p], 0, 0);
    };
    ask(0);
#pragma unroll
    for (int t = 0; t < TU; ++t) {
#pragma unroll
      for (int u = 0; u < FU; ++u)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          float y[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            y[r] = acc[u][t][4 * r4 + r];
            if constexpr (GELU) y[r] = gelu(y[r]);
          }
          const u32x2 two = {pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
          *reinterpret_cast<u32x2 __attribute__((address_space(3)))*>(
              (__attribute__((address_space(3))) unsigned char*)(turn + n * ROW + (((4 * u + r4) ^ (n & (RC - 1))) << 4) + 8 * g)) = two;
        }
      wave_lds_fence();
#pragma unroll
      for (int p = 0; p < PASSES; ++p) {
        const int r = p * PASS + rr;
        u32x4 y = *LDS_PTR(u32x4, turn + r * ROW + ((rc ^ (r & (RC - 1))) << 4));
        if (a.residual != nullptr) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            y[e] = pack_bf16(low_bf16(y[e]) + low_bf16(res[p][e]), high_bf16(y[e]) + high_bf16(res[p][e]));
        }
        __builtin_amdgcn_raw_buffer_store_b128(y, orsrc, at[t][p], 0, 0);
      }
      if (t + 1 < TU) ask(t + 1);
      wave_lds_fence();
    }
    if (last) break;
    start_sums();
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // loads that nobody uses have arrived before the LDS is given back
}

// out[i] = layer norm of x[index[i]] (or of x[i]), a row to a wave, the row in registers: mean, then the mean of squared
// distances from it, in fp32.  Bound by memory: one pass over either.
template <int SLOTS>  // chunks of eight values per lane
__global__ __launch_bounds__(256) void layer_norm_kernel(const unsigned char* __restrict__ x, const unsigned char* __restrict__ weight,
                                                         const unsigned char* __restrict__ bias, const int32_t* __restrict__ index,
                                                         unsigned char* __restrict__ out, int n, int d, float eps) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i >= n) return;  // whole wave; the kernel has no barriers
  const int row = index != nullptr ? min(max(index[i], 0), n - 1) : i;
  const int chunks = d >> 3;
  const u32x4* src = reinterpret_cast<const u32x4*>(x + int64_t(row) * d * 2);
  float v[SLOTS][8];
  u32x4 w[SLOTS], b[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    w[s] = reinterpret_cast<const u32x4*>(weight)[min(s * 64 + lane, chunks - 1)];
    b[s] = reinterpret_cast<const u32x4*>(bias)[min(s * 64 + lane, chunks - 1)];
  }
  float sum = 0.f;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int c = s * 64 + lane;
    const u32x4 raw = src[min(c, chunks - 1)];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[s][2 * e] = low_bf16(raw[e]);
      v[s][2 * e + 1] = high_bf16(raw[e]);
      sum += c < chunks ? v[s][2 * e] + v[s][2 * e + 1] : 0.f;
    }
  }
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  float mean = sum / d;
  if (!(fabsf(mean) < INFINITY)) {  // the whole wave: the sum of values that fit may not, but their mean does
    mean = 0.f;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
#pragma unroll
      for (int e = 0; e < 8; ++e) mean += s * 64 + lane < chunks ? v[s][e] / d : 0.f;
    for (int o = 32; o > 0; o >>= 1) mean += __shfl_xor(mean, o);
  }
  float squares = 0.f;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[s][e] -= mean;
      squares += s * 64 + lane < chunks ? v[s][e] * v[s][e] : 0.f;
    }
  for (int o = 32; o > 0; o >>= 1) squares += __shfl_xor(squares, o);
  const float scale = 1.f / sqrtf(squares / d + eps);
  u32x4* dst = reinterpret_cast<u32x4*>(out + int64_t(i) * d * 2);
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int c = s * 64 + lane;
    if (c >= chunks) continue;
    u32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      y[e] = pack_bf16(fmaf(v[s][2 * e] * scale, low_bf16(w[s][e]), low_bf16(b[s][e])),
                       fmaf(v[s][2 * e + 1] * scale, high_bf16(w[s][e]), high_bf16(b[s][e])));
    dst[c] = y;
  }
}

template <int FU, int TU, int S>
int launch_tiles(LinearArgs a, bool with_gelu, hipStream_t stream) {
  a.token_tiles = static_cast<int>(ceil_div(a.n_tokens, 64 * TU));
  a.feature_tiles = static_cast<int>(ceil_div(a.features, 64 * FU));
  constexpr int places = 256 * kLinearPerCu<FU, TU, S>;
  const int64_t tiles = int64_t(a.token_tiles) * a.feature_tiles;
  const dim3 grid(static_cast<unsigned>(min(tiles, int64_t(places))));
  auto launch = [&](auto kernel, size_t lds) { hipLaunchKernelGGL(kernel, grid, dim3(256), lds, stream, a); };
  if constexpr (S == 2) {
    // another tile to store the result under, with a step for each of its pieces
    if (tiles > places && a.residual == nullptr && a.row_index == nullptr && a.steps >= (with_gelu ? TU * FU : TU * FU / 2)) {
      if (with_gelu) launch(linear_kernel<FU, TU, S, true, true>, kLinearLds<FU, TU, S, true>);
      else launch(linear_kernel<FU, TU, S, false, true>, kLinearLds<FU, TU, S, true>);
      return check_hip(hipGetLastError(), "bsga_linear launch");
    }
  }
  if (with_gelu) launch(linear_kernel<FU, TU, S, true, false>, kLinearLds<FU, TU, S, false>);
  else launch(linear_kernel<FU, TU, S, false, false>, kLinearLds<FU, TU, S, false>);
  return check_hip(hipGetLastError(), "bsga_linear launch");
}

}  // namespace

int launch_linear(const void* x, bool x_heads, const void* weight, const void* bias, int64_t n_tokens, int in_features, int out_features, bool gelu,
                  const int32_t* row_index, const void* residual, bool out_heads, void* out, hipStream_t stream) {
  LinearArgs a = {};
  a.x = static_cast<const unsigned char*>(x);
  a.w = static_cast<const unsigned char*>(weight);
  a.bias = static_cast<const unsigned char*>(bias);
  a.residual = static_cast<const unsigned char*>(residual);
  a.out = static_cast<unsigned char*>(out);
  a.row_index = row_index;
  a.x_bytes = static_cast<unsigned>(n_tokens * in_features * 2);
  a.x_row = x_heads ? 128 : in_features * 2;
  a.x_step = x_heads ? static_cast<unsigned>(n_tokens * 128) : 128;
  a.w_bytes = static_cast<unsigned>(int64_t(out_features) * in_features * 2);
  a.w_row = in_features * 2;
  a.out_bytes = static_cast<unsigned>(n_tokens * out_features * 2);
  a.n_tokens = static_cast<int>(n_tokens);
  a.features = out_features;
  a.steps = in_features / 64;
  a.heads = out_heads;
  // The kernel with the least rounds of the chip times time of a tile, (steps * step + rest) ns as fitted to sequences of 800 to 33,000
  // tokens at 1024 features.  Wide tiles move least, narrow ones with many buffers hide the latency of a launch of one round and leave
  // less of the last round idle.  us, 256 x 192 / 128 x 192 / 128 x 128, two to a CU / 128 x 128, four buffers / 128 x 64, five:
  // 10,992 tokens 1024 -> 3072 78 / 85 / 89 / 85 / 109, 4096 -> 1024 82 / 97 / 134 / 102 / 129; 4,122 45 / 39 / 39 / 38 / 45, 69 / 44 / 64 /
  // 59 / 61; 1,374 24 / 16 / 19 / 20 / 21, 65 / 39 / 59 / 30 / 23.
  struct Shape {
    int features, tokens, places, step, rest;
    int (*launch)(LinearArgs, bool, hipStream_t);
  };
  static const Shape shapes[] = {{256, 192, 256, 1000, 10000, launch_tiles<4, 3, 2>},
                                 {128, 192, 256, 560, 6000, launch_tiles<2, 3, 3>},
                                 {128, 128, 512, 950, 3000, launch_tiles<2, 2, 2>},
                                 {128, 128, 256, 480, 2500, launch_tiles<2, 2, 4>},
                                 {128, 64, 256, 310, 2000, launch_tiles<2, 1, 5>}};
  const Shape* best = nullptr;
  int64_t least = 0;
  for (const Shape& c : shapes) {
    const int64_t tiles = ceil_div(n_tokens, c.tokens) * ceil_div(out_features, c.features);
    const int64_t ns = ceil_div(tiles, c.places) * (int64_t(a.steps) * c.step + c.rest);
    if (best != nullptr && ns >= least) continue;
    best = &c;
    least = ns;
  }
  return best->launch(a, gelu, stream);
}

int launch_layer_norm(const void* x, const void* weight, const void* bias, float eps, int64_t n_tokens, int features, const int32_t* index, void* out,
                      hipStream_t stream) {
  const dim3 grid(static_cast<unsigned>(ceil_div(n_tokens, 4)));
  const unsigned char *xp = static_cast<const unsigned char*>(x), *wp = static_cast<const unsigned char*>(weight),
                      *bp = static_cast<const unsigned char*>(bias);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, xp, wp, bp, index, static_cast<unsigned char*>(out), static_cast<int>(n_tokens),
                       features, eps);
  };
  if (features <= 512) launch(layer_norm_kernel<1>);
  else if (features <= 1024) launch(layer_norm_kernel<2>);
  else if (features <= 2048) launch(layer_norm_kernel<4>);
  else launch(layer_norm_kernel<8>);
  return check_hip(hipGetLastError(), "bsga_layer_norm launch");
}

}  // namespace bsga
