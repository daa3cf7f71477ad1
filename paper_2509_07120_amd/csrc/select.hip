// Block scores, block softmax and block selection (Sec. 4.1, "Predicting Block Masks" and
// "Selecting Blocks"), all in float64.
//
// Scores.  logits[I][J] = scale * <q_pool[I], k_pool[J]> on v_mfma_f64_16x16x4: a wave keeps 16 query
//   rows (A operand) in registers and meets 16 key blocks (B operand) per 16 instructions.  Lane
//   (i = lane%16, g = lane/16) holds dims 8c + 2g and 8c + 2g + 1, c = 0..7, of row i of either operand: a
//   16-byte load then covers 64 consecutive bytes of 16 rows.  (With 16 consecutive dims to a lane every
//   load touches 64 cache lines.)
//   Accumulator register r of the lane is (row g + 4r, column i).
//
// Selection.  One WAVE per row, the whole row in registers (lane l holds blocks l, l+64, ...).  The
//   ranked prefix the method keeps is found without sorting: with key(p) = the bit pattern of p
//   (monotone for p >= 0) and, for a threshold key C,
//       M(C) = sum of p over {key >= C},   cnt(C) = number of blocks with key >= C,
//   the block at which the ranked cumulative mass first reaches tau is the one with key
//       T = max{C : cnt(C) >= 1 and M(C) >= tau},
//   found by bisection over the key range [key(p_min), key(p_max)].  Steps over the whole row are
//   taken only until 64 blocks are left in the window; those are then put one to a lane and the rest of
//   the steps cost one value per lane.  It stops as soon as one block is left in the window.
//   Blocks above T are kept; blocks that tie with T are kept in ascending block order while the
//   running mass is below tau.  The top-k floor is the same search with the predicate cnt(C) >= k.
//   The sums are taken in a fixed order (lane-local in ascending block order, then a butterfly), so
//   results are deterministic; adding non-negative terms in a fixed order is monotone, which the
//   bisection needs.  Bound by vector issue: about 65 instructions per slot, a third of them the
//   exponential.  2440 blocks x 39,040 rows: 320 us (1209 us when every step ran over the whole row and every
//   reduction over six LDS permutes); four waves per SIMD up to 40 slots.
//
// Two ways to launch.  Up to 512 key blocks one kernel does both: a workgroup of 16 waves computes the
//   scores of 16 rows into LDS (72 KB at 512 key blocks with the candidates, so two workgroups share a CU) and each wave then
//   selects one of the rows.  Longer rows go through the workspace, [heads, nb_q, nb_k] float64, because
//   16 of them do not fit the LDS.
#include <type_traits>

#include "bsga_internal.h"

namespace bsga {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kD = 64;
constexpr int kFusedRows = 16;       // rows (= waves) of a workgroup of the fused kernel
constexpr int kFusedMaxBlocks = 512;

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// ---- wave-wide reductions over DPP and row swaps (no LDS round trips) -----------------------------
// Six steps pair up lanes 1, 2, 4, 8, 16 and 32 apart (the mirrors do 4 and 8: lanes of a quad, then of
// half a row, already agree); every lane ends with the same bits.
template <typename T, typename Op>
__device__ __forceinline__ T wave_all(T v, Op op) {
  static_assert(sizeof(T) == 8, "64-bit values");
  auto step = [&](auto ctrl) {
    const uint2 x = __builtin_bit_cast(uint2, v);
    const uint2 y = make_uint2(
        static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x.x), decltype(ctrl)::value, 0xf, 0xf, false)),
        static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x.y), decltype(ctrl)::value, 0xf, 0xf, false)));
    v = op(v, __builtin_bit_cast(T, y));
  };
  step(std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
  step(std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
  step(std::integral_constant<int, 0x141>{});  // row_half_mirror
  step(std::integral_constant<int, 0x140>{});  // row_mirror
  {
    const uint2 x = __builtin_bit_cast(uint2, v);
    const auto lo = __builtin_amdgcn_permlane16_swap(x.x, x.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(x.y, x.y, false, false);
    v = op(__builtin_bit_cast(T, make_uint2(lo[0], hi[0])), __builtin_bit_cast(T, make_uint2(lo[1], hi[1])));
  }
  {
    const uint2 x = __builtin_bit_cast(uint2, v);
    const auto lo = __builtin_amdgcn_permlane32_swap(x.x, x.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(x.y, x.y, false, false);
    v = op(__builtin_bit_cast(T, make_uint2(lo[0], hi[0])), __builtin_bit_cast(T, make_uint2(lo[1], hi[1])));
  }
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
  return wave_all(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_max(double v) {
  return wave_all(v, [](double a, double b) { return fmax(a, b); });
}
__device__ __forceinline__ double wave_min(double v) {
  return wave_all(v, [](double a, double b) { return fmin(a, b); });
}
__device__ __forceinline__ uint64_t uniform_key(double v) {
  const uint2 x = __builtin_bit_cast(uint2, v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(x.x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane(x.y);
  return (uint64_t(hi) << 32) | lo;
}
__device__ __forceinline__ double key_value(uint64_t key) { return __longlong_as_double(static_cast<long long>(key)); }
__device__ __forceinline__ int votes(bool b) { return static_cast<int>(__popcll(__ballot(b))); }

// What lanes of a wave wrote to LDS before this is what its other lanes read after it.  LDS operations of one
// wave run in order; this keeps the compiler from answering a lane's load with the lane's own earlier store.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// exp(x) for x <= 0 (NaN stays NaN): x = n ln2 + r with |r| <= ln2 / 2, ln2 split in two so that n * hi is
// exact (Cody and Waite's reduction, with fdlibm's two halves), then the Taylor series to r^13 / 13! (the next term is below 2^-57 of the result) and a
// scaling by 2^n.  Largest error against 80-bit exp over 4 million arguments in [-700, 0]: 0.87 units in the
// last place.
__device__ __forceinline__ double exp_nonpos(double x) {
  const double t = x < -800.0 ? -800.0 : x;  // e^-800 is 0 in float64; keeps n finite for -inf
  const double n = __builtin_rint(t * 1.4426950408889634074);
  double r = fma(n, -6.93147180369123816490e-01, t);
  r = fma(n, -1.90821492927058770002e-10, r);
  double e = 1.0 / 6227020800.0;
  e = fma(e, r, 1.0 / 479001600.0);
  e = fma(e, r, 1.0 / 39916800.0);
  e = fma(e, r, 1.0 / 3628800.0);
  e = fma(e, r, 1.0 / 362880.0);
  e = fma(e, r, 1.0 / 40320.0);
  e = fma(e, r, 1.0 / 5040.0);
  e = fma(e, r, 1.0 / 720.0);
  e = fma(e, r, 1.0 / 120.0);
  e = fma(e, r, 1.0 / 24.0);
  e = fma(e, r, 1.0 / 6.0);
  e = fma(e, r, 0.5);
  e = fma(e, r, 1.0);
  e = fma(e, r, 1.0);
  return __builtin_amdgcn_ldexp(e, static_cast<int>(n));
}

// Threshold search.  MASS: largest C with cnt(C) >= 1 and M(C) >= tau; otherwise largest C with
// cnt(C) >= k_target.  Requires the predicate to hold at key_min.  Returns the threshold key T and
// n_gt = cnt(T+1), mass_gt = M(T+1), ties = number of blocks whose key equals T.  Blocks that take no
// part hold a negative p.  `lot`: 64 doubles of LDS of this wave's own.
template <int E, bool MASS>
__device__ __forceinline__ uint64_t find_threshold(const double (&p)[E], uint64_t key_min, uint64_t key_max, int nb_ranked,
                                                   double tau, int k_target, double* lot, int& n_gt, double& mass_gt,
                                                   int& ties) {
  uint64_t lo = key_min, hi = key_max + 1;
  int cnt_lo = nb_ranked, cnt_hi = 0;
  double mass_hi = 0.0;
  auto decide = [&](uint64_t mid, int c, double m) {
    const bool holds = MASS ? (c >= 1 && m >= tau) : (c >= k_target);
    if (__builtin_amdgcn_readfirstlane(holds ? 1 : 0)) {
      lo = mid;
      cnt_lo = c;
    } else {
      hi = mid;
      cnt_hi = c;
      mass_hi = m;
    }
  };
  while (cnt_lo - cnt_hi > 64 && hi - lo > 1) {
    const uint64_t mid = lo + ((hi - lo) >> 1);  // > 0, so negative p never count
    const double at = key_value(mid);
    double s = 0.0;
    int c = 0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const bool ge = p[r] >= at;
      if constexpr (MASS) s += ge ? p[r] : 0.0;
      c += votes(ge);
      if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the scalar registers that hold votes
    }
    if constexpr (MASS) s = wave_sum(s);
    decide(mid, c, s);
  }
  uint64_t T = lo;
  if (hi - lo > 1) {
    // at most 64 blocks are left in [lo, hi): one to a lane, in ascending block order
    const int lane = static_cast<int>(threadIdx.x & 63);
    const double lo_v = key_value(lo), hi_v = key_value(hi);
    int n = 0;
    lot[lane] = -1.0;
    wave_lds_fence();
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const bool in = p[r] >= lo_v && p[r] < hi_v;
      const unsigned long long b = __ballot(in);
      if (in) lot[n + __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(b), 0))] = p[r];
      n += static_cast<int>(__popcll(b));
      if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    wave_lds_fence();
    const double x = lot[lane];
    const int cnt_base = cnt_hi;
    const double mass_base = mass_hi;
    while (cnt_lo - cnt_hi > 1 && hi - lo > 1) {
      const uint64_t mid = lo + ((hi - lo) >> 1);
      const bool ge = x >= key_value(mid);
      decide(mid, cnt_base + votes(ge), MASS ? mass_base + wave_sum(ge ? x : 0.0) : 0.0);
    }
    T = lo;
    if (hi - lo > 1) {  // one block left in [lo, hi): its key is the threshold
      const unsigned long long b = __ballot(x >= key_value(lo) && x < key_value(hi));
      const int src = b != 0 ? __builtin_ctzll(b) : 0;
      const uint2 w = __builtin_bit_cast(uint2, x);
      const uint32_t wl = __builtin_amdgcn_readlane(w.x, src), wh = __builtin_amdgcn_readlane(w.y, src);
      T = (uint64_t(wh) << 32) | wl;
    }
  }
  n_gt = cnt_hi;
  mass_gt = mass_hi;
  ties = cnt_lo - cnt_hi;
  return T;
}

// What the selection of one row needs besides its logits.
struct SelectArgs {
  int nb_q, nb_k;
  double tau, one_minus_rho;
  const uint8_t* force_q;
  const uint8_t* force_k;
  uint32_t* mask_bits;
  int32_t* kv_idx;
  int32_t* kv_cnt;
  int idx_stride;
};

// One wave selects row `row` = head * nb_q + I of which `lrow` holds the nb_k logits (global or LDS).
// FULL: slots 0 .. FULL-1 are known to be whole (64 * FULL <= nb_k); FORCE: force_q or force_k is given.
template <int E, int FULL, bool FORCE, typename Ptr>
__device__ __forceinline__ void select_row(Ptr lrow, int64_t row, int I, const SelectArgs& a, double* lot) {
  const int lane = static_cast<int>(threadIdx.x & 63);
  const int nb_k = a.nb_k;
  const double tau = a.tau;
  // ---- softmax over the ranked blocks: p[r] belongs to block J = 64 r + lane.  Padding (J >= nb_k)
  // and blocks with force_k[J] == 2 (always kept, not ranked) get p = -1 and take no part below.
  double p[E];
  uint32_t ranked[(E + 31) / 32] = {};  // bit r: block 64 r + lane is ranked
  double mx = -INFINITY;
  int nb_ranked = FORCE ? 0 : nb_k;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int J = r * 64 + lane;
    if constexpr (!FORCE) {
      p[r] = r < FULL ? lrow[J] : lrow[min(J, nb_k - 1)];
      if (r >= FULL) p[r] = J < nb_k ? p[r] : -INFINITY;
    } else {
      bool rk = J < nb_k;
      const int Jc = min(J, nb_k - 1);
      if (a.force_k != nullptr) rk = rk && a.force_k[Jc] != 2;
      p[r] = lrow[Jc];
      p[r] = rk ? p[r] : -INFINITY;
      ranked[r / 32] |= rk ? 1u << (r % 32) : 0u;
      nb_ranked += votes(rk);
    }
    mx = fmax(mx, p[r]);
  }
  mx = wave_max(mx);
  // opaque: the compiler would otherwise keep one scalar register pair per slot alive instead of
  // comparing again
#pragma unroll
  for (int w = 0; w < (E + 31) / 32; ++w) asm("" : "+v"(ranked[w]));
  int l = lane;
  asm("" : "+v"(l));
  double z = 0.0;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    p[r] = exp_nonpos(p[r] - mx);
    if constexpr (FORCE) p[r] = (ranked[r / 32] >> (r % 32)) & 1 ? p[r] : -1.0;
    else if (r >= FULL) p[r] = r * 64 + l < nb_k ? p[r] : -1.0;
    z += (!FORCE && r < FULL) ? p[r] : (p[r] < 0.0 ? 0.0 : p[r]);
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the registers that hold comparisons
  }
  z = wave_sum(z);
  // p = e / z, rounded as the division rounds it: with the rounded reciprocal of z one correction of
  // the quotient by its exact remainder suffices (Markstein).  Below e = 1e-296 the remainder can be inexact
  // and p a unit of its last place off; it stays monotone in e, so the ranking is the same.
  const double rz = 1.0 / z;
  auto over_z = [&](double e) {
    const double q0 = e * rz;
    return fma(fma(-q0, z, e), rz, q0);
  };
  double total = 0.0, p_min = INFINITY;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const double q = over_z(p[r]);
    if (!FORCE && r < FULL) {
      p[r] = q;
      total += q;
      p_min = fmin(p_min, q);
    } else {
      const bool out = p[r] < 0.0;
      p[r] = out ? -1.0 : q;
      total += out ? 0.0 : q;
      p_min = fmin(p_min, out ? INFINITY : q);
    }
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  total = wave_sum(total);
  // smallest and largest key among the ranked blocks: the range the bisection works on.  The largest
  // exponential is exp(0) = 1.
  const uint64_t key_min = uniform_key(wave_min(p_min)), key_max = uniform_key(over_z(1.0));

  // ---- threshold ----------------------------------------------------------------------------
  // k = floor(B (1 - rho)) in binary64 as the definition is written, B = number of ranked blocks
  const int k_floor = static_cast<int>(floor(static_cast<double>(nb_ranked) * a.one_minus_rho));
  const int k_target = min(nb_ranked, max(k_floor, 1));
  // tau >= 1 keeps every block by definition (the summed mass may round to 1.0 before blocks of
  // negligible mass are counted); so does a mass that never gets to tau, and a row with nothing ranked
  const bool keep_all = tau >= 1.0 || !(total >= tau) || nb_ranked == 0;
  uint64_t T = 0;
  int n_ties = 0, ties = 0;
  if (!keep_all) {
    int n_gt;
    double mass_gt;
    int n_cdf = 1;  // tau <= 0: the first ranked block already covers it (top-k only selection)
    if (tau > 0.0) {
      T = find_threshold<E, true>(p, key_min, key_max, nb_ranked, tau, 0, lot, n_gt, mass_gt, ties);
      const double pt = key_value(T);
      double run = mass_gt;
      n_ties = 0;
      do {
        run += pt;
        ++n_ties;
      } while (run < tau && n_ties < ties);
      n_cdf = n_gt + n_ties;
    }
    if (n_cdf < k_target || !(tau > 0.0)) {  // the top-k floor decides
      T = find_threshold<E, false>(p, key_min, key_max, nb_ranked, tau, k_target, lot, n_gt, mass_gt, ties);
      n_ties = k_target - n_gt;
    }
  }
  const double cut = key_value(T);  // 0 when everything is kept
  const bool some_ties = n_ties < ties;

  // ---- emit: 64 blocks per slot = two mask words; ties are ranked by block index ---------------
  const int words = (nb_k + 31) >> 5;
  const bool whole_row = FORCE && a.force_q != nullptr && a.force_q[I] != 0;
  int32_t* const idx_row = a.kv_idx != nullptr ? a.kv_idx + row * a.idx_stride : nullptr;
  int running = 0, tie_run = 0;
  auto rank = [](unsigned long long b, int first) {  // first + lanes below this one that voted
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(b >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(b), first)));
  };
  uint32_t word[(E + 31) / 32] = {};  // mask word 64 w + lane
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int J = r * 64 + l;
    asm("" : "+v"(l));  // (each slot's J is made when it is needed)
    // padding never passes (p = -1, cut >= 0); NaN does: only a row that keeps everything can hold one
    bool f = !(p[r] < cut);
    if (some_ties) {
      const bool tied = p[r] == cut;
      const unsigned long long tb = __ballot(tied);
      f = f && !(tied && rank(tb, tie_run) >= n_ties);
      tie_run += static_cast<int>(__popcll(tb));
    }
    if constexpr (FORCE) {
      f = f || whole_row;
      if (a.force_k != nullptr) f = f || a.force_k[min(J, nb_k - 1)] != 0;
      f = f && J < nb_k;
    }
    const unsigned long long bal = __ballot(f);
    word[r / 32] = l == 2 * (r % 32) ? static_cast<uint32_t>(bal) : word[r / 32];
    word[r / 32] = l == 2 * (r % 32) + 1 ? static_cast<uint32_t>(bal >> 32) : word[r / 32];
    asm volatile("" : "+v"(word[r / 32]));  // here, not from 2 E saved scalars at the end
    if (f && idx_row != nullptr) idx_row[rank(bal, running)] = J;
    running += static_cast<int>(__popcll(bal));
    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  if (a.mask_bits != nullptr) {
#pragma unroll
    for (int w = 0; w < (E + 31) / 32; ++w)
      if (w * 64 + l < words) a.mask_bits[row * words + w * 64 + l] = word[w];
  }
  if (l == 0 && a.kv_cnt != nullptr) a.kv_cnt[row] = running;
}

// One row of pooled vectors per lane of a 16-lane group, as an MFMA operand (the last row stands in for rows
// past the end; its products are not stored).
__device__ __forceinline__ void load_rows(double (&x)[16], const double* __restrict__ pool, int row, int n) {
  const int lane = static_cast<int>(threadIdx.x & 63);
  const f64x2* src = reinterpret_cast<const f64x2*>(pool + int64_t(min(row, n - 1)) * kD + (lane >> 4) * 2);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const f64x2 v = src[4 * i];
    x[2 * i] = v[0];
    x[2 * i + 1] = v[1];
  }
}
__device__ __forceinline__ f64x4 products(const double (&a)[16], const double (&b)[16]) {
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 16; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
  return acc;
}

// Logits of 48 (16) query rows against 128 key blocks per wave, four waves of a workgroup below each other.
// Column 2i of a pair of column tiles comes from the first, column 2i + 1 from the second, so a lane holds
// two neighbours and 16 lanes store 256 consecutive bytes (8-byte aligned: nb_k may be odd).  The stores bypass
// the L2, which holds the key rows all workgroups share: at 2440 x 2440 blocks and 16 heads (762 MB
// written, 12.2 GFLOP) 250 us, 349 us with plain stores; a plain fill of the same buffer takes 157 us and the
// products alone 230 us.  32 rows per wave: 312 us, 64 rows: 313 us.  The version before this one (vector
// fp64, four rows per workgroup, every key row read by each) took 810 us.
constexpr int kLogitCols = 128;
template <int ROW_TILES>  // 16 query rows each
__global__ __launch_bounds__(kThreads) void logits_kernel(const double* __restrict__ q_pool, const double* __restrict__ k_pool,
                                                          int nb_q, int nb_k, double score_scale, double* __restrict__ logits) {
  typedef double f64x2_at8 __attribute__((ext_vector_type(2), aligned(8)));
  const int h = blockIdx.z;
  const int lane = threadIdx.x & 63;
  const int i16 = lane & 15;
  const int I0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * 16 * ROW_TILES;
  const int J0 = blockIdx.x * kLogitCols;
  if (I0 >= nb_q) return;  // whole wave; the kernel has no barriers
  const double* qh = q_pool + int64_t(h) * nb_q * kD;
  const double* kh = k_pool + int64_t(h) * nb_k * kD;
  double a[ROW_TILES][16], b[2][16];
#pragma unroll
  for (int rt = 0; rt < ROW_TILES; ++rt) load_rows(a[rt], qh, I0 + rt * 16 + i16, nb_q);
  load_rows(b[0], kh, J0 + 2 * i16, nb_k);
#pragma unroll
  for (int cp = 0; cp < kLogitCols / 32; ++cp) {
    const int J = J0 + cp * 32 + 2 * i16;
    f64x4 even[ROW_TILES], odd[ROW_TILES];
    load_rows(b[1], kh, J + 1, nb_k);
#pragma unroll
    for (int rt = 0; rt < ROW_TILES; ++rt) even[rt] = products(a[rt], b[0]);
    if (cp + 1 < kLogitCols / 32) load_rows(b[0], kh, J + 32, nb_k);
#pragma unroll
    for (int rt = 0; rt < ROW_TILES; ++rt) odd[rt] = products(a[rt], b[1]);
#pragma unroll
    for (int rt = 0; rt < ROW_TILES; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int I = I0 + rt * 16 + (lane >> 4) + 4 * r;
        if (I >= nb_q) continue;
        double* dst = logits + (int64_t(h) * nb_q + I) * nb_k + J;
        if (J + 1 < nb_k)
          __builtin_nontemporal_store(f64x2_at8{score_scale * even[rt][r], score_scale * odd[rt][r]}, reinterpret_cast<f64x2_at8*>(dst));
        else if (J < nb_k)
          __builtin_nontemporal_store(score_scale * even[rt][r], dst);
      }
  }
}

template <int E, int FULL, bool FORCE>
__global__ __launch_bounds__(kThreads, E <= 40 ? 4 : 1) void select_kernel(const double* __restrict__ logits, int64_t rows, SelectArgs args) {
  __shared__ double lot[kWaves][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = int64_t(blockIdx.x) * kWaves + wave;  // = head * nb_q + I
  if (row >= rows) return;  // whole wave; the kernel has no barriers
  select_row<E, FULL, FORCE>(logits + row * args.nb_k, row, static_cast<int>(row % args.nb_q), args, lot[wave]);
}

// Scores and selection of 16 rows of one head; LDS: [16][stride] logits, then 64 doubles per wave.
template <int E, int FULL, bool FORCE>
__global__ __launch_bounds__(kFusedRows * 64) void score_select_kernel(const double* __restrict__ q_pool,
                                                                       const double* __restrict__ k_pool,
                                                                       double score_scale, SelectArgs args) {
  extern __shared__ __align__(16) double rows_lds[];
  const int h = blockIdx.y;
  const int I0 = blockIdx.x * kFusedRows;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int stride = args.nb_k | 1;  // odd: the four rows a lane group writes fall into different banks
  const double* kh = k_pool + int64_t(h) * args.nb_k * kD;
  if (wave * 16 < args.nb_k) {
    double a[16];
    load_rows(a, q_pool + int64_t(h) * args.nb_q * kD, I0 + (lane & 15), args.nb_q);
    for (int c0 = wave * 16; c0 < args.nb_k; c0 += kFusedRows * 16) {
      double b[16];
      load_rows(b, kh, c0 + (lane & 15), args.nb_k);
      const f64x4 acc = products(a, b);
      const int J = c0 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (J < args.nb_k) rows_lds[((lane >> 4) + 4 * r) * stride + J] = score_scale * acc[r];
    }
  }
  __syncthreads();
  const int I = I0 + wave;
  if (I >= args.nb_q) return;  // whole wave, after the only barrier
  select_row<E, FULL, FORCE>(rows_lds + wave * stride, int64_t(h) * args.nb_q + I, I, args, rows_lds + kFusedRows * stride + wave * 64);
}

}  // namespace

size_t select_workspace_bytes(int heads, int nb_q, int nb_k) {
  return size_t(heads) * size_t(nb_q) * size_t(nb_k) * sizeof(double);
}

int launch_select(const double* q_pool, const double* k_pool, int heads, int nb_q, int nb_k, double score_scale,
                  double tau, double one_minus_rho, const uint8_t* force_q, const uint8_t* force_k, uint32_t* mask_bits,
                  int32_t* kv_idx, int32_t* kv_cnt, int idx_stride, void* workspace, hipStream_t stream) {
  const SelectArgs args = {nb_q, nb_k, tau, one_minus_rho, force_q, force_k, mask_bits, kv_idx, kv_cnt, idx_stride};
  const bool force = force_q != nullptr || force_k != nullptr;
  // per-lane register tile: the smallest instantiation that holds ceil(nb_k / 64) blocks per lane; nb_k is
  // above the one before it, whose slots are therefore whole
  const int e = (nb_k + 63) / 64;
  if (nb_k <= kFusedMaxBlocks) {
    const dim3 grid(static_cast<unsigned>(ceil_div(nb_q, kFusedRows)), heads), blk(kFusedRows * 64);
    const size_t lds = (size_t(kFusedRows) * (nb_k | 1) + kFusedRows * 64) * sizeof(double);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, blk, lds, stream, q_pool, k_pool, score_scale, args); };
    // (slots that hold nothing cost what the others do: 22 blocks in four slots, the layer of one frame 29.8 us, in one 28.9)
    if (e <= 1) launch(force ? score_select_kernel<1, 0, true> : score_select_kernel<1, 0, false>);
    else if (e <= 2) launch(force ? score_select_kernel<2, 1, true> : score_select_kernel<2, 1, false>);
    else if (e <= 4) launch(force ? score_select_kernel<4, 2, true> : score_select_kernel<4, 2, false>);
    else launch(force ? score_select_kernel<8, 4, true> : score_select_kernel<8, 4, false>);
    return check_hip(hipGetLastError(), "bsga_select_blocks launch");
  }
  double* logits = static_cast<double*>(workspace);
  auto scores = [&](auto kernel, int row_tiles) {
    const dim3 g(static_cast<unsigned>(ceil_div(nb_k, kLogitCols)), static_cast<unsigned>(ceil_div(nb_q, 4 * 16 * row_tiles)), heads);
    hipLaunchKernelGGL(kernel, g, dim3(kThreads), 0, stream, q_pool, k_pool, nb_q, nb_k, score_scale, logits);
  };
  // Three row tiles to a wave use a loaded key row most; one spreads a few heads over more of the card.  The whole selection,
  // three / one: 60 workgroups of the first kind (4 heads of 513 x 513 blocks) 32 / 24 us, 54 (1 x 1074) 35 / 28, 96 (4 x
  // 700) 34 / 35, 120 (8 x 513) 37 / 38, 192 (8 x 700) 44 / 52, 240 (16 x 513) 49 / 58; 20 rows of 1074, 16 heads 29 / 21.
  const bool few = nb_q <= 64 || ceil_div(nb_k, kLogitCols) * ceil_div(nb_q, 4 * 16 * 3) * heads < 90;
  if (few) scores(logits_kernel<1>, 1);
  else scores(logits_kernel<3>, 3);
  if (int rc = check_hip(hipGetLastError(), "bsga_select_blocks (logits) launch")) return rc;
  const int64_t rows = int64_t(heads) * nb_q;
  const dim3 grid(static_cast<unsigned>(ceil_div(rows, kWaves)));
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, logits, rows, args); };
#define BSGA_SELECT_CASE(E_, FULL_) \
  if (e <= E_) launch(force ? select_kernel<E_, FULL_, true> : select_kernel<E_, FULL_, false>); else
  BSGA_SELECT_CASE(12, 8)
  BSGA_SELECT_CASE(20, 12)
  BSGA_SELECT_CASE(28, 20)
  BSGA_SELECT_CASE(40, 28)
  BSGA_SELECT_CASE(52, 40)
  BSGA_SELECT_CASE(64, 52)
  BSGA_SELECT_CASE(96, 64)
  BSGA_SELECT_CASE(128, 96) { return fail(BSGA_ERR_UNSUPPORTED, "bsga_select_blocks: nb_k = %d exceeds 8192", nb_k); }
#undef BSGA_SELECT_CASE
  return check_hip(hipGetLastError(), "bsga_select_blocks launch");
}

}  // namespace bsga
