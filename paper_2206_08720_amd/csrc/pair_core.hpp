// pair_core.hpp -- fp32 products on the 16-bit matrix cores (v_mfma_f32_32x32x16_f16).
//
// The fp32 matrix cores run at 1/16 of the f16 rate.  A float is therefore held as a pair of f16
// values, x = 2^e (hi + lo) with hi = f16(x 2^-e) and lo = f16(x 2^-e - hi) rounded to nearest,
// and a product is three MFMAs into one fp32 accumulator: hi hi' + hi lo' + lo hi'.  hi and lo
// together hold 23 significant bits, the dropped lo lo' is below 2^-22 of the product, and one
// MFMA adds 16 products per rounding of the fp32 accumulator where v_mfma_f32_32x32x2_f32 adds
// two, so the sums come out closer to the 64-bit ones than the fp32 MFMA's: 5.0e-7 against
// 8.1e-7 (2-norm, K = 2048, normal operands), 7.1e-7 against 1.13e-6 at K = 4096.  A
// 5120 x 5120 x 2048 product takes 309 us against 745 us with the fp32 MFMA (347 and 144
// TFLOP/s of the product's own count; 1.04 PFLOP/s of f16 MFMA work, the rate a large bf16
// library product reaches on the card).
//
// One exponent e per row of an operand (a row is what a sum runs along), so that a row of any
// magnitude uses the f16 range: |x| 2^-e < 2^15, and values down to 2^-18 of the largest keep all
// 23 bits (below that the absolute error is 2^-25 2^e, 2^-40 of the row's largest).  Two rules follow
// for whoever makes pairs.  The exponent is that of the row's true largest element: a bound that multiplies
// maxima of different elements can lie any number of bits above it.  And where the sum's terms count alike
// although one factor is small where the other is large, the factors are balanced by powers of two first
// (kernels_pair.hip).  The error of a sum is then relative to the product of its rows' norms, like the
// rounding of the sum itself; what is lost is the relative precision of a sum whose rows have their large
// elements at different k.
//
// Pair rows in memory: groups of 8 consecutive k, 16 bytes of hi then 16 bytes of lo, so a row of
// K floats takes the same 4 K bytes, is loaded into LDS by the same 16-byte chunks as fp32 rows
// (DmaRowMajor, 32 k per 128-byte tile row) and a 16-byte LDS read is one MFMA operand.  Rows are
// padded with zeros to a multiple of 32 k, so any K is a whole number of K tiles.
//
// MFMA 32x32x16 f16 operand layout (lane l): A[i = l % 32][k = 8 (l / 32) + j] in element j,
// B[k][j = l % 32] likewise; D as the 32x32x2 form.
#pragma once
#include "gemm_core.hpp"

namespace ntk {

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kPairPad = 32;
__host__ __device__ inline long long pair_stride(long long K) { return (K + kPairPad - 1) / kPairPad * kPairPad; }

// largest scaled magnitude 2^15: one bit of headroom below the f16 range
constexpr int kPairTop = 15;
// exponent E with |m| < 2^E (any E for 0 or a value that is not finite, whose products are not
// finite either way)
__device__ __forceinline__ int pair_exp(float m) { return (m > 0.f && m < __builtin_inff()) ? ilogbf(m) + 1 : 0; }

// The same with the elements' own exponents, as integers, so that exponents of rows and of columns add
// up without leaving the range of a float: |x| < 2^pair_e(x) for a finite x != 0; a value that is not
// finite sets no exponent (its row's sums are not finite in any case).
constexpr int kPairNone = -4096;
__device__ __forceinline__ int pair_e(float x) {
  const float a = fabsf(x);
  return a > 0.f && a < __builtin_inff() ? __builtin_amdgcn_frexp_expf(x) : kPairNone;
}
__device__ __forceinline__ float pair_max(float m, float x) {
  const float a = fabsf(x);
  return a < __builtin_inff() ? fmaxf(m, a) : m;
}
// exponent of the balancing factor of a column whose counterpart's largest magnitude is m: a value times the
// factor overflows no earlier than its product with that element
__device__ __forceinline__ int pair_bal_exp(float m) { return m > 0.f && m < __builtin_inff() ? pair_e(m) - 1 : 0; }
// the row's exponent from its elements' largest one
__device__ __forceinline__ int pair_row_e(int e) { return (e <= kPairNone / 2 ? 0 : e) - kPairTop; }

__device__ __forceinline__ void pair_split(float v, _Float16& hi, _Float16& lo) {
  hi = (_Float16)v;
  lo = (_Float16)(v - (float)hi);
}

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N < 64, "vmcnt is 6 bits");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkm0() {
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

// K loop over [k0, k0 + K) (multiples of 32) of the tile at (m0, n0) of A B^T, both operands pair rows:
// the direct-to-LDS loop of gemm_core.hpp with NSTAGE stages and one barrier per K tile.  A K
// tile is 2 FM steps, one A fragment against the wave's FN B fragments (3 FN MFMAs) each; the
// next step's fragments are read while a step's MFMAs run.  With one fragment per wave (small
// tiles, bound by LDS reads and latency) the lo lo' product is added too: the error of a 256-wide
// product drops from 7.5e-8 to 6.2e-8, below the fp32 MFMA's also for short sums.  Ends with a
// barrier.
template <class Cfg, int NSTAGE>
__device__ __forceinline__ void pair_mainloop(const float* __restrict__ A, long long lda, int rowsA,
                                              const float* __restrict__ B, long long ldb, int rowsB, int m0, int n0,
                                              int k0, int K, float* smem, f32x16 (&acc)[Cfg::FM][Cfg::FN]) {
  static_assert(Cfg::BK == 32 && NSTAGE >= 2, "32 k per stage");
  constexpr int AF = Cfg::BM * 32, STAGE = (Cfg::BM + Cfg::BN) * 32;
  constexpr int PER_TILE = (Cfg::BM + Cfg::BN) / (8 * Cfg::WAVES);   // loads per wave and K tile
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm0 = (wave / Cfg::WAVES_N) * Cfg::WM, wn0 = (wave % Cfg::WAVES_N) * Cfg::WN;
  const int lr = lane & 31, lc = (lane >> 5) * 2;
  const int nk = K / 32;
  if (nk <= 0) return;
  DmaRowMajor<Cfg::BM, Cfg::WAVES> ia{A, lda, rowsA};
  DmaRowMajor<Cfg::BN, Cfg::WAVES> ib{B, ldb, rowsB};
  ia.prepare(m0, wave, lane);
  ib.prepare(n0, wave, lane);
  auto issue = [&](int kt, float* st) {
    ia.template issue<Cfg::WAVES>(k0 + kt * 32, st, wave, lane);
    ib.template issue<Cfg::WAVES>(k0 + kt * 32, st + AF, wave, lane);
  };
  const int pre = nk < NSTAGE - 1 ? nk : NSTAGE - 1;
  for (int j = 0; j < pre; ++j) issue(j, smem + j * STAGE);
  if (pre == NSTAGE - 1) wait_vmcnt<(NSTAGE - 2) * PER_TILE>();
  else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  f16x8 a[2][2], b[2][Cfg::FN][2];   // [buffer][hi, lo], [k half][fragment][hi, lo]
  auto frag = [&](const float* st, int row, int chunk) {
    return *reinterpret_cast<const f16x8*>(&st[row * 32 + (DmaTile<32>::swz(row, chunk) << 2)]);
  };
  auto load_a = [&](const float* st, int half, int i, f16x8 (&x)[2]) {
#pragma unroll
    for (int p = 0; p < 2; ++p) x[p] = frag(st, wm0 + i * 32 + lr, half * 4 + lc + p);
  };
  auto load_b = [&](const float* st, int half, f16x8 (&x)[Cfg::FN][2]) {
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p) x[j][p] = frag(st + AF, wn0 + j * 32 + lr, half * 4 + lc + p);
  };
  // the cross products first: the small terms meet a smaller sum
  auto mma = [&](int i, const f16x8 (&x)[2], const f16x8 (&y)[Cfg::FN][2]) {
    if constexpr (Cfg::FM * Cfg::FN == 1)
      acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[1], y[0][1], acc[i][0], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[1], y[j][0], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[0], y[j][1], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[0], y[j][0], acc[i][j], 0, 0, 0);
  };
  load_b(smem, 0, b[0]);
  load_a(smem, 0, 0, a[0]);
  auto tile = [&](int kt, auto stage_tag) {
    constexpr int S = decltype(stage_tag)::value;
    const float* st = smem + S * STAGE;
    if (kt + NSTAGE - 1 < nk) issue(kt + NSTAGE - 1, smem + ((S + NSTAGE - 1) % NSTAGE) * STAGE);
#pragma unroll
    for (int q = 0; q + 1 < 2 * Cfg::FM; ++q) {
      const int half = q / Cfg::FM, next = (q + 1) / Cfg::FM;
      if (next != half) load_b(st, next, b[1]);
      load_a(st, next, (q + 1) % Cfg::FM, a[(q + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      mma(q % Cfg::FM, a[q & 1], b[half]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (kt + 1 < nk) {
      // this wave's loads of tile kt+1 landed and its reads of tile kt returned; after the
      // barrier every wave's have, so tile kt's stage may be overwritten
      if (NSTAGE > 2 && kt + NSTAGE - 1 < nk) wait_vmcnt_lgkm0<(NSTAGE - 2) * PER_TILE>();
      else wait_vmcnt_lgkm0<0>();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      const float* sn = smem + ((S + 1) % NSTAGE) * STAGE;
      load_b(sn, 0, b[0]);
      load_a(sn, 0, 0, a[0]);
      __builtin_amdgcn_sched_barrier(0);
    }
    mma(Cfg::FM - 1, a[1], b[1]);
    __builtin_amdgcn_sched_barrier(0);
  };
  int kb = 0;
  for (; kb + NSTAGE <= nk; kb += NSTAGE) static_for<0, NSTAGE>([&](auto t) { tile(kb + decltype(t)::value, t); });
  static_for<0, NSTAGE - 1>([&](auto t) {
    if (kb + decltype(t)::value < nk) tile(kb + decltype(t)::value, t);
  });
  __syncthreads();
}

// ------------------------------------------------------------------------------ fp32 tiles
// The same products from operands that stay fp32 in memory (the convolutions' gathers, the rows of J):
// a kernel splits them in registers on their way into LDS, scaled by one factor per row.
__device__ __forceinline__ float pair_factor(int e) { return ldexpf(1.f, -max(e, -126)); }
// the exponent of a row whose largest magnitude is at most m (its factor: pair_factor)
__device__ __forceinline__ int pair_row_exp(float m) { return max(pair_exp(m) - kPairTop, -126); }

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
// (mul, v_cvt_pk_f16_f32, v_fma_mix_f32, v_cvt_pk_f16_f32: 12 cycles per value and wave; the
// v_fma_mixlo/hi_f16 forms, which need fewer instructions, take 9 cycles each)
__device__ __forceinline__ void pair_split8(const f32x4& x, const f32x4& y, float s, f16x8& hi, f16x8& lo) {
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    const float a = j < 4 ? x[j] : y[j - 4], b = j < 4 ? x[j + 1] : y[j - 3];
    const f32x2 p = {a * s, b * s};
    const f16x2 h = __builtin_convertvector(p, f16x2);
    const f32x2 r = {__builtin_fmaf(a, s, -(float)h[0]), __builtin_fmaf(b, s, -(float)h[1])};
    const f16x2 l = __builtin_convertvector(r, f16x2);
    hi[j] = h[0];
    hi[j + 1] = h[1];
    lo[j] = l[0];
    lo[j + 1] = l[1];
  }
}

}  // namespace ntk
