// kernels_pair.hip -- the cotangent backward of a fully-connected net on pair rows (pair_core.hpp):
// fp32 products on the f16 matrix cores.
//
//   k_pair_wstats, k_pair_weights  rows of W_l^T as pair rows, all layers
//   k_pair_rows     pair rows of cotangents: of fp32 rows, or the readout's Wr[o, c] act'(z[n, c])
//   k_pair_bwd      G_{l-1} = (G_l W_l) * act'(z_{l-1}), pair rows in, fp32 rows out
//
// Exponents.  A pair holds 23 bits of what lies within 2^18 of its row's largest element, so a row's
// exponent has to follow that element itself, and units of very different scales must not meet in
// one row where the small ones count as much as the large ones.
//   * k_pair_bwd stores fp32 and k_pair_rows, which sees whole rows, makes pair rows of them with the
//     exponent of the true largest element.  (A bound formed beforehand, max |G_l| times the largest
//     column sum of W_l, saves that pass but multiplies maxima of different units: with one unit of
//     width 512 at 2^-14 of the others' scale its error was 1e-2, with log-normal scales of 4 bits 0.7.)
//   * In the contraction G1 G2^T the large elements of a row carry the result: rows as they are.
//   * In the backward sum_k G_l[r, k] W_l[k, n] a unit k whose incoming weights W_l[k, :] are small has
//     large cotangents in return, and all k count alike.  The operands are therefore balanced: row k of
//     W_l is scaled by 2^-d_k (2^d_k: the power of two below its largest element) and G_l[:, k] by 2^d_k,
//     which is exact.  Scaling a unit's incoming weights by a power of two and its outgoing ones by the inverse
//     then changes no bit of the operands but the exponents.
#include "gram_small.hpp"
#include "launch.hpp"
#include "pair_core.hpp"

namespace ntk {

static inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------------------------------------ weights
// Two launches over all layers.  Workgroup (chunk, layer) of k_pair_wstats takes kWChunk rows k of W:
// their d_k, then per column the largest exponent of the balanced chunk (the second read comes from
// the caches).  k_pair_weights transposes 64 x 64 tiles through LDS, 32 bytes (8 k of hi and of lo)
// per thread and step.  Bound by memory: W is read twice and written once.
constexpr int kWChunk = 32;
// layers of the one-launch form (its batches are kernel arguments)
constexpr int kPrepLayers = 12;
__global__ void __launch_bounds__(1024) k_pair_wstats(PairWeights b) {
  __shared__ int kd[kWChunk];
  static_assert(kWChunk == 32 && kPairPad % kWChunk == 0, "two rows per wave; the last chunk holds the padding");
  const int z = blockIdx.y;
  const int K = b.K[z], N = b.N[z], k0 = blockIdx.x * kWChunk;
  if (k0 >= K) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* __restrict__ W = b.W[z] + (long long)k0 * N;
  const int rows = min(kWChunk, K - k0);
  const bool vec = N % 4 == 0 && (reinterpret_cast<uintptr_t>(b.W[z]) & 15) == 0;
  const float* __restrict__ x[2];
  float m[2] = {0.f, 0.f};   // over finite elements
#pragma unroll
  for (int i = 0; i < 2; ++i) x[i] = W + (long long)min(2 * wave + i, rows - 1) * N;
  if (vec) {
#pragma unroll 8
    for (int n = 4 * lane; n < N; n += 256) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(x[i] + n);
#pragma unroll
        for (int j = 0; j < 4; ++j) m[i] = pair_max(m[i], v[j]);
      }
    }
  } else {
#pragma unroll 8
    for (int n = lane; n < N; n += 64)
#pragma unroll
      for (int i = 0; i < 2; ++i) m[i] = pair_max(m[i], x[i][n]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int q = 32; q; q >>= 1) m[i] = fmaxf(m[i], __shfl_xor(m[i], q));
    const int r = 2 * wave + i;
    const int e = r < rows ? pair_bal_exp(m[i]) : 0;
    if (lane == 0) {
      kd[r] = e;
      b.kexps[z][k0 + r] = e;
      b.kfac[z][k0 + r] = ldexpf(1.f, e);
    }
  }
  __syncthreads();
  for (int n = threadIdx.x; n < N; n += 1024) {
    int mx = kPairNone;
#pragma unroll
    for (int i = 0; i < kWChunk; ++i) {
      const int r = min(i, rows - 1);
      mx = max(mx, pair_e(W[(long long)r * N + n]) - kd[r]);
    }
    b.stats[z][(long long)blockIdx.x * N + n] = mx;
  }
}

// One 64 x 64 tile (columns n0.., rows k0..) of W_z, 256 threads.
struct PairWeightsLds {
  int ex[64], kd[64];
  int red[4][64];
  float tile[64][65];
};
template <class PW>
__device__ __forceinline__ void pair_weights_tile(const PW& b, int z, int nt, int kt, PairWeightsLds& lds) {
  const int K = b.K[z], N = b.N[z];
  const int n0 = nt * 64, k0 = kt * 64;
  const int ldo = (int)pair_stride(K);
  if (n0 >= N || k0 >= ldo) return;
  const int c = threadIdx.x & 63, kr = threadIdx.x >> 6;
  const float* __restrict__ W = b.W[z] + min(n0 + c, N - 1);
  float v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = W[(long long)min(k0 + kr + 4 * i, K - 1) * N];
  const int* __restrict__ st = b.stats[z] + min(n0 + c, N - 1);
  const int chunks = (K + kWChunk - 1) / kWChunk;
  int m = kPairNone;
#pragma unroll 8
  for (int i = kr; i < chunks; i += 4) m = max(m, st[(long long)i * N]);
  lds.red[kr][c] = m;
  if (threadIdx.x < 64) lds.kd[c] = b.kexps[z][min(k0 + c, K - 1)];
  __syncthreads();
  if (threadIdx.x < 64) {
    const int e = pair_row_e(max(max(lds.red[0][c], lds.red[1][c]), max(lds.red[2][c], lds.red[3][c])));
    lds.ex[c] = e;
    if (kt == 0 && n0 + c < N) b.exps[z][n0 + c] = e;
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) lds.tile[kr + 4 * i][c] = k0 + kr + 4 * i < K ? v[i] : 0.f;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int rn = (threadIdx.x >> 3) + 32 * i, g = threadIdx.x & 7;   // output row, group of 8 k
    if (n0 + rn < N && k0 + 8 * g < ldo) {
      f16x8 hi, lo;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        _Float16 x, y;
        pair_split(ldexpf(lds.tile[8 * g + j][rn], -lds.kd[8 * g + j] - lds.ex[rn]), x, y);
        hi[j] = x;
        lo[j] = y;
      }
      f16x8* o = reinterpret_cast<f16x8*>(b.out[z] + (long long)(n0 + rn) * ldo + k0 + 8 * g);
      o[0] = hi;
      o[1] = lo;
    }
  }
}

__global__ void __launch_bounds__(256) k_pair_weights(PairWeights b) {
  __shared__ PairWeightsLds lds;
  pair_weights_tile(b, blockIdx.z, blockIdx.x, blockIdx.y, lds);
}

long long pair_stats_ints(long long K, long long N) { return (K + kWChunk - 1) / kWChunk * N; }

hipError_t launch_pair_wstats(hipStream_t s, const PairWeights& b) {
  if (b.count <= 0) return hipSuccess;
  if (b.count > kMaxLayers) return hipErrorInvalidValue;
  int maxK = 0;
  for (int z = 0; z < b.count; ++z) maxK = std::max(maxK, b.K[z]);
  k_pair_wstats<<<dim3(cdiv(maxK, kWChunk), b.count), dim3(1024), 0, s>>>(b);
  return hipGetLastError();
}

hipError_t launch_pair_weights(hipStream_t s, const PairWeights& b) {
  if (b.count <= 0) return hipSuccess;
  if (b.count > kMaxLayers) return hipErrorInvalidValue;
  int maxN = 0, maxK = 0;
  for (int z = 0; z < b.count; ++z) {
    maxN = std::max(maxN, b.N[z]);
    maxK = std::max(maxK, b.K[z]);
  }
  if (cdiv(maxK, 64) > 65535) return hipErrorInvalidValue;
  k_pair_weights<<<dim3(cdiv(maxN, 64), cdiv(pair_stride(maxK), 64), b.count), dim3(256), 0, s>>>(b);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------ cotangent rows
// Pair rows of R rows r = (n, o) of K values, WPR waves per row: the first kRowGroups groups of 8 per
// lane stay in registers between the row's exponents and the writes, later ones are read again.  A
// group of 8 floats and its pairs are the same 32 bytes of a row, read and written by one lane, so the
// result may replace its source.  Bound by memory, one read and two writes: 5120 rows of 2048 take
// 49 us beside the backward of the other half of the samples, 2.6 TB/s (78 us with an integer exponent
// per element in place of maxima of products); depth 8, width 2048, 512 + 512 samples: 0.24 of 5.25 ms.
constexpr int kRowGroups = 4;
// VEC: whole groups of 8 can be read from 16-byte addresses (values past K are replaced by zeros)
template <int WPR, bool VEC, bool SEED>
__device__ __forceinline__ void pair_rows_block(const PairRows& p, int bx, float (*red)[2]) {
  const int t = WPR == 1 ? threadIdx.x & 63 : threadIdx.x;
  const int r = WPR == 1 ? bx * 4 + (threadIdx.x >> 6) : bx;
  if (r >= p.R) return;   // whole waves, and with WPR > 1 whole workgroups
  const int n = SEED ? (int)p.fO.div(r) : 0;
  const float* a = SEED ? p.Wr + (long long)(r - n * (int)p.fO.d) * p.K : p.in + (long long)r * p.ldin;
  const float* d = SEED ? p.dphi + (long long)n * p.K : nullptr;
  const int K = p.K, Kp = (int)pair_stride(K);
  auto load = [&](int k0, float (&v)[8]) {
    if (VEC) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 x = *reinterpret_cast<const f32x4*>(a + k0 + 4 * h);
        if (SEED) {
          const f32x4 y = *reinterpret_cast<const f32x4*>(d + k0 + 4 * h);
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] *= y[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 * h + j] = k0 + 4 * h + j < K ? x[j] : 0.f;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = min(k0 + j, K - 1);
        const float x = SEED ? a[k] * d[k] : a[k];
        v[j] = k0 + j < K ? x : 0.f;
      }
    }
  };
  float mp = 0.f, mb = 0.f;
  auto factors = [&](int k0, float (&f)[8]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(p.kfac + k0 + 4 * h);
#pragma unroll
      for (int j = 0; j < 4; ++j) f[4 * h + j] = x[j];
    }
  };
  auto scan = [&](int k0, const float (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) mp = fmaxf(mp, fabsf(v[j]));
    if (p.kfac) {
      float f[8];
      factors(k0, f);
#pragma unroll
      for (int j = 0; j < 8; ++j) mb = fmaxf(mb, fabsf(v[j] * f[j]));
    }
  };
  constexpr int STEP = WPR * 64 * 8;
  float v[kRowGroups][8];
#pragma unroll
  for (int i = 0; i < kRowGroups; ++i)
    if (8 * t + i * STEP < K) load(8 * t + i * STEP, v[i]);
#pragma unroll
  for (int i = 0; i < kRowGroups; ++i)
    if (8 * t + i * STEP < K) scan(8 * t + i * STEP, v[i]);
  for (int k0 = 8 * t + kRowGroups * STEP; k0 < K; k0 += STEP) {
    float x[8];
    load(k0, x);
    scan(k0, x);
  }
#pragma unroll
  for (int q = 32; q; q >>= 1) {
    mp = fmaxf(mp, __shfl_xor(mp, q));
    mb = fmaxf(mb, __shfl_xor(mb, q));
  }
  if (WPR > 1) {
    if ((t & 63) == 0) {
      red[t >> 6][0] = mp;
      red[t >> 6][1] = mb;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WPR; ++w) {
      mp = fmaxf(mp, red[w][0]);
      mb = fmaxf(mb, red[w][1]);
    }
  }
  const int ep = pair_row_exp(mp), eb = pair_row_exp(mb);
  if (t == 0) {
    if (p.out) p.exps[r] = ep;
    if (p.kfac) p.bexps[r] = eb;
  }
  auto write = [&](int k0, const float (&v)[8]) {
    auto put = [&](float* row, const f16x8& hi, const f16x8& lo) {
      f16x8* o = reinterpret_cast<f16x8*>(row + k0);
      o[0] = hi;
      o[1] = lo;
    };
    f16x8 hi, lo;
    if (p.kfac) {
      float f[8];
      factors(k0, f);
      const f32x4 a = {v[0] * f[0], v[1] * f[1], v[2] * f[2], v[3] * f[3]};
      const f32x4 b = {v[4] * f[4], v[5] * f[5], v[6] * f[6], v[7] * f[7]};
      pair_split8(a, b, pair_factor(eb), hi, lo);
      put(p.bout + (long long)r * Kp, hi, lo);
    }
    if (p.out) {
      const f32x4 a = {v[0], v[1], v[2], v[3]}, b = {v[4], v[5], v[6], v[7]};
      pair_split8(a, b, pair_factor(ep), hi, lo);
      put(p.out + (long long)r * Kp, hi, lo);
    }
  };
  const float zeros[8] = {};
#pragma unroll
  for (int i = 0; i < kRowGroups; ++i) {
    const int k0 = 8 * t + i * STEP;
    if (k0 < K) write(k0, v[i]);
    else if (k0 < Kp) write(k0, zeros);
  }
  for (int k0 = 8 * t + kRowGroups * STEP; k0 < Kp; k0 += STEP) {
    float x[8] = {};
    if (k0 < K) load(k0, x);
    write(k0, x);
  }
}

template <int WPR, bool VEC, bool SEED>
__global__ void __launch_bounds__(256) k_pair_rows(PairRows p) {
  __shared__ float red[4][2];
  pair_rows_block<WPR, VEC, SEED>(p, blockIdx.x, red);
}

static bool pair_rows_vec(const PairRows& p) {
  if (!p.in) return p.K % 8 == 0 && vec_ok(p.Wr, p.K, p.K) && vec_ok(p.dphi, p.K, p.K);
  return p.ldin % 4 == 0 && p.ldin >= (p.K + 7) / 8 * 8 && (reinterpret_cast<uintptr_t>(p.in) & 15) == 0;
}

hipError_t launch_pair_rows(hipStream_t s, const PairRows& p) {
  if (p.R <= 0 || p.K <= 0 || (!p.out && !p.kfac)) return hipSuccess;
  auto go = [&](auto wpr, auto vec, auto seed) {
    constexpr int WPR = decltype(wpr)::value;
    k_pair_rows<WPR, decltype(vec)::value, decltype(seed)::value>
        <<<dim3(WPR == 1 ? cdiv(p.R, 4) : p.R), dim3(256), 0, s>>>(p);
    return hipGetLastError();
  };
  auto by_seed = [&](auto wpr, auto vec) { return p.in ? go(wpr, vec, std::false_type{}) : go(wpr, vec, std::true_type{}); };
  auto by_vec = [&](auto wpr) {
    return pair_rows_vec(p) ? by_seed(wpr, std::true_type{}) : by_seed(wpr, std::false_type{});
  };
  // a wave holds up to 2048 values of a row in registers
  return p.K <= 64 * 8 * kRowGroups ? by_vec(std::integral_constant<int, 1>{}) : by_vec(std::integral_constant<int, 4>{});
}

// Small problems: the weights' pair rows, the seed and the Grams in one launch (each alone leaves
// most of the chip idle and costs a launch): the first nw workgroups take 64 x 64 weight tiles,
// the next ns the seed's rows, the others the 16 x 16 Gram blocks (gblocks per layer input).
template <bool SVEC, bool GVEC>
__global__ void __launch_bounds__(256)
k_pair_prep(PairWeightsT<kPrepLayers> b, int wtn, int wtk, int nw, PairRows p, int ns, GramBatchT<kPrepLayers + 1> g,
            int N1, int N2, int gtiles_n, int gblocks) {
  __shared__ union {
    PairWeightsLds w;
    double red[4][256];
  } lds;
  int bx = blockIdx.x;
  if (bx < nw) {
    const int z = bx / (wtn * wtk);
    bx -= z * wtn * wtk;
    pair_weights_tile(b, z, bx % wtn, bx / wtn, lds.w);
  } else if (bx - nw < ns) {
    pair_rows_block<1, SVEC, true>(p, bx - nw, nullptr);
  } else {
    bx -= nw + ns;
    gram_small_block<GVEC>(g, N1, N2, gtiles_n, bx % gblocks, bx / gblocks, lds.red);
  }
}

hipError_t launch_pair_prep(hipStream_t s, const PairWeights& b, const PairRows& p, const GramBatch& g, int N1, int N2,
                            int num_cu) {
  if (p.R <= 0 || p.K <= 0 || p.in) return hipErrorInvalidValue;
  int maxN = 0, maxK = 0;
  for (int z = 0; z < b.count; ++z) {
    maxN = std::max(maxN, b.N[z]);
    maxK = std::max(maxK, b.K[z]);
  }
  if (b.count > kPrepLayers || g.count > kPrepLayers + 1 || !gram_small_fits(g, N1, N2, num_cu)) {
    hipError_t e = launch_pair_weights(s, b);
    if (e == hipSuccess) e = launch_pair_rows(s, p);
    return e != hipSuccess ? e : launch_gram(s, g, N1, N2, num_cu);
  }
  const int wtn = cdiv(maxN, 64), wtk = b.count ? cdiv(pair_stride(maxK), 64) : 0;
  const int nw = wtn * wtk * b.count, ns = cdiv(p.R, 4);
  const int gtn = cdiv(N2, 16), gblocks = cdiv(N1, 16) * gtn;
  const dim3 grid((unsigned)(nw + ns + gblocks * g.count));
  PairWeightsT<kPrepLayers> bs{};
  bs.count = b.count;
  for (int z = 0; z < b.count; ++z) {
    bs.W[z] = b.W[z];
    bs.out[z] = b.out[z];
    bs.exps[z] = b.exps[z];
    bs.kexps[z] = b.kexps[z];
    bs.kfac[z] = b.kfac[z];
    bs.stats[z] = b.stats[z];
    bs.K[z] = b.K[z];
    bs.N[z] = b.N[z];
  }
  GramBatchT<kPrepLayers + 1> gs{};
  gs.count = g.count;
  for (int z = 0; z < g.count; ++z) {
    gs.h1[z] = g.h1[z];
    gs.h2[z] = g.h2[z];
    gs.out[z] = g.out[z];
    gs.K[z] = g.K[z];
    gs.beta[z] = g.beta[z];
  }
  auto go = [&](auto kern) {
    kern<<<grid, dim3(256), 0, s>>>(bs, wtn, wtk, nw, p, ns, gs, N1, N2, gtn, gblocks);
    return hipGetLastError();
  };
  const bool sv = pair_rows_vec(p), gv = gram_batch_vec(g);
  if (sv) return gv ? go(k_pair_prep<true, true>) : go(k_pair_prep<true, false>);
  return gv ? go(k_pair_prep<false, true>) : go(k_pair_prep<false, false>);
}

// ------------------------------------------------------------------------------ backward
using CfgPair = TileCfg<128, 128, 32, 64, 32>;      // 8 waves, two workgroups per CU
using CfgPairBig = TileCfg<256, 128, 32, 64, 64>;   // 8 waves, one workgroup per CU
using CfgPairSmall = TileCfg<64, 64, 32, 32, 32>;   // 4 waves

// The product is formed transposed, rows n of W_l^T by columns r of G_l, so that a lane holds four
// consecutive n of one row r of the result: 16-byte stores.  Tiles: the row tiles in groups of 8 with
// all their n tiles, in contiguous ranges per XCD, so the workgroups in flight on an XCD share few
// panels of both operands.
template <class Cfg, int NSTAGE>
__global__ void __launch_bounds__(Cfg::THREADS, (Cfg::BM == 256 ? 1 : 2) * Cfg::THREADS / 256)
k_pair_bwd(PairBwd p, int tiles_n, int tiles_r) {
  extern __shared__ float smem[];
  int blk;
  if (!xcd_block(blockIdx.x, tiles_n * tiles_r, blk)) return;
  constexpr int GR = 8;
  const int gi = blk / (GR * tiles_n), first = gi * GR, gr = min(GR, tiles_r - first);
  const int rem = blk - gi * GR * tiles_n;
  const int tr = first + rem % gr, tn = rem / gr;
  const int n0 = tn * Cfg::BM, r0 = tr * Cfg::BN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn0 = (wave / Cfg::WAVES_N) * Cfg::WM, wr0 = (wave % Cfg::WAVES_N) * Cfg::WN;
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  pair_mainloop<Cfg, NSTAGE>(p.W, p.Kp, p.N, p.G, p.Kp, p.R, n0, r0, 0, p.Kp, smem, acc);
  const int h4 = 4 * (lane >> 5);
#pragma unroll
  for (int j = 0; j < Cfg::FN; ++j) {
    const int r = r0 + wr0 + j * 32 + (lane & 31);
    const int rc = min(r, p.R - 1);
    const float* __restrict__ d = p.dphi + (long long)p.fO.div(rc) * p.N;
    float* __restrict__ o = p.out + (long long)rc * p.ldo;
    const int er = p.exps_in[rc];
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n0 + wn0 + i * 32 + 8 * q + h4;   // this lane holds n .. n + 3
        if (n >= p.N) continue;
        if (p.vec) {   // N % 4 == 0 and aligned
          const f32x4 dv = *reinterpret_cast<const f32x4*>(d + n);
          const int4 e4 = *reinterpret_cast<const int4*>(p.wexps + n);
          const f32x4 v = {ldexpf(acc[i][j][4 * q] * dv[0], er + e4.x), ldexpf(acc[i][j][4 * q + 1] * dv[1], er + e4.y),
                           ldexpf(acc[i][j][4 * q + 2] * dv[2], er + e4.z),
                           ldexpf(acc[i][j][4 * q + 3] * dv[3], er + e4.w)};
          if (r < p.R) *reinterpret_cast<f32x4*>(o + n) = v;
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int nc = min(n + k, p.N - 1);
            const float v = ldexpf(acc[i][j][4 * q + k] * d[nc], er + p.wexps[nc]);
            if (r < p.R && n + k < p.N) o[n + k] = v;
          }
        }
      }
  }
}

static bool pair_bwd_big(int R, int N, int num_cu) {
  return (long long)cdiv(R, CfgPair::BN) * cdiv(N, CfgPair::BM) >= num_cu;
}
static bool pair_bwd_huge(int R, int N, int num_cu) {
  return (long long)cdiv(R, CfgPairBig::BN) * cdiv(N, CfgPairBig::BM) >= num_cu;
}

hipError_t launch_pair_bwd(hipStream_t s, PairBwd p, int num_cu) {
  if (p.R <= 0 || p.N <= 0 || p.Kp <= 0) return hipSuccess;
  if (!dma_span_ok(p.Kp, p.Kp, 256)) return hipErrorInvalidValue;
  p.vec = p.N % 4 == 0 && vec_ok(p.dphi, p.N, p.N) && vec_ok(p.out, p.ldo, p.N) &&
          (reinterpret_cast<uintptr_t>(p.wexps) & 15) == 0;
  auto go = [&](auto cfg_tag, auto stage_tag) -> hipError_t {
    using Cfg = decltype(cfg_tag);
    constexpr int NSTAGE = decltype(stage_tag)::value;
    const int tn = cdiv(p.N, Cfg::BM), tr = cdiv(p.R, Cfg::BN);
    constexpr int bytes = NSTAGE * (Cfg::BM + Cfg::BN) * 32 * 4;
    hipError_t e = hipFuncSetAttribute((const void*)k_pair_bwd<Cfg, NSTAGE>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    k_pair_bwd<Cfg, NSTAGE><<<dim3(8 * cdiv((long long)tn * tr, 8)), dim3(Cfg::THREADS), bytes, s>>>(p, tn, tr);
    return hipGetLastError();
  };
  if (pair_bwd_huge(p.R, p.N, num_cu)) return go(CfgPairBig{}, std::integral_constant<int, 3>{});
  if (pair_bwd_big(p.R, p.N, num_cu)) return go(CfgPair{}, std::integral_constant<int, 2>{});
  // Few tiles are bound by the latency of their loads: the more K tiles in flight the better, as
  // far as the LDS of a CU holds the workgroups it is given
  const long long tiles = (long long)cdiv(p.R, CfgPairSmall::BN) * cdiv(p.N, CfgPairSmall::BM);
  if (tiles <= num_cu) return go(CfgPairSmall{}, std::integral_constant<int, 8>{});
  if (tiles <= 2LL * num_cu) return go(CfgPairSmall{}, std::integral_constant<int, 4>{});
  return go(CfgPairSmall{}, std::integral_constant<int, 2>{});
}

}  // namespace ntk
