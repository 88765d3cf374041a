// kernels_pair.hip -- the cotangent backward of a fully-connected net on pair rows (pair_core.hpp):
// fp32 products on the f16 matrix cores.
//
//   k_pair_weights  rows of W_l^T as pair rows, one launch for all layers
//   k_pair_seed     the readout cotangents Wr[o, c] act'(z[n, c]) as pair rows
//   k_pair_bwd      G_{l-1} = (G_l W_l) * act'(z_{l-1}), pair rows in, pair rows (or fp32) out
//
// Exponents.  A row's exponent has to be known before its elements are rounded to pairs, while
// the row is written by many workgroups.  k_pair_bwd therefore scales by a bound that every
// workgroup of a row can form alone,
//   |G_{l-1}[r, n]| <= max_k |G_l[r, k]| * max_n sum_k |W_l[k, n]| * max |act'|,
// with the true largest element of row r of G_l (each workgroup stores its tile's row maxima) and
// the largest column sum of W_l (from k_pair_weights).  For random signs the bound lies a factor
// of about sqrt(K) above the elements (2^6 to 2^8 at the widths in use), which the f16 pairs hold
// at full precision (2^18 below the row's largest possible value; pair_core.hpp).
#include "gram_small.hpp"
#include "launch.hpp"
#include "pair_core.hpp"

namespace ntk {

static inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------------------------------------ weights
// Two launches over all layers: column maxima and sums of magnitudes of 64-column strips by
// chunks of kWChunk rows, then 64 x 64 tiles transposed through LDS, 32 bytes (8 k of hi and of
// lo) per thread and step.  Bound by memory: W is read twice and written once.
constexpr int kWChunk = 128;
// up to this many k a weight tile reads its whole column strip for the statistics itself
constexpr int kPairPrepK = 1024;
// layers of the one-launch form (its batches are kernel arguments)
constexpr int kPrepLayers = 12;
__global__ void __launch_bounds__(256) k_pair_wstats(PairWeights b) {
  __shared__ float red[2][4][64];
  const int z = blockIdx.z;
  const int K = b.K[z], N = b.N[z];
  const int n0 = blockIdx.x * kPairStrip, k0 = blockIdx.y * kWChunk;
  if (n0 >= N || k0 >= K) return;
  const int c = threadIdx.x & 63, kr = threadIdx.x >> 6;
  const float* __restrict__ W = b.W[z] + min(n0 + c, N - 1);
  float m = 0.f, sum = 0.f;
#pragma unroll
  for (int i = 0; i < kWChunk / 4; ++i) {
    const int k = k0 + kr + 4 * i;
    const float v = fabsf(W[(long long)min(k, K - 1) * N]);
    m = fmaxf(m, k < K ? v : 0.f);
    sum += k < K ? v : 0.f;
  }
  red[0][kr][c] = m;
  red[1][kr][c] = sum;
  __syncthreads();
  if (threadIdx.x < 64 && n0 + c < N) {
#pragma unroll
    for (int i = 1; i < 4; ++i) {
      m = fmaxf(m, red[0][i][c]);
      sum += red[1][i][c];
    }
    float* st = b.stats[z] + (long long)blockIdx.y * 2 * N + n0 + c;
    st[0] = m;
    st[N] = sum;
  }
}

// One 64 x 64 tile (columns n0.., rows k0..) of W_z, 256 threads.  OWN: the column statistics are
// formed here from all of K (small layers, one launch) instead of read from k_pair_wstats.
struct PairWeightsLds {
  int ex[64];
  float red[2][4][64];
  float tile[64][65];
};
template <bool OWN, class PW>
__device__ __forceinline__ void pair_weights_tile(const PW& b, int z, int nt, int kt, PairWeightsLds& lds) {
  const int K = b.K[z], N = b.N[z];
  const int n0 = nt * kPairStrip, k0 = kt * 64;
  const int ldo = (int)pair_stride(K);
  if (n0 >= N || k0 >= ldo) return;
  const int c = threadIdx.x & 63, kr = threadIdx.x >> 6;
  const float* __restrict__ W = b.W[z] + min(n0 + c, N - 1);
  float v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = W[(long long)min(k0 + kr + 4 * i, K - 1) * N];
  float m = 0.f, sum = 0.f;
  if (OWN) {
    // 32 loads in flight, from clamped addresses
    for (int k = kr; k < K; k += 128) {
      float x[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) x[i] = W[(long long)min(k + 4 * i, K - 1) * N];
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const float a = k + 4 * i < K ? fabsf(x[i]) : 0.f;
        m = fmaxf(m, a);
        sum += a;
      }
    }
    lds.red[0][kr][c] = m;
    lds.red[1][kr][c] = sum;
    __syncthreads();
  }
  if (threadIdx.x < 64) {
    if (OWN) {
#pragma unroll
      for (int i = 1; i < 4; ++i) {
        m = fmaxf(m, lds.red[0][i][c]);
        sum += lds.red[1][i][c];
      }
    } else {
      const float* st = b.stats[z] + min(n0 + c, N - 1);
      for (int i = 0; i < (K + kWChunk - 1) / kWChunk; ++i) {
        m = fmaxf(m, st[(long long)i * 2 * N]);
        sum += st[(long long)i * 2 * N + N];
      }
    }
    const int e = pair_exp(m) - kPairTop;
    lds.ex[c] = e;
    if (kt == 0) {
      if (n0 + c < N) b.exps[z][n0 + c] = e;
#pragma unroll
      for (int o = 32; o; o >>= 1) sum = fmaxf(sum, __shfl_xor(sum, o));
      if (c == 0) b.l1[z][nt] = sum;
    }
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
        pair_split(ldexpf(lds.tile[8 * g + j][rn], -lds.ex[rn]), x, y);
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
  pair_weights_tile<false>(b, blockIdx.z, blockIdx.x, blockIdx.y, lds);
}

long long pair_stats_floats(long long K, long long N) { return (K + kWChunk - 1) / kWChunk * 2 * N; }

hipError_t launch_pair_weights(hipStream_t s, const PairWeights& b) {
  if (b.count <= 0) return hipSuccess;
  if (b.count > kMaxLayers) return hipErrorInvalidValue;
  int maxN = 0, maxK = 0;
  for (int z = 0; z < b.count; ++z) {
    maxN = std::max(maxN, b.N[z]);
    maxK = std::max(maxK, b.K[z]);
  }
  if (cdiv(maxK, 64) > 65535) return hipErrorInvalidValue;
  k_pair_wstats<<<dim3(cdiv(maxN, kPairStrip), cdiv(maxK, kWChunk), b.count), dim3(256), 0, s>>>(b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_pair_weights<<<dim3(cdiv(maxN, kPairStrip), cdiv(pair_stride(maxK), 64), b.count), dim3(256), 0, s>>>(b);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------ seed
// One wave per row r = (n, o): the row's true maximum first, then the pair rows (Wr and act' come
// from the caches the second time).  Bound by the write of the rows.
template <bool VEC>
__device__ __forceinline__ void seed_group(const float* __restrict__ w, const float* __restrict__ d, int k0, int K,
                                           float (&v)[8]) {
  if (VEC) {   // K % 8 == 0 and aligned rows
    const f32x4 w0 = *reinterpret_cast<const f32x4*>(w + k0), w1 = *reinterpret_cast<const f32x4*>(w + k0 + 4);
    const f32x4 d0 = *reinterpret_cast<const f32x4*>(d + k0), d1 = *reinterpret_cast<const f32x4*>(d + k0 + 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = w0[j] * d0[j];
      v[4 + j] = w1[j] * d1[j];
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = min(k0 + j, K - 1);
      const float x = w[k] * d[k];
      v[j] = k0 + j < K ? x : 0.f;
    }
  }
}

// rows 4 bx .. 4 bx + 3, one per wave (256 threads)
template <bool VEC>
__device__ __forceinline__ void pair_seed_rows(const float* __restrict__ Wr, const float* __restrict__ dphi, int R,
                                               FastDiv fO, int K, float* __restrict__ out, int* __restrict__ exps,
                                               float* __restrict__ rmax, int bx) {
  const int lane = threadIdx.x & 63;
  const int r = bx * 4 + (threadIdx.x >> 6);
  if (r >= R) return;
  const int n = (int)fO.div(r), o = r - n * (int)fO.d;
  const float* __restrict__ w = Wr + (long long)o * K;
  const float* __restrict__ d = dphi + (long long)n * K;
  const int Kp = (int)pair_stride(K);
  float m = 0.f;
#pragma unroll 4
  for (int k0 = 8 * lane; k0 < K; k0 += 512) {
    float v[8];
    seed_group<VEC>(w, d, k0, K, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf(v[j]));
  }
#pragma unroll
  for (int q = 32; q; q >>= 1) m = fmaxf(m, __shfl_xor(m, q));
  const int e = pair_exp(m) - kPairTop;
  if (lane == 0) {
    exps[r] = e;
    rmax[r] = ldexpf(m, -e);
  }
#pragma unroll 4
  for (int k0 = 8 * lane; k0 < Kp; k0 += 512) {
    float v[8];
    if (VEC && k0 >= K) {   // the padding
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = 0.f;
    } else {
      seed_group<VEC>(w, d, k0, K, v);
    }
    f16x8 hi, lo;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      _Float16 x, y;
      pair_split(ldexpf(v[j], -e), x, y);
      hi[j] = x;
      lo[j] = y;
    }
    f16x8* p = reinterpret_cast<f16x8*>(out + (long long)r * Kp + k0);
    p[0] = hi;
    p[1] = lo;
  }
}

template <bool VEC>
__global__ void __launch_bounds__(256)
k_pair_seed(const float* __restrict__ Wr, const float* __restrict__ dphi, int R, FastDiv fO, int K,
            float* __restrict__ out, int* __restrict__ exps, float* __restrict__ rmax) {
  pair_seed_rows<VEC>(Wr, dphi, R, fO, K, out, exps, rmax, blockIdx.x);
}

static bool pair_seed_vec(const float* Wr, const float* dphi, int K) {
  return K % 8 == 0 && vec_ok(Wr, K, K) && vec_ok(dphi, K, K);
}

hipError_t launch_pair_seed(hipStream_t s, const float* Wr, const float* dphi, int R, int O, int K, float* out,
                            int* exps, float* rmax) {
  if (R <= 0 || K <= 0) return hipSuccess;
  if (O <= 0) return hipErrorInvalidValue;
  const FastDiv fO((uint32_t)O);
  if (pair_seed_vec(Wr, dphi, K))
    k_pair_seed<true><<<dim3(cdiv(R, 4)), dim3(256), 0, s>>>(Wr, dphi, R, fO, K, out, exps, rmax);
  else
    k_pair_seed<false><<<dim3(cdiv(R, 4)), dim3(256), 0, s>>>(Wr, dphi, R, fO, K, out, exps, rmax);
  return hipGetLastError();
}

// Small problems: the weights' pair rows, the seed and the Grams in one launch (each alone leaves
// most of the chip idle and costs a launch): the first nw workgroups take 64 x 64 weight tiles,
// the next ns the seed's rows, the others the 16 x 16 Gram blocks (gblocks per layer input).
template <bool SVEC, bool GVEC>
__global__ void __launch_bounds__(256)
k_pair_prep(PairWeightsT<kPrepLayers> b, int wtn, int wtk, int nw, const float* __restrict__ Wr, const float* __restrict__ dphi,
            int R, FastDiv fO, int K, float* __restrict__ out, int* __restrict__ exps, float* __restrict__ rmax,
            int ns, GramBatchT<kPrepLayers + 1> g, int N1, int N2, int gtiles_n, int gblocks) {
  __shared__ union {
    PairWeightsLds w;
    double red[4][256];
  } lds;
  int bx = blockIdx.x;
  if (bx < nw) {
    const int z = bx / (wtn * wtk);
    bx -= z * wtn * wtk;
    pair_weights_tile<true>(b, z, bx % wtn, bx / wtn, lds.w);
  } else if (bx - nw < ns) {
    pair_seed_rows<SVEC>(Wr, dphi, R, fO, K, out, exps, rmax, bx - nw);
  } else {
    bx -= nw + ns;
    gram_small_block<GVEC>(g, N1, N2, gtiles_n, bx % gblocks, bx / gblocks, lds.red);
  }
}

hipError_t launch_pair_prep(hipStream_t s, const PairWeights& b, const float* Wr, const float* dphi, int R, int O, int K,
                            float* out, int* exps, float* rmax, const GramBatch& g, int N1, int N2, int num_cu) {
  if (R <= 0 || K <= 0 || O <= 0) return hipErrorInvalidValue;
  int maxN = 0, maxK = 0;
  for (int z = 0; z < b.count; ++z) {
    maxN = std::max(maxN, b.N[z]);
    maxK = std::max(maxK, b.K[z]);
  }
  if (maxK > kPairPrepK || b.count > kPrepLayers || g.count > kPrepLayers + 1 || !gram_small_fits(g, N1, N2, num_cu)) {
    hipError_t e = launch_pair_weights(s, b);
    if (e == hipSuccess) e = launch_pair_seed(s, Wr, dphi, R, O, K, out, exps, rmax);
    return e != hipSuccess ? e : launch_gram(s, g, N1, N2, num_cu);
  }
  const int wtn = cdiv(maxN, kPairStrip), wtk = b.count ? cdiv(pair_stride(maxK), 64) : 0;
  const int nw = wtn * wtk * b.count, ns = cdiv(R, 4);
  const int gtn = cdiv(N2, 16), gblocks = cdiv(N1, 16) * gtn;
  const dim3 grid((unsigned)(nw + ns + gblocks * g.count));
  PairWeightsT<kPrepLayers> bs{};
  bs.count = b.count;
  for (int z = 0; z < b.count; ++z) {
    bs.W[z] = b.W[z];
    bs.out[z] = b.out[z];
    bs.exps[z] = b.exps[z];
    bs.l1[z] = b.l1[z];
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
    kern<<<grid, dim3(256), 0, s>>>(bs, wtn, wtk, nw, Wr, dphi, R, FastDiv((uint32_t)O), K, out, exps, rmax, ns, gs,
                                    N1, N2, gtn, gblocks);
    return hipGetLastError();
  };
  const bool sv = pair_seed_vec(Wr, dphi, K), gv = gram_batch_vec(g);
  if (sv) return gv ? go(k_pair_prep<true, true>) : go(k_pair_prep<true, false>);
  return gv ? go(k_pair_prep<false, true>) : go(k_pair_prep<false, false>);
}

// ------------------------------------------------------------------------------ backward
using CfgPair = TileCfg<128, 128, 32, 64, 32>;      // 8 waves, two workgroups per CU
using CfgPairBig = TileCfg<256, 128, 32, 64, 64>;   // 8 waves, one workgroup per CU
using CfgPairSmall = TileCfg<64, 64, 32, 32, 32>;   // 4 waves

// The product is formed transposed, rows n of W_l^T by columns r of G_l, so that a lane holds four
// consecutive n of one row r of the result: 8-byte stores of hi and of lo into its pair row.
// Tiles: the row tiles in groups of 8 with all their n tiles, in contiguous ranges per XCD, so
// the workgroups in flight on an XCD share few panels of both operands.
template <class Cfg, int NSTAGE>
__global__ void __launch_bounds__(Cfg::THREADS, (Cfg::BM == 256 ? 1 : 2) * Cfg::THREADS / 256)
k_pair_bwd(PairBwd p, int tiles_n, int tiles_r) {
  extern __shared__ float smem[];
  constexpr int LOOP = NSTAGE * (Cfg::BM + Cfg::BN) * 32;
  int* sc = reinterpret_cast<int*>(smem + LOOP);          // per row of the tile: the scaling exponent
  float* sr = smem + LOOP + Cfg::BN;                      // per wave row and row: the tile's row maxima
  float* sl = sr + Cfg::WAVES_M * Cfg::BN;                // per wave: the largest column sum
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
  // exponents: the largest column sum of W, the row's largest element, and their sum
  float l1 = 0.f;
  for (int i = threadIdx.x; i < p.l1_parts; i += Cfg::THREADS) l1 = fmaxf(l1, p.l1[i]);
#pragma unroll
  for (int q = 32; q; q >>= 1) l1 = fmaxf(l1, __shfl_xor(l1, q));
  if (lane == 0) sl[wave] = l1;
  float m = 0.f;
  const int rr = min(r0 + (int)threadIdx.x, p.R - 1);
  if (threadIdx.x < Cfg::BN)
    for (int i = 0; i < p.rmax_parts; ++i) m = fmaxf(m, p.rmax_in[(long long)i * p.rmax_ld + rr]);
  __syncthreads();
  if (threadIdx.x < Cfg::BN) {
#pragma unroll
    for (int w = 0; w < Cfg::WAVES; ++w) l1 = fmaxf(l1, sl[w]);
    const int c = kPairTop - pair_exp(m) - pair_exp(l1) - p.act_exp;
    sc[threadIdx.x] = c;
    if (tn == 0 && r0 + (int)threadIdx.x < p.R) p.exps_out[r0 + threadIdx.x] = p.exps_in[r0 + threadIdx.x] - c;
  }
  __syncthreads();
  const int h4 = 4 * (lane >> 5);
  const int Np = (int)pair_stride(p.N);
#pragma unroll
  for (int j = 0; j < Cfg::FN; ++j) {
    const int lr = wr0 + j * 32 + (lane & 31);
    const int r = r0 + lr;
    const int rc = min(r, p.R - 1);
    const int c = sc[lr];
    const float* __restrict__ d = p.dphi + (long long)p.fO.div(rc) * p.N;
    const int eo = p.exps_in[rc] - c;
    float mx = 0.f;
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nb = n0 + wn0 + i * 32 + 8 * q;   // the group of 8 n; this lane holds nb + h4 ..
        const int n = nb + h4;
        if (nb < Np) {
          f32x4 dv;
          int tv[4];
          if (p.vec) {   // N % 4 == 0 and aligned: the four n are all in or all past the end
            const int nc = min(n, p.N - 4);
            dv = *reinterpret_cast<const f32x4*>(d + nc);
            const int4 t4 = *reinterpret_cast<const int4*>(p.wexps + nc);
            tv[0] = t4.x;
            tv[1] = t4.y;
            tv[2] = t4.z;
            tv[3] = t4.w;
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              dv[k] = d[min(n + k, p.N - 1)];
              tv[k] = p.wexps[min(n + k, p.N - 1)];
            }
          }
          f16x4 hi, lo;
          f32x4 f;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float v = n + k < p.N ? ldexpf(acc[i][j][4 * q + k] * dv[k], tv[k] + c) : 0.f;
            mx = fmaxf(mx, fabsf(v));
            _Float16 x, y;
            pair_split(v, x, y);
            hi[k] = x;
            lo[k] = y;
            f[k] = v;
          }
          if (r < p.R) {
            if (p.out) {
              f16x4* o = reinterpret_cast<f16x4*>(p.out + (long long)r * Np + nb) + (lane >> 5);
              o[0] = hi;
              o[2] = lo;
            }
            if (p.out32) {
              float* o = p.out32 + (long long)r * p.N + n;
#pragma unroll
              for (int k = 0; k < 4; ++k)
                if (n + k < p.N) o[k] = ldexpf(f[k], eo);
            }
          }
        }
      }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (lane < 32) sr[(wave / Cfg::WAVES_N) * Cfg::BN + lr] = mx;
  }
  __syncthreads();
  if (threadIdx.x < Cfg::BN && r0 + (int)threadIdx.x < p.R) {
    float x = sr[threadIdx.x];
#pragma unroll
    for (int w = 1; w < Cfg::WAVES_M; ++w) x = fmaxf(x, sr[w * Cfg::BN + threadIdx.x]);
    p.rmax_out[(long long)tn * p.rmax_ld + r0 + threadIdx.x] = x;
  }
}

static bool pair_bwd_big(int R, int N, int num_cu) {
  return (long long)cdiv(R, CfgPair::BN) * cdiv(N, CfgPair::BM) >= num_cu;
}
static bool pair_bwd_huge(int R, int N, int num_cu) {
  return (long long)cdiv(R, CfgPairBig::BN) * cdiv(N, CfgPairBig::BM) >= num_cu;
}
int pair_bwd_parts(int R, int N, int num_cu) {
  if (pair_bwd_huge(R, N, num_cu)) return cdiv(N, CfgPairBig::BM);
  return cdiv(N, pair_bwd_big(R, N, num_cu) ? CfgPair::BM : CfgPairSmall::BM);
}

hipError_t launch_pair_bwd(hipStream_t s, PairBwd p, int num_cu) {
  if (p.R <= 0 || p.N <= 0 || p.Kp <= 0) return hipSuccess;
  if (!dma_span_ok(p.Kp, p.Kp, 256)) return hipErrorInvalidValue;
  p.vec = p.N % 4 == 0 && vec_ok(p.dphi, p.N, p.N) && (reinterpret_cast<uintptr_t>(p.wexps) & 15) == 0;
  auto go = [&](auto cfg_tag, auto stage_tag) -> hipError_t {
    using Cfg = decltype(cfg_tag);
    constexpr int NSTAGE = decltype(stage_tag)::value;
    const int tn = cdiv(p.N, Cfg::BM), tr = cdiv(p.R, Cfg::BN);
    constexpr int bytes = (NSTAGE * (Cfg::BM + Cfg::BN) * 32 + Cfg::BN + Cfg::WAVES_M * Cfg::BN + Cfg::WAVES) * 4;
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
