// gram_small.hpp -- the layer-input Grams of small batches, one 16 x 16 block per workgroup; also run
// inside other kernels' launches.
#pragma once
#include "gemm_core.hpp"
#include "launch.hpp"

namespace ntk {

// Small batches: the 64 x 64 tiles of k_gram would leave most compute units idle, so workgroup
// (block, z) computes one 16 x 16 block of layer z's Gram with the 16x16x4 fp32 MFMA, its four
// waves taking every fourth 16-column slice of K; the waves' partial blocks are then added in
// wave order through LDS.  The MFMA takes A[i][k] from lane i + 16 k and B[k][j] from lane
// j + 16 k, and returns D[4 (l / 16) + v][l % 16] in register v of lane l.  Lane l loads the four
// columns k0 + 4 (l / 16) + q (q = 0..3) of row l % 16 of both operands, and MFMA q contracts
// element q of both, so the four MFMAs cover the 16 columns of the slice (in a permuted order,
// the same for both operands).  The sums of the batches of slices are added in fp64.
template <bool VEC, class GB>
__device__ __forceinline__ void gram_small_block(const GB& g, int N1, int N2, int tiles_n, int bx, int z,
                                                 double (*red)[256]) {
  const int m0 = (bx / tiles_n) * 16, n0 = (bx % tiles_n) * 16;
  const int K = g.K[z];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, kq = 4 * (lane >> 4);
  const bool va = m0 + i < N1, vb = n0 + i < N2;
  const float* __restrict__ pa = g.h1[z] + (long long)min(m0 + i, N1 - 1) * K;
  const float* __restrict__ pb = g.h2[z] + (long long)min(n0 + i, N2 - 1) * K;
  f64x4 tot = {0.0, 0.0, 0.0, 0.0};
  // batches of U slices: every load of a batch is issued before its MFMAs, from addresses
  // clamped into the rows (a column past K reads a valid element and is zeroed), so that the
  // loop body has no branch
  constexpr int U = 4;
  for (int kb = 16 * wave; kb < K; kb += 64 * U) {
    f32x4 a[U], b[U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = kb + 64 * u + kq;
      if (VEC) {   // K % 4 == 0 and 16-byte aligned rows: the 4 columns are all in or all out
        in[u] = k < K;
        const int kc = min(k, K - 4);
        a[u] = *reinterpret_cast<const f32x4*>(pa + kc);
        b[u] = *reinterpret_cast<const f32x4*>(pb + kc);
      } else {
        in[u] = true;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int kc = min(k + q, K - 1);
          const float x = pa[kc], y = pb[kc];
          a[u][q] = k + q < K ? x : 0.f;
          b[u][q] = k + q < K ? y : 0.f;
        }
      }
    }
    // keep the loads of the batch ahead of its MFMAs
    __builtin_amdgcn_sched_barrier(0);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool use_a = va && in[u], use_b = vb && in[u];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(use_a ? a[u][q] : 0.f, use_b ? b[u][q] : 0.f, acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) tot[v] += (double)acc[v];
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][(4 * (lane >> 4) + v) * 16 + i] = tot[v];
  __syncthreads();
  const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
  if (m0 + r < N1 && n0 + c < N2) {
    const double v = ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
    g.out[z][(long long)(m0 + r) * N2 + n0 + c] = (float)(v + g.beta[z]);
  }
}

inline bool gram_small_fits(const GramBatch& g, int N1, int N2, int num_cu) {
  return g.count > 0 && (long long)((N1 + 63) / 64) * ((N2 + 63) / 64) * g.count < num_cu;
}

inline bool gram_batch_vec(const GramBatch& g) {
  bool v = true;
  for (int z = 0; z < g.count; ++z) v = v && vec_ok(g.h1[z], g.K[z], g.K[z]) && vec_ok(g.h2[z], g.K[z], g.K[z]);
  return v;
}

}  // namespace ntk
