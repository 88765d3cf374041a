// kernels_conv.hip -- convolutional path of the structured-derivatives NTK on gfx950.
//
// A 3x3 SAME, stride-1 convolution z[p, c] = sum_k patch[p, k] K[c, k] has a
// Jacobian dz/dK that is constant-block diagonal along the output channel (the
// appendix "Constant-block Diagonal" structure, C = W for a convolution), so the
// smallest sub-array to keep is the patch matrix of the layer input (appendix
// "CNN NTK Complexity": D x F*Cin per sample, formed here implicitly inside the
// GEMM loaders).  The kernels compute
//   * the forward pass keeping every layer input and act'(z) (fp64 accumulation, as
//     for dense layers, so ReLU decisions are a function of the fp32-stored input)
//   * global average pooling (the input block-tiled structure of a mean)
//   * the cotangent of the last conv pre-activation, W_d[o, c] / D * act'(z)
//   * the transposed convolution pulling the (N1+N2)*O cotangent images back one
//     layer (a SAME convolution with the spatially flipped, channel-transposed kernel)
//   * the outside-in weight-sharing contraction: per sample and layer the weight-space
//     cotangent J[(n,o),(c,k)] = sum_p G[n,o,p,c] patch[n,p,k]
//   * J1 J2^T with a deterministic split over K, then a reduction adding the readout
//     summand (g1.g2) delta_{o1 o2} and writing theta[n1][n2][o1][o2].
#include <type_traits>

#include "gemm_core.hpp"
#include "launch_conv.hpp"
#include "pair_core.hpp"

namespace ntk {

using CfgConvF64 = TileCfg<64, 64, 32, 32, 32>;    // forward, fp64 MFMA
using CfgConv = TileCfg<128, 64, 32, 32, 32>;      // backward / wgrad, fp32 MFMA: 8 waves
// direct-to-LDS backward and weight-space cotangent kernels: tiles and LDS stages.  The
// backward takes 256-row tiles with a 32x64 block per wave (two independent accumulators per
// wave) and two stages (80 KB: two workgroups per CU); the weight-space product keeps 128x64
// tiles and two stages (48 KB: three workgroups per CU).  Both measured best among 128/256-row
// tiles, 4/8 waves and 2/3 stages at the CNN workload.
using CfgConvBwd = TileCfg<256, 64, 32, 32, 64>;
using CfgConvWg = CfgConv;
using CfgConvWgSmall = TileCfg<64, 64, 32, 32, 32>;   // one-output rows (O C <= 64): 4 waves
constexpr int kConvBwdStages = 2, kConvWgStages = 2;
// the same on pairs (three f16 MFMAs): 64-wide wave tiles, so that a fragment is split into pairs
// and read from LDS for at least two of the other operand
using CfgConvBwdPair = TileCfg<256, 64, 32, 64, 64>;       // 4 waves
using CfgConvBwdPairN = TileCfg<256, 32, 32, 64, 32>;      // at most 32 input channels
using CfgConvBwdPairSmall = TileCfg<128, 64, 32, 32, 64>;
using CfgConvBwdPairSmallN = TileCfg<128, 32, 32, 32, 32>;
using CfgConvWgPair = TileCfg<128, 128, 32, 64, 64>;       // 4 waves
using CfgConvWgPairN = TileCfg<128, 64, 32, 64, 32>;
using CfgConvWgPairM = TileCfg<64, 64, 32, 32, 32>;
// Small images (few output rows): below kConvFewTiles tiles of the shapes above, the backward
// takes 128x64 tiles (8 waves of 32x32) and the fp64 forward 32x32 tiles (4 waves of 16x16), so
// that the launch still spreads over the compute units.
constexpr int kConvFewTiles = 512;
using CfgConvF64Small = TileCfg<32, 32, 32, 16, 16>;
using CfgSplitK = TileCfg<128, 128, 32, 64, 64>;   // J1 J2^T partial products
using CfgSplitKDma = TileCfg<128, 128, 32, 32, 64>;  // the same, direct-to-LDS: 8 waves of 32x64

static inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }
static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <class Cfg, class LA, class LB>
static hipError_t set_smem(const void* fn) {
  constexpr int bytes = gemm_smem_bytes<Cfg, LA, LB>();
  if (bytes > 65536)
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  return hipSuccess;
}

// ------------------------------------------------------------------------------ loaders
// All loaders read from clamped in-range addresses and report per-element validity (bit j
// of `valid`); the zero fill happens at the LDS store (see TileIO).
//
// Patch matrix of an NHWC batch as a K-inner operand: row = img*D + p, p = y*W + x,
// k = (kh*3 + kw)*C + ci; the tap (kh, kw) reads pixel (y + kh - 1, x + kw - 1), zero
// outside the image.  VEC: C % 4 == 0 and x 16-byte aligned (4 k share one tap).
template <bool VEC>
struct LoadPatchesKInnerT {
  static constexpr bool K_INNER = true;
  static constexpr bool UNIFORM_VALID = VEC;   // VEC: the 4 elements are valid together
  const float* x;
  int rows, H, W, C, K;  // K = 9*C
  FastDiv fD, fW, fC;
  __device__ __forceinline__ float tap(int img, int y, int xx, int k, bool& ok) const {
    const int kc = min(k, K - 1);
    const int t = (int)fC.div(kc), ci = kc - t * C;
    const int kh = (t * 11) >> 5, kw = t - 3 * kh;  // t / 3 for t < 9
    const int yy = y + kh - 1, xq = xx + kw - 1;
    ok = k < K && yy >= 0 && yy < H && xq >= 0 && xq < W;
    const int yc = min(max(yy, 0), H - 1), xc = min(max(xq, 0), W - 1);
    return x[(((long long)img * H + yc) * W + xc) * C + ci];
  }
  // the row's pixel, computed once per tile: element offset of (img, y, x) (clamped row), y, x
  struct RowState {
    long long base;
    int y, x, ok;
  };
  __device__ __forceinline__ RowState row_state(int row) const {
    const int rc = min(row, rows - 1);
    const int img = (int)fD.div(rc), p = rc - img * (int)fD.d;
    const int y = (int)fW.div(p), xx = p - y * W;
    return {(((long long)img * H + y) * W + xx) * C, y, xx, row < rows ? 1 : 0};
  }
  // element (row, k): tap (kh, kw) = k / C reads the pixel (y + kh - 1, x + kw - 1); outside the
  // image the row's own pixel is read and masked
  __device__ __forceinline__ f32x4 load4s(const RowState& s, int k, uint32_t& valid) const {
    if (VEC) {
      const int kc = min(k, K - 4);
      const int t = (int)fC.div(kc), ci = kc - t * C;
      const int kh = (t * 11) >> 5, kw = t - 3 * kh;
      const int yy = s.y + kh - 1, xq = s.x + kw - 1;
      const bool ok = s.ok & (k < K) & ((unsigned)yy < (unsigned)H) & ((unsigned)xq < (unsigned)W);
      const int off = ok ? ((kh - 1) * W + (kw - 1)) * C + ci : ci;
      valid = ok ? 0xFu : 0u;
      return *reinterpret_cast<const f32x4*>(x + s.base + off);
    } else {
      f32x4 v;
      valid = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kc = min(k + j, K - 1);
        const int t = (int)fC.div(kc), ci = kc - t * C;
        const int kh = (t * 11) >> 5, kw = t - 3 * kh;
        const int yy = s.y + kh - 1, xq = s.x + kw - 1;
        const bool ok = s.ok && k + j < K && yy >= 0 && yy < H && xq >= 0 && xq < W;
        const long long off = ok ? (long long)((kh - 1) * W + (kw - 1)) * C : 0;
        v[j] = x[s.base + off + ci];
        valid |= ok ? (1u << j) : 0u;
      }
      return v;
    }
  }
  __device__ __forceinline__ f32x4 load4(int row, int k, uint32_t& valid) const {
    const int rc = min(row, rows - 1);
    const int img = (int)fD.div(rc), p = rc - img * (int)fD.d;
    const int y = (int)fW.div(p), xx = p - y * W;
    if (VEC) {
      const int kc = min(k, K - 4);
      const int t = (int)fC.div(kc), ci = kc - t * C;
      const int kh = (t * 11) >> 5, kw = t - 3 * kh;
      const int yy = y + kh - 1, xq = xx + kw - 1;
      const bool ok = row < rows && k < K && yy >= 0 && yy < H && xq >= 0 && xq < W;
      const int yc = min(max(yy, 0), H - 1), xc = min(max(xq, 0), W - 1);
      valid = ok ? 0xFu : 0u;
      return *reinterpret_cast<const f32x4*>(x + (((long long)img * H + yc) * W + xc) * C + ci);
    } else {
      f32x4 v;
      valid = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bool ok;
        v[j] = tap(img, y, xx, k + j, ok);
        valid |= (ok && row < rows) ? (1u << j) : 0u;
      }
      return v;
    }
  }
};

// G of one sample as a K-outer operand of the weight-space cotangent product:
// row = o*C + c, k = p;  element = G[((s*O + o)*D + p)*C + c]  (base already at sample s).
// VEC: C % 4 == 0 and g 16-byte aligned.
template <bool VEC>
struct LoadCotangentKOuterT {
  static constexpr bool K_INNER = false;
  static constexpr bool UNIFORM_VALID = VEC;
  const float* g;
  int rows, K, C, D;     // rows = O*C, K = D
  FastDiv fC;
  // offset o*D*C + c of the row block (VEC: rows row..row+3 are contiguous), once per tile
  struct RowState {
    long long off;
    int row;
  };
  __device__ __forceinline__ RowState row_state(int row) const {
    const int rc = min(row, VEC ? rows - 4 : rows - 1);
    const int o = (int)fC.div(rc), c = rc - o * C;
    return {(long long)o * D * C + c, row};
  }
  __device__ __forceinline__ f32x4 load4s(const RowState& s, int k, uint32_t& valid) const {
    if (VEC) {
      const int kc = min(k, K - 1);
      valid = (s.row < rows && k < K) ? 0xFu : 0u;
      return *reinterpret_cast<const f32x4*>(g + s.off + (long long)kc * C);
    }
    return load4(s.row, k, valid);
  }
  __device__ __forceinline__ f32x4 load4(int row, int k, uint32_t& valid) const {
    const int kc = min(k, K - 1);
    if (VEC) {
      const int rc = min(row, rows - 4);
      const int o = (int)fC.div(rc), c = rc - o * C;
      valid = (row < rows && k < K) ? 0xFu : 0u;
      return *reinterpret_cast<const f32x4*>(g + ((long long)o * D + kc) * C + c);
    } else {
      f32x4 v;
      valid = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int rc = min(row + j, rows - 1);
        const int o = (int)fC.div(rc), c = rc - o * C;
        v[j] = g[((long long)o * D + kc) * C + c];
        valid |= (row + j < rows && k < K) ? (1u << j) : 0u;
      }
      return v;
    }
  }
};

// Patch matrix of one sample as a K-outer operand: row = k (tap, ci), kdim = p.
// VEC: C % 4 == 0 and x 16-byte aligned.
template <bool VEC>
struct LoadPatchesKOuterT {
  static constexpr bool K_INNER = false;
  static constexpr bool UNIFORM_VALID = VEC;
  const float* x;        // sample base, [H, W, C]
  int rows, K, H, W, C;  // rows = 9*C, K = D
  FastDiv fW, fC;
  // the rows' tap offset (dy, dx) and first channel (VEC: 4 consecutive channels of one
  // tap), once per tile
  struct RowState {
    int dy, dx, dd, ci, row;   // dd = dy * W + dx
  };
  __device__ __forceinline__ RowState row_state(int row) const {
    const int rc = min(row, VEC ? rows - 4 : rows - 1);
    const int t = (int)fC.div(rc), ci = rc - t * C;
    const int kh = (t * 11) >> 5, kw = t - 3 * kh;
    return {kh - 1, kw - 1, (kh - 1) * W + (kw - 1), ci, row};
  }
  __device__ __forceinline__ f32x4 load4s(const RowState& s, int p, uint32_t& valid) const {
    if (VEC) {
      const int pc = min(p, K - 1);
      const int y = (int)fW.div(pc), xx = pc - y * W;
      const int yy = y + s.dy, xq = xx + s.dx;
      const bool ok = (s.row < rows) & (p < K) & ((unsigned)yy < (unsigned)H) & ((unsigned)xq < (unsigned)W);
      valid = ok ? 0xFu : 0u;
      const int q = ok ? pc + s.dd : pc;   // outside the image: the pixel itself, masked
      return *reinterpret_cast<const f32x4*>(x + (long long)q * C + s.ci);
    }
    return load4(s.row, p, valid);
  }
  __device__ __forceinline__ f32x4 load4(int row, int p, uint32_t& valid) const {
    const int pc = min(p, K - 1);
    const int y = (int)fW.div(pc), xx = pc - y * W;
    if (VEC) {
      const int rc = min(row, rows - 4);
      const int t = (int)fC.div(rc), ci = rc - t * C;
      const int kh = (t * 11) >> 5, kw = t - 3 * kh;
      const int yy = y + kh - 1, xq = xx + kw - 1;
      const bool ok = row < rows && p < K && yy >= 0 && yy < H && xq >= 0 && xq < W;
      const int yc = min(max(yy, 0), H - 1), xc = min(max(xq, 0), W - 1);
      valid = ok ? 0xFu : 0u;
      return *reinterpret_cast<const f32x4*>(x + ((long long)yc * W + xc) * C + ci);
    } else {
      f32x4 v;
      valid = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int rc = min(row + j, rows - 1);
        const int t = (int)fC.div(rc), ci = rc - t * C;
        const int kh = (t * 11) >> 5, kw = t - 3 * kh;
        const int yy = y + kh - 1, xq = xx + kw - 1;
        const bool ok = row + j < rows && p < K && yy >= 0 && yy < H && xq >= 0 && xq < W;
        const int yc = min(max(yy, 0), H - 1), xc = min(max(xq, 0), W - 1);
        v[j] = x[((long long)yc * W + xc) * C + ci];
        valid |= ok ? (1u << j) : 0u;
      }
      return v;
    }
  }
};

template <bool VEC>
static LoadPatchesKInnerT<VEC> patches_kinner(const float* x, int images, int H, int W, int C) {
  LoadPatchesKInnerT<VEC> l;
  l.x = x;
  l.rows = images * H * W;
  l.H = H;
  l.W = W;
  l.C = C;
  l.K = 9 * C;
  l.fD = FastDiv((uint32_t)(H * W));
  l.fW = FastDiv((uint32_t)W);
  l.fC = FastDiv((uint32_t)C);
  return l;
}

// Patch matrix of an NHWC batch as a direct-to-LDS operand (see DmaTile): row = img*D + p,
// column k = tap*C + ci with C % 32 == 0, so the 32 columns of a K tile lie inside one tap.
// Every lane loads 16 bytes of one row through a buffer resource over the whole batch (less
// than 2 GiB); a tap that falls outside the image (the zero padding) takes an offset past the
// resource, which reads zeros.  The rows' pixels are computed once per tile (prepare).
constexpr uint32_t kDmaPastEnd = 0x80000000u;   // past every resource: the load reads zeros

template <int ROWS, int WAVES>
struct DmaPatches {
  using Tile = DmaTile<ROWS>;
  const float* __restrict__ x;
  int rows, H, W, C;
  FastDiv fD, fW, fC;
  static constexpr int NI = ROWS / (8 * WAVES);
  template <int WV>
  static constexpr int OPS = ROWS / (8 * WV);
  __amdgpu_buffer_rsrc_t rsrc;
  // per issued row: the byte offset of its pixel's 16-byte chunk (channel block 0) through a
  // resource that starts W + 1 pixels before the batch, so that every tap's shift is a
  // non-negative uniform offset (the scalar offset of the load), and a 9-bit mask, bit t set
  // when tap t of the pixel lies OUTSIDE the image (all set for rows past the end).  An issue
  // is then a bit extract and a shift-or: the offset with bit 31 set is past the resource's end
  // (base4 + the largest tap offset stays below 2^31), which loads zeros.
  int base4[NI];
  unsigned omask[NI];
  __device__ __forceinline__ void prepare(int row0, int wave, int lane) {
    rsrc = buffer_rsrc(x - (long long)(W + 1) * C, (uint32_t)((long long)(rows + 2 * (W + 1)) * C * 4));
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = (i * WAVES + wave) * 8 + (lane >> 3);
      const int row = row0 + r;
      const int rc = min(row, rows - 1);
      const int img = (int)fD.div(rc), p = rc - img * (int)fD.d;
      const int yy = (int)fW.div(p), xq = p - yy * W;
      const int c = DmaTile<ROWS>::swz(r, lane & 7);   // global chunk stored at lane & 7
      base4[i] = (((img * H + yy) * W + xq) * C + 4 * c) * 4;
      // opaque: the compiler would otherwise re-derive the offset from its factors at every
      // issue (a 64-bit multiply-add and three more instructions per row)
      asm volatile("" : "+v"(base4[i]));
      unsigned m = 0;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int ky = yy + t / 3 - 1, kx = xq + t % 3 - 1;
        m |= ((unsigned)ky < (unsigned)H && (unsigned)kx < (unsigned)W) ? 0u : (1u << t);
      }
      omask[i] = row < rows ? m : 0x1FFu;
    }
  }
  template <int WV>
  __device__ __forceinline__ void issue(int k0, float* lds, int wave, int lane) const {
    static_assert(WV == WAVES, "issuer built for this workgroup shape");
    const int t = (int)fC.div(k0), cb = k0 - t * C;
    const int kh = (t * 11) >> 5, kw = t - 3 * kh;
    const uint32_t soff = (uint32_t)(((kh * W + kw) * C + cb) * 4);   // uniform, >= 0
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r0 = (i * WAVES + wave) * 8;
      const uint32_t voff = (((omask[i] >> t) & 1u) << 31) | (uint32_t)base4[i];
      buffer_dma16(rsrc, voff, soff, lds + __builtin_amdgcn_readfirstlane(r0 * DmaTile<ROWS>::BK));
    }
  }
};

template <int ROWS, int WAVES>
static DmaPatches<ROWS, WAVES> dma_patches(const float* x, int images, int H, int W, int C) {
  DmaPatches<ROWS, WAVES> d;
  d.x = x;
  d.rows = images * H * W;
  d.H = H;
  d.W = W;
  d.C = C;
  d.fD = FastDiv((uint32_t)(H * W));
  d.fW = FastDiv((uint32_t)W);
  d.fC = FastDiv((uint32_t)C);
  return d;
}

// The direct-to-LDS path needs C % 32 == 0, 16-byte aligned operands, an activation batch of
// `elems` floats (images of width W) and weight tiles within the buffer-resource span; the
// patch resource spans the batch and W + 1 pixels on either side.
static bool conv_dma_ok(const void* x, long long elems, int W, int C, const void* K) {
  return C % 32 == 0 && aligned16(x) && aligned16(K) && (elems + 2LL * (W + 1) * C) * 4 < (1LL << 31) &&
         dma_span_ok(9LL * C, 9LL * C, 256);
}

// K-outer direct-to-LDS operands of the weight-space cotangent product of one sample (k = the
// pixel p, 4 consecutive rows per 16-byte load, see DmaTileKOuter), through a buffer resource
// over the sample's tensor.  Each lane's (k-row, row chunk) inside the tile is fixed, so its row
// part is computed once per tile; pixels past D and padding taps read past the resource (zeros).
// G of the sample: rows (o, c) of O*C (C % 4 == 0), element G[o, p, c].
template <int ROWS, int WAVES, bool WHOLE = false>
struct DmaCotangentKOuter {
  using Tile = DmaTileKOuter<ROWS>;
  const float* __restrict__ g;
  int rows, D, C;
  FastDiv fC;
  static constexpr int NI = ROWS / (8 * WAVES);
  template <int WV>
  static constexpr int OPS = ROWS / (8 * WV);
  __amdgpu_buffer_rsrc_t rsrc;
  // per issued row: the byte offset of its 16-byte chunk at pixel kl (the K tile's first pixel
  // k0 adds the uniform k0 C 4 through the scalar offset), with bit 31 set for rows past the end
  // (past the resource's end: zeros), and the bound k0 < klim of the pixels inside the sample
  // (klim = D - kl), tested unless WHOLE (D a multiple of the K tile)
  int pre4[NI], klim[NI];
  __device__ __forceinline__ void prepare(int row0, int wave, int lane) {
    rsrc = buffer_rsrc(g, (uint32_t)((long long)rows * D * 4));
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int o = (i * WAVES + wave) * 256 + 4 * lane;     // float offset in the tile
      const int k = o / ROWS, pos = (o % ROWS) >> 2;
      const int row = row0 + 4 * Tile::swz(k, pos);
      const int rc = min(row, rows - 4);
      const int oo = (int)fC.div(rc), cc = rc - oo * C;
      pre4[i] = (int)((uint32_t)((oo * D * C + cc + k * C) * 4) | (row < rows ? 0u : kDmaPastEnd));
      asm volatile("" : "+v"(pre4[i]));   // kept whole, not re-derived at each issue
      klim[i] = D - k;
    }
  }
  template <int WV>
  __device__ __forceinline__ void issue(int k0, float* lds, int wave, int lane) const {
    static_assert(WV == WAVES, "issuer built for this workgroup shape");
    const uint32_t soff = (uint32_t)k0 * C * 4u;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      // WHOLE (D % 32 == 0): every pixel of every K tile is inside the sample
      const uint32_t voff = WHOLE ? (uint32_t)pre4[i] : ((uint32_t)pre4[i] | (k0 < klim[i] ? 0u : kDmaPastEnd));
      buffer_dma16(rsrc, voff, soff, lds + __builtin_amdgcn_readfirstlane((i * WAVES + wave) * 256));
    }
  }
};

// Patches of the sample's layer input [H, W, C] (C % 4 == 0): rows (tap, ci) of 9*C.
template <int ROWS, int WAVES, bool ROW32 = false>
struct DmaPatchesKOuter {
  using Tile = DmaTileKOuter<ROWS>;
  const float* __restrict__ x;
  int rows, K, H, W, C;   // K = D pixels
  FastDiv fW, fC;
  static constexpr int NI = ROWS / (8 * WAVES);
  template <int WV>
  static constexpr int OPS = ROWS / (8 * WV);
  __amdgpu_buffer_rsrc_t rsrc;
  // per issued row (tap (dy, dx), channel ci) at pixel kl of the K tile: the byte offset of its
  // shifted pixel kl + dy W + dx through a resource that starts W + 1 pixels before the sample
  // (so the offset is never negative; the K tile's first pixel k0 adds the uniform k0 C 4 through
  // the scalar offset), and what the tap's bounds test needs.  With ROW32 (W a multiple of the K
  // tile of 32 pixels) a K tile is a run of 32 pixels of one image row, and a row's tap is outside the
  // image exactly when one of the uniform conditions in its 5-bit mask `out` holds: bit 0 the
  // tile is the image's first row (dy = -1), bit 1 its last row (dy = 1), bit 2 the tile starts
  // an image row (kl = 0, dx = -1), bit 3 it ends one (kl = 31, dx = 1), bit 4 always (rows past
  // the end).
  int base4[NI], kl[NI], dy[NI], dx[NI], ok[NI];
  unsigned out[NI];
  __device__ __forceinline__ void prepare(int row0, int wave, int lane) {
    rsrc = buffer_rsrc(x - (long long)(W + 1) * C, (uint32_t)((long long)(K + W + 1) * C * 4));
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int o = (i * WAVES + wave) * 256 + 4 * lane;
      const int k = o / ROWS, pos = (o % ROWS) >> 2;
      const int row = row0 + 4 * Tile::swz(k, pos);
      const int rc = min(row, rows - 4);
      const int t = (int)fC.div(rc);
      const int kh = (t * 11) >> 5, kw = t - 3 * kh;
      const int ci = rc - t * C;
      kl[i] = k;
      dy[i] = kh - 1;
      dx[i] = kw - 1;
      base4[i] = ((k + (kh - 1) * W + (kw - 1) + W + 1) * C + ci) * 4;
      asm volatile("" : "+v"(base4[i]));   // kept whole, not re-derived at each issue
      ok[i] = row < rows ? 1 : 0;
      out[i] = (kh == 0 ? 1u : 0u) | (kh == 2 ? 2u : 0u) | (k == 0 && kw == 0 ? 4u : 0u) |
               (k == 31 && kw == 2 ? 8u : 0u) | (row < rows ? 0u : 16u);
    }
  }
  template <int WV>
  __device__ __forceinline__ void issue(int k0, float* lds, int wave, int lane) const {
    static_assert(WV == WAVES, "issuer built for this workgroup shape");
    const uint32_t soff = (uint32_t)k0 * C * 4u;
    if constexpr (ROW32) {
      const int y0 = (int)fW.div(k0), x0 = k0 - y0 * W;   // uniform
      const unsigned bad = (y0 == 0 ? 1u : 0u) | (y0 == H - 1 ? 2u : 0u) | (x0 == 0 ? 4u : 0u) |
                           (x0 + 32 == W ? 8u : 0u) | 16u;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t voff = (uint32_t)base4[i] | ((out[i] & bad) ? kDmaPastEnd : 0u);
        buffer_dma16(rsrc, voff, soff, lds + __builtin_amdgcn_readfirstlane((i * WAVES + wave) * 256));
      }
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
      const int p = k0 + kl[i];
      const int pc = min(p, K - 1);
      const int y = (int)fW.div(pc), xx = pc - y * W;
      const bool good = ok[i] & (p < K) & ((unsigned)(y + dy[i]) < (unsigned)H) & ((unsigned)(xx + dx[i]) < (unsigned)W);
      const uint32_t voff = good ? (uint32_t)base4[i] : kDmaPastEnd;
      buffer_dma16(rsrc, voff, soff, lds + __builtin_amdgcn_readfirstlane((i * WAVES + wave) * 256));
      }
    }
  }
};

// ------------------------------------------------------------------------------ forward
template <class Cfg>
__device__ __forceinline__ void conv_fwd_epilogue(f64x4 (&acc)[Cfg::FM16][Cfg::FN16], int m0, int n0,
                                                  int M, int N, int act, const float* __restrict__ bias,
                                                  float* __restrict__ hn, float* __restrict__ dphi) {
  for_each_acc<Cfg>(acc, m0, n0, [&](int r, int c, double z) {
    if (bias) z += (double)bias[min(c, N - 1)];
    float h, d;
    if (act == 1) {
      h = z > 0.0 ? (float)z : 0.f;
      d = z > 0.0 ? 1.f : 0.f;
    } else {
      const float zf = (float)z;
      h = act_fwd(act, zf);
      d = act_deriv(act, zf);
    }
    if (r < M && c < N) {
      hn[(long long)r * N + c] = h;
      dphi[(long long)r * N + c] = d;
    }
  });
}

// direct-to-LDS form (C % 32 == 0): patches gathered by the DMA, three LDS stages
template <class Cfg>
__global__ void __launch_bounds__(Cfg::THREADS)
k_conv_fwd_dma(DmaPatches<Cfg::BM, Cfg::WAVES> pa, DmaRowMajor<Cfg::BN, Cfg::WAVES> pb, int K, int M, int N, int act,
               const float* __restrict__ bias, float* __restrict__ hn, float* __restrict__ dphi, int tiles_n) {
  extern __shared__ float smem[];
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  f64x4 acc[Cfg::FM16][Cfg::FN16];
  zero_acc<Cfg>(acc);
  gemm_mainloop_dma_ops<Cfg, 3>(pa, pb, m0, n0, 0, K, smem, acc);
  conv_fwd_epilogue<Cfg>(acc, m0, n0, M, N, act, bias, hn, dphi);
}

template <class Cfg, bool VEC>
__global__ void __launch_bounds__(Cfg::THREADS)
k_conv_fwd(LoadPatchesKInnerT<VEC> la, LoadKInnerT<VEC> lb, int M, int N, int act,
           const float* __restrict__ bias, float* __restrict__ hn, float* __restrict__ dphi, int tiles_n) {
  extern __shared__ float smem[];
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  f64x4 acc[Cfg::FM16][Cfg::FN16];
  zero_acc<Cfg>(acc);
  gemm_mainloop<Cfg>(la, lb, m0, n0, 0, la.K, smem, acc);
  conv_fwd_epilogue<Cfg>(acc, m0, n0, M, N, act, bias, hn, dphi);
}

template <bool VEC>
static hipError_t conv_fwd_vec(hipStream_t s, const float* x, int images, int H, int W, int Cin,
                               const float* K, int Cout, int act, const float* bias, float* hn, float* dphi) {
  using Cfg = CfgConvF64;
  using LA = LoadPatchesKInnerT<VEC>;
  using LB = LoadKInnerT<VEC>;
  LA la = patches_kinner<VEC>(x, images, H, W, Cin);
  LB lb{K, Cout, 9 * Cin, 9 * Cin};
  const int M = images * H * W;
  const int tn = cdiv(Cout, Cfg::BN), tm = cdiv(M, Cfg::BM);
  hipError_t e = set_smem<Cfg, LA, LB>((const void*)k_conv_fwd<Cfg, VEC>);
  if (e != hipSuccess) return e;
  k_conv_fwd<Cfg, VEC><<<dim3(tm * tn), dim3(Cfg::THREADS), gemm_smem_bytes<Cfg, LA, LB>(), s>>>(
      la, lb, M, Cout, act, bias, hn, dphi, tn);
  return hipGetLastError();
}

template <class Cfg>
static hipError_t conv_fwd_dma_cfg(hipStream_t s, const float* x, int images, int H, int W, int Cin,
                                   const float* K, int Cout, int act, const float* bias, float* hn, float* dphi) {
  const int M = images * H * W, Kd = 9 * Cin;
  const int tn = cdiv(Cout, Cfg::BN), tm = cdiv(M, Cfg::BM);
  auto pa = dma_patches<Cfg::BM, Cfg::WAVES>(x, images, H, W, Cin);
  DmaRowMajor<Cfg::BN, Cfg::WAVES> pb{K, Kd, Cout};
  constexpr int bytes = gemm_dma_smem_bytes<Cfg, 3>();
  hipError_t e = hipFuncSetAttribute((const void*)k_conv_fwd_dma<Cfg>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  k_conv_fwd_dma<Cfg><<<dim3(tm * tn), dim3(Cfg::THREADS), bytes, s>>>(pa, pb, Kd, M, Cout, act, bias, hn, dphi, tn);
  return hipGetLastError();
}

hipError_t launch_conv_fwd(hipStream_t s, const float* x, int images, int H, int W, int Cin,
                           const float* K, int Cout, int act, const float* bias, float* hn, float* dphi) {
  if (conv_dma_ok(x, (long long)images * H * W * Cin, W, Cin, K)) {
    const long long tiles = (long long)cdiv((long long)images * H * W, CfgConvF64::BM) * cdiv(Cout, CfgConvF64::BN);
    if (tiles < kConvFewTiles)
      return conv_fwd_dma_cfg<CfgConvF64Small>(s, x, images, H, W, Cin, K, Cout, act, bias, hn, dphi);
    return conv_fwd_dma_cfg<CfgConvF64>(s, x, images, H, W, Cin, K, Cout, act, bias, hn, dphi);
  }
  if (Cin % 4 == 0 && aligned16(x) && vec_ok(K, 9 * Cin, 9 * Cin))
    return conv_fwd_vec<true>(s, x, images, H, W, Cin, K, Cout, act, bias, hn, dphi);
  return conv_fwd_vec<false>(s, x, images, H, W, Cin, K, Cout, act, bias, hn, dphi);
}

// ------------------------------------------------------------------------------ GAP, seed
// g[img, c] = mean over the D pixels of h[img, p, c]: one workgroup per image.  Generic form:
// 256 threads, lanes over channels and groups of pixels; vector form (C % 4 == 0, C / 4 dividing
// 1024, 16-byte aligned): 1024 threads, a float4 of channels per lane, groups of pixels over the
// rest.  The groups' partial sums are added in a fixed order.
__global__ void __launch_bounds__(256) k_gap(const float* __restrict__ h, int D, int C, float* __restrict__ g) {
  __shared__ float part[256];
  const int img = blockIdx.x;
  const int lanes_c = C < 256 ? C : 256;
  const int groups = 256 / lanes_c;
  const int t = threadIdx.x;
  const int grp = t / lanes_c, cl = t % lanes_c;
  for (int c0 = 0; c0 < C; c0 += lanes_c) {
    const int c = c0 + cl;
    float acc = 0.f;
    if (grp < groups && c < C)
      for (int p = grp; p < D; p += groups) acc += h[((long long)img * D + p) * C + c];
    part[t] = acc;
    __syncthreads();
    if (t < lanes_c && c0 + t < C) {
      float v = 0.f;
      for (int q = 0; q < groups; ++q) v += part[q * lanes_c + t];
      g[(long long)img * C + c0 + t] = v / (float)D;
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(1024) k_gap4(const float* __restrict__ h, int D, int C, float* __restrict__ g) {
  __shared__ float4 part[1024];
  const int img = blockIdx.x;
  const int C4 = C >> 2, groups = 1024 / C4;
  const int t = threadIdx.x, grp = t / C4, c4 = t - grp * C4;
  const float4* src = reinterpret_cast<const float4*>(h + (long long)img * D * C);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p = grp; p < D; p += groups) {
    const float4 v = src[(long long)p * C4 + c4];
    acc.x += v.x;
    acc.y += v.y;
    acc.z += v.z;
    acc.w += v.w;
  }
  part[t] = acc;
  __syncthreads();
  if (t < C4) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int q = 0; q < groups; ++q) {
      const float4 w = part[q * C4 + t];
      v.x += w.x;
      v.y += w.y;
      v.z += w.z;
      v.w += w.w;
    }
    const float d = (float)D;
    float* dst = g + (long long)img * C + 4 * t;
    dst[0] = v.x / d;
    dst[1] = v.y / d;
    dst[2] = v.z / d;
    dst[3] = v.w / d;
  }
}

hipError_t launch_gap(hipStream_t s, const float* h, int images, int D, int C, float* g) {
  if (C % 4 == 0 && C / 4 <= 1024 && 1024 % (C / 4) == 0 && aligned16(h))
    k_gap4<<<dim3(images), dim3(1024), 0, s>>>(h, D, C, g);
  else
    k_gap<<<dim3(images), dim3(256), 0, s>>>(h, D, C, g);
  return hipGetLastError();
}

// G[(img*O + o), p, c] = Wd[o, c] / D * dphi[img, p, c]; blockIdx.y = img*O + o, the x-blocks
// stride over the D*C elements of that cotangent image (no 64-bit division per element).
__global__ void __launch_bounds__(256)
k_conv_seed(const float* __restrict__ Wd, const float* __restrict__ dphi, int IO, int O, int DC, FastDiv fC,
            float inv_d, float* __restrict__ G) {
  const int C = (int)fC.d;
  for (int io = blockIdx.y; io < IO; io += gridDim.y) {
    const int img = io / O, o = io - img * O;
    const float* wrow = Wd + (long long)o * C;
    const float* drow = dphi ? dphi + (long long)img * DC : nullptr;
    float* grow = G + (long long)io * DC;
    for (int q = blockIdx.x * 256 + threadIdx.x; q < DC; q += gridDim.x * 256) {
      const int c = q - (int)fC.div(q) * C;
      grow[q] = drow ? wrow[c] * inv_d * drow[q] : wrow[c] * inv_d;
    }
  }
}

// Vector form (C % 4 == 0, 16-byte aligned): workgroup w takes image w / pb and 256 float4s of
// its [D, C] plane (pixel-block w % pb); each lane loads its float4 of dphi once and writes it,
// scaled by Wd[o, c] / D, into the O cotangent images.
__global__ void __launch_bounds__(256)
k_conv_seed4(const float* __restrict__ Wd, const float* __restrict__ dphi, int images, int O, int DC4, int C4,
             float inv_d, float* __restrict__ G) {
  const int pb = (DC4 + 255) / 256;
  for (long long w = blockIdx.x; w < (long long)images * pb; w += gridDim.x) {
    const int img = (int)(w / pb);
    const int q = (int)(w - (long long)img * pb) * 256 + threadIdx.x;   // float4 index in the plane
    if (q >= DC4) continue;
    const int c4 = q % C4;
    const float4 d = dphi ? reinterpret_cast<const float4*>(dphi)[(long long)img * DC4 + q]
                          : make_float4(1.f, 1.f, 1.f, 1.f);
    for (int o = 0; o < O; ++o) {
      const float4 wv = reinterpret_cast<const float4*>(Wd)[(long long)o * C4 + c4];
      reinterpret_cast<float4*>(G)[((long long)img * O + o) * DC4 + q] =
          make_float4(wv.x * inv_d * d.x, wv.y * inv_d * d.y, wv.z * inv_d * d.z, wv.w * inv_d * d.w);
    }
  }
}

hipError_t launch_conv_seed(hipStream_t s, const float* Wd, const float* dphi, int images, int O, int D,
                            int C, float* G) {
  const int DC = D * C;
  if (C % 4 == 0 && aligned16(Wd) && aligned16(dphi) && aligned16(G)) {
    const int DC4 = DC / 4, pb = cdiv(DC4, 256);
    const long long work = (long long)images * pb;
    k_conv_seed4<<<dim3((unsigned)std::min<long long>(work, 1 << 20)), dim3(256), 0, s>>>(
        Wd, dphi, images, O, DC4, C / 4, 1.0f / (float)D, G);
    return hipGetLastError();
  }
  const int bx = std::min(cdiv(DC, 256), 64);
  const int IO = images * O;
  k_conv_seed<<<dim3(bx, std::min(IO, 32768)), dim3(256), 0, s>>>(Wd, dphi, IO, O, DC, FastDiv((uint32_t)C),
                                                                 1.0f / (float)D, G);
  return hipGetLastError();
}

// The last convolution's summand when its cotangent is the readout's (through the global pool):
// theta[n1, n2, o1, o2] += scale sum_c Wr[o1, c] Wr[o2, c] Mc[c, n1, n2].  LDS form: a workgroup
// stages Wr and w2[c][o1 O + o2] = Wr[o1, c] Wr[o2, c] once, then per block of kFoldPairs input pairs
// their Mc columns, and each thread sums entries (pair, o1, o2) from LDS.  Otherwise one thread
// per entry reads Wr and Mc directly.
constexpr int kFoldPairs = 16, kFoldIlp = 8;
constexpr int kFoldLdsFloats = 16384;
template <bool LDS>
__global__ void __launch_bounds__(256)
k_readout_fold(const float* __restrict__ Wr, int C, int O, const float* __restrict__ Mc, int N1, int N2,
               float scale, float* __restrict__ theta) {
  extern __shared__ float sm[];
  const int OO = O * O;
  const long long plane = (long long)N1 * N2;
  if (!LDS) {
    for (long long idx = blockIdx.x * 256LL + threadIdx.x; idx < plane * OO; idx += (long long)gridDim.x * 256) {
      const long long pr = idx / OO;
      const int oo = (int)(idx - pr * OO);
      const int o1 = oo / O, o2 = oo - o1 * O;
      float acc = 0.f;
      for (int c = 0; c < C; ++c) acc += (Wr[o1 * C + c] * Wr[o2 * C + c]) * Mc[c * plane + pr];
      theta[idx] += scale * acc;
    }
    return;
  }
  float* w2 = sm;
  float* mc = sm + C * OO;
  float* wr = mc + C * kFoldPairs;
  for (int i = threadIdx.x; i < O * C; i += 256) wr[i] = Wr[i];
  __syncthreads();
  for (int oo = threadIdx.x; oo < OO; oo += 256) {
    const int o1 = oo / O, o2 = oo - o1 * O;
    for (int c = 0; c < C; ++c) w2[c * OO + oo] = wr[o1 * C + c] * wr[o2 * C + c];
  }
  for (long long p0 = (long long)blockIdx.x * kFoldPairs; p0 < plane; p0 += (long long)gridDim.x * kFoldPairs) {
    const int np = (int)min<long long>(kFoldPairs, plane - p0);
    __syncthreads();   // w2 staged; the previous block's reads of mc done
    for (int i = threadIdx.x; i < C * kFoldPairs; i += 256) {
      const int c = i / kFoldPairs, j = i - c * kFoldPairs;
      mc[i] = j < np ? Mc[c * plane + p0 + j] : 0.f;
    }
    __syncthreads();
    // kFoldIlp entries per thread at once (independent sums, their LDS reads in flight together)
    const int ne = np * OO;
    for (int e0 = threadIdx.x; e0 < ne; e0 += 256 * kFoldIlp) {
      float acc[kFoldIlp];
      int wo[kFoldIlp], mo[kFoldIlp];
#pragma unroll
      for (int q = 0; q < kFoldIlp; ++q) {
        const int e = min(e0 + q * 256, ne - 1);
        const int j = e / OO;
        wo[q] = e - j * OO;
        mo[q] = j;
        acc[q] = 0.f;
      }
#pragma unroll 4
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int q = 0; q < kFoldIlp; ++q) acc[q] += w2[c * OO + wo[q]] * mc[c * kFoldPairs + mo[q]];
#pragma unroll
      for (int q = 0; q < kFoldIlp; ++q)
        if (e0 + q * 256 < ne) theta[(p0 + mo[q]) * OO + wo[q]] += scale * acc[q];
    }
  }
}

hipError_t launch_readout_fold(hipStream_t s, const float* Wr, int C, int O, const float* Mc, int N1, int N2,
                               float scale, float* theta) {
  const long long plane = (long long)N1 * N2;
  if (plane <= 0 || O <= 0 || C <= 0) return hipSuccess;
  const long long lds = (long long)C * ((long long)O * O + kFoldPairs + O);
  if (lds <= kFoldLdsFloats) {
    const unsigned grid = (unsigned)std::min<long long>((plane + kFoldPairs - 1) / kFoldPairs, 4096);
    k_readout_fold<true><<<dim3(grid), dim3(256), (size_t)lds * 4, s>>>(Wr, C, O, Mc, N1, N2, scale, theta);
  } else {
    const unsigned grid = (unsigned)std::min<long long>((plane * O * O + 255) / 256, 65536);
    k_readout_fold<false><<<dim3(grid), dim3(256), 0, s>>>(Wr, C, O, Mc, N1, N2, scale, theta);
  }
  return hipGetLastError();
}

// The batch diagonal of the folded last convolution's per-channel Grams: Mc[c][n] =
// A1[n, c, :] . A2[n, c, :] (rows of KC floats, sample n's channel c at (n C + c) KC), one wave
// per (c, n), the lanes' partial sums added in a fixed butterfly order.
__global__ void __launch_bounds__(256)
k_fold_rowdot(const float* __restrict__ A1, const float* __restrict__ A2, int n, int C, int KC,
              float* __restrict__ Mc) {
  const long long item = blockIdx.x * 4LL + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (item >= (long long)n * C) return;   // the whole wave
  const int c = (int)(item / n), i = (int)(item - (long long)c * n);
  const float* a = A1 + ((long long)i * C + c) * KC;
  const float* b = A2 + ((long long)i * C + c) * KC;
  float v = 0.f;
  for (int k = lane; k < KC; k += 64) v += a[k] * b[k];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  if (lane == 0) Mc[item] = v;
}

hipError_t launch_fold_rowdot(hipStream_t s, const float* A1, const float* A2, int n, int C, int KC, float* Mc) {
  const long long items = (long long)n * C;
  if (items <= 0) return hipSuccess;
  if ((items + 3) / 4 > 0x7fffffffLL) return hipErrorInvalidValue;
  k_fold_rowdot<<<dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s>>>(A1, A2, n, C, KC, Mc);
  return hipGetLastError();
}

// The traced output of the folded last convolution: theta[n1, n2] += scale sum_c w_c Mc[c][n1, n2]
// with w_c = sum_o Wr[o, c]^2 (the trace of Wr[o1, c] Wr[o2, c] over o), staged in LDS when the C
// weights fit (LDS), else formed per channel from Wr; one pair per thread, channels in order.
template <bool LDS>
__global__ void __launch_bounds__(256)
k_readout_fold_trace(const float* __restrict__ Wr, int C, int O, const float* __restrict__ Mc, long long plane,
                     float scale, float* __restrict__ theta) {
  extern __shared__ float wsum[];
  auto weight = [&](int c) -> float {
    float v = 0.f;
    for (int o = 0; o < O; ++o) {
      const float x = Wr[(long long)o * C + c];
      v += x * x;
    }
    return v;
  };
  if (LDS) {
    for (int c = threadIdx.x; c < C; c += 256) wsum[c] = weight(c);
    __syncthreads();
  }
  for (long long p = blockIdx.x * 256LL + threadIdx.x; p < plane; p += (long long)gridDim.x * 256) {
    float acc = 0.f;
    for (int c = 0; c < C; ++c) acc += (LDS ? wsum[c] : weight(c)) * Mc[(long long)c * plane + p];
    theta[p] += scale * acc;
  }
}

hipError_t launch_readout_fold_trace(hipStream_t s, const float* Wr, int C, int O, const float* Mc, int N1, int N2,
                                     float scale, float* theta) {
  const long long plane = (long long)N1 * N2;
  if (plane <= 0 || O <= 0 || C <= 0) return hipSuccess;
  const unsigned grid = (unsigned)std::min<long long>((plane + 255) / 256, 4096);
  if (C <= kFoldLdsFloats)
    k_readout_fold_trace<true><<<dim3(grid), dim3(256), (size_t)C * 4, s>>>(Wr, C, O, Mc, plane, scale, theta);
  else
    k_readout_fold_trace<false><<<dim3(grid), dim3(256), 0, s>>>(Wr, C, O, Mc, plane, scale, theta);
  return hipGetLastError();
}

// Kt[ci, kh, kw, co] = K[co, 2 - kh, 2 - kw, ci]
__global__ void k_conv_flip(const float* __restrict__ K, int Cout, int Cin, float* __restrict__ Kt) {
  const int total = Cout * 9 * Cin;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int co = i % Cout;
    const int rest = i / Cout;
    const int tap = rest % 9, ci = rest / 9;
    const int kh = tap / 3, kw = tap % 3;
    Kt[i] = K[((co * 3 + (2 - kh)) * 3 + (2 - kw)) * Cin + ci];
  }
}

hipError_t launch_conv_flip(hipStream_t s, const float* K, int Cout, int Cin, float* Kt) {
  const int total = Cout * 9 * Cin;
  k_conv_flip<<<dim3(cdiv(total, 256)), dim3(256), 0, s>>>(K, Cout, Cin, Kt);
  return hipGetLastError();
}

// Kernel z of the batch: blockIdx.y; tap t of T is read from tap T - 1 - t (the 3x3 flip:
// (kh, kw) -> (2 - kh, 2 - kw); with T = 1 a transpose).
__global__ void __launch_bounds__(256) k_conv_flip_batch(FlipBatch b) {
  const int z = blockIdx.y;
  const int Cout = b.Cout[z], Cin = b.Cin[z], T = b.taps[z];
  const int total = Cout * T * Cin;
  const float* __restrict__ K = b.K[z];
  float* __restrict__ Kt = b.Kt[z];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int co = i % Cout;
    const int rest = i / Cout;
    const int tap = rest % T, ci = rest / T;
    Kt[i] = K[((long long)co * T + (T - 1 - tap)) * Cin + ci];
  }
}

hipError_t launch_conv_flip_batch(hipStream_t s, const FlipBatch& b) {
  if (b.count <= 0) return hipSuccess;
  if (b.count > kMaxLayers) return hipErrorInvalidValue;
  long long most = 0;
  for (int z = 0; z < b.count; ++z) {
    if (b.taps[z] != 1 && b.taps[z] != 9) return hipErrorInvalidValue;
    most = std::max(most, (long long)b.Cout[z] * b.taps[z] * b.Cin[z]);
  }
  if (most >= (1LL << 31)) return hipErrorInvalidValue;
  k_conv_flip_batch<<<dim3((unsigned)std::min<long long>(cdiv(most, 256), 1024), b.count), dim3(256), 0, s>>>(b);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------ pair preparation
// A row of a pair operand has the exponent of its true largest element, and where a sum runs over
// channels of different scales (the backward) both operands are balanced, as kernels_pair.hip explains.
// k_conv_prep: one wave per row of a flipped kernel (pair rows), one workgroup per layer for its balancing
// factors, one per image for its O seed cotangents' maxima, then workgroups that zero the others.  The
// seed is Wd[o, c] / D act'(z[p, c]): rounding is monotone, so its largest element over the pixels is that
// of the channel's largest act', and the maxima of the seed need no pass over it (taken in the kernel that
// writes it, they took that from 70 to 235 us: 1280 cotangent images of 32 x 32 x 64, six shuffles and an
// atomic per wave and image).
__global__ void __launch_bounds__(256) k_conv_prep(ConvPrep p, int nrow_blocks) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int bx = blockIdx.x;
  if (bx < nrow_blocks) {
    int row = bx * 4 + wave, z = 0;
    while (z < p.count && row >= p.N[z]) row -= p.N[z++];
    if (z >= p.count) return;   // the whole wave
    // nine taps of C channels, each padded to Cp
    const int C = p.C[z], Cp = (int)pair_stride(C), K = 9 * C, Kp = 9 * Cp;
    const float* __restrict__ x = p.Kt[z] + (long long)row * K;
    const float* __restrict__ km = p.kmax[z];
    int m = kPairNone;
    for (int k = lane; k < K; k += 64) {
      const int e = pair_e(x[k]);
      if (e > kPairNone) m = max(m, e - pair_bal_exp(km[k % C]));
    }
#pragma unroll
    for (int q = 32; q; q >>= 1) m = max(m, __shfl_xor(m, q));
    const int e = pair_row_e(m);
    if (lane == 0) p.kexps[z][row] = e;
    for (int g = lane; g < Kp / 8; g += 64) {
      f16x8 hi, lo;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int tap = 8 * g / Cp, c = 8 * g - tap * Cp + j, cc = min(c, C - 1);
        _Float16 a, b;
        pair_split(c < C ? ldexpf(x[tap * C + cc], -pair_bal_exp(km[cc]) - e) : 0.f, a, b);
        hi[j] = a;
        lo[j] = b;
      }
      f16x8* o = reinterpret_cast<f16x8*>(p.Kp[z] + (long long)row * Kp + 8 * g);
      o[0] = hi;
      o[1] = lo;
    }
    return;
  }
  bx -= nrow_blocks;
  if (bx < p.count) {
    const int C = p.C[bx];
    for (int c = threadIdx.x; c < (int)pair_stride(C); c += 256)
      p.kfac[bx][c] = c < C ? ldexpf(1.f, pair_bal_exp(p.kmax[bx][c])) : 1.f;
    return;
  }
  bx -= p.count;
  const int nseed = p.seed ? p.M : 0;
  if (bx < nseed) {
    const float* __restrict__ dm = p.dmax ? p.dmax + (long long)bx * p.Cl : nullptr;
    for (int o = wave; o < p.O; o += 4) {
      float a = 0.f, b = 0.f;
      for (int c = lane; c < p.Cl; c += 64) {
        const float w = p.Wd[(long long)o * p.Cl + c] * p.inv_d;
        const float x = fabsf(dm ? w * dm[c] : w);
        a = fmaxf(a, x);
        if (p.seed_kmax) b = fmaxf(b, x * ldexpf(1.f, pair_bal_exp(p.seed_kmax[c])));
      }
#pragma unroll
      for (int q = 32; q; q >>= 1) {
        a = fmaxf(a, __shfl_xor(a, q));
        b = fmaxf(b, __shfl_xor(b, q));
      }
      if (lane == 0) {
        p.seed[(long long)bx * p.O + o] = a;
        if (p.seed_kmax) p.seed_bal[(long long)bx * p.O + o] = b;
      }
    }
    return;
  }
  bx -= nseed;
  const int nz = gridDim.x - nrow_blocks - p.count - nseed;
  for (long long i = bx * 256LL + threadIdx.x; i < p.nzero; i += (long long)nz * 256) p.zero[i] = 0.f;
}

hipError_t launch_conv_prep(hipStream_t s, const ConvPrep& p) {
  long long rows = 0;
  for (int z = 0; z < p.count; ++z) rows += p.N[z];
  const int nr = cdiv(rows, 4), nz = (int)std::min<long long>((p.nzero + 1023) / 1024, 256);
  const long long blocks = (long long)nr + p.count + (p.seed ? p.M : 0) + nz;
  if (blocks <= 0) return hipSuccess;
  k_conv_prep<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(p, nr);
  return hipGetLastError();
}

// Workgroup (row, item), eight loads in flight per thread; behind the items, one image of cx each, by
// channel: threads as groups of V channels (CL groups at a time, a power of two) by pixels.
template <int V>
__device__ __forceinline__ void chan_max_image(const float* __restrict__ x, int D, int C, int CL, float* __restrict__ out,
                                               float (*red)[4]) {
  const int CG = C / V, c = threadIdx.x & (CL - 1), pg = threadIdx.x / CL, np = 256 / CL;
  for (int c0 = 0; c0 < CG; c0 += CL) {
    const int cc = min(c0 + c, CG - 1);
    float m[V] = {};
    for (int p = pg; p < D; p += 8 * np) {
      float v[8][V];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float* a = x + ((long long)min(p + u * np, D - 1) * CG + cc) * V;
        if constexpr (V == 4) {
          const f32x4 t = *reinterpret_cast<const f32x4*>(a);
#pragma unroll
          for (int q = 0; q < 4; ++q) v[u][q] = t[q];
        } else {
          v[u][0] = *a;
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int q = 0; q < V; ++q) m[q] = fmaxf(m[q], fabsf(v[u][q]));
    }
#pragma unroll
    for (int q = 0; q < V; ++q) red[threadIdx.x][q] = m[q];
    __syncthreads();
    if (pg == 0 && c0 + c < CG)
#pragma unroll
      for (int q = 0; q < V; ++q) {
        for (int u = 1; u < np; ++u) m[q] = fmaxf(m[q], red[u * CL + c][q]);
        out[(c0 + c) * V + q] = m[q];
      }
    __syncthreads();
  }
}
__global__ void __launch_bounds__(256) k_conv_max(ConvMax b) {
  __shared__ float cred[256][4];
  float* red = &cred[0][0];
  const int z = blockIdx.y;
  if (z == b.count) {
    if ((int)blockIdx.x >= b.M) return;
    const float* x = b.cx + (long long)blockIdx.x * b.D * b.C;
    float* out = b.cout + (long long)blockIdx.x * b.C;
    const bool vec = b.C % 4 == 0 && (reinterpret_cast<uintptr_t>(b.cx) & 15) == 0;
    int CL = 4;
    while (CL < (vec ? b.C / 4 : b.C) && CL < 64) CL *= 2;
    if (vec) chan_max_image<4>(x, b.D, b.C, CL, out, cred);
    else chan_max_image<1>(x, b.D, b.C, CL, out, cred);
    return;
  }
  const int n = b.plane[z];
  if ((int)blockIdx.x >= b.rows[z]) return;
  const float* __restrict__ x = b.x[z] + (long long)blockIdx.x * n;
  float m = 0.f;
  if (n % 4 == 0 && (reinterpret_cast<uintptr_t>(b.x[z]) & 15) == 0) {
    const f32x4* __restrict__ x4 = reinterpret_cast<const f32x4*>(x);
    for (int i = threadIdx.x; i < n / 4; i += 2048) {
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = x4[min(i + 256 * u, n / 4 - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        m = fmaxf(m, fmaxf(fmaxf(fabsf(v[u][0]), fabsf(v[u][1])), fmaxf(fabsf(v[u][2]), fabsf(v[u][3]))));
    }
  } else {
    for (int i = threadIdx.x; i < n; i += 2048) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = x[min(i + 256 * u, n - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) m = fmaxf(m, fabsf(v[u]));
    }
  }
#pragma unroll
  for (int q = 32; q; q >>= 1) m = fmaxf(m, __shfl_xor(m, q));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) b.out[z][blockIdx.x] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

hipError_t launch_conv_max(hipStream_t s, const ConvMax& m) {
  int rows = m.cx ? m.M : 0;
  for (int z = 0; z < m.count; ++z) rows = std::max(rows, m.rows[z]);
  if (rows <= 0) return hipSuccess;
  k_conv_max<<<dim3(rows, m.count + (m.cx ? 1 : 0)), dim3(256), 0, s>>>(m);
  return hipGetLastError();
}

// J[(s*O + o), off + c*KCs + js] = acc[r = o*C + c, k] for the GEMM columns k of KC = F Cin
// (F taps of Cin computed input channels), stored as the columns js of KCs = F Cst (the first Cst
// channels of each tap: a layer input padded from Cst to Cin channels has zero columns that are
// not stored; Cst = Cin: js = k).  A fragment inside R = O*C and inside one o (no multiple of C
// in (r0, r0 + 31]) writes 32 consecutive c of one row of J, addressed from one base (32-bit byte
// offsets: KCs < 2^25).
template <class Cfg>
__device__ __forceinline__ void conv_wgrad_store(f32x16 (&acc)[Cfg::FM][Cfg::FN], int m0, int n0, int s,
                                                 int O, FastDiv fC, int KC, FastDiv fCin, int Cst,
                                                 float* __restrict__ J, long long ldJ, long long off) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm0 = (wave / Cfg::WAVES_N) * Cfg::WM;
  const int wn0 = (wave % Cfg::WAVES_N) * Cfg::WN;
  const int C = (int)fC.d, R = O * C;
  const int Cin = (int)fCin.d, KCs = Cst == Cin ? KC : (KC / Cin) * Cst;
  // the stored column of GEMM column k, or -1 (a padded channel or past KC)
  auto col = [&](int k) {
    if (k >= KC) return -1;
    if (Cst == Cin) return k;
    const int tap = (int)fCin.div(k), ci = k - tap * Cin;
    return ci < Cst ? tap * Cst + ci : -1;
  };
#pragma unroll
  for (int fm = 0; fm < Cfg::FM; ++fm) {
    const int r0 = __builtin_amdgcn_readfirstlane(m0 + wm0 + fm * 32);
    if (r0 >= R) continue;
    const int o0 = (int)fC.div(r0);
    if (r0 + 32 <= R && KCs < (1 << 25) && (int)fC.div(r0 + 31) == o0) {
      float* base = J + ((long long)s * O + o0) * ldJ + off + (long long)(r0 - o0 * C) * KCs;
#pragma unroll
      for (int fn = 0; fn < Cfg::FN; ++fn) {
        const int js = col(n0 + wn0 + fn * 32 + (lane & 31));
        if (js < 0) continue;
#pragma unroll
        for (int v = 0; v < 16; ++v) at_bytes(base, (uint32_t)(frag_row(v, lane) * KCs + js) * 4u) = acc[fm][fn][v];
      }
    } else {
#pragma unroll
      for (int fn = 0; fn < Cfg::FN; ++fn) {
        const int js = col(n0 + wn0 + fn * 32 + (lane & 31));
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = r0 + frag_row(v, lane);
          if (r < R && js >= 0) {
            const int o = (int)fC.div(r), c = r - o * C;
            J[((long long)s * O + o) * ldJ + off + (long long)c * KCs + js] = acc[fm][fn][v];
          }
        }
      }
    }
  }
}
// out[(img*O+o), p, ci] = (sum_k patch(G)[.., p, k] Kt[ci, k]) * dphi[img, p, ci]
template <class Cfg, bool VEC>
__global__ void __launch_bounds__(Cfg::THREADS)
k_conv_bwd(LoadPatchesKInnerT<VEC> la, LoadKInnerT<VEC> lb, const float* __restrict__ dphi, int R,
           int N, FastDiv fOD, FastDiv fD, float* __restrict__ out, int tiles_n, ImageMax mx) {
  extern __shared__ float smem[];
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  gemm_mainloop<Cfg>(la, lb, m0, n0, 0, la.K, smem, acc);
  store_pixel_rows<Cfg>(acc, m0, n0, dphi, out, R, N, fOD, fD, mx);
}

// direct-to-LDS form (Cg % 32 == 0): the cotangent patches gathered by the DMA, NS LDS stages
template <class Cfg, int NS>
__global__ void __launch_bounds__(Cfg::THREADS)
k_conv_bwd_dma(DmaPatches<Cfg::BM, Cfg::WAVES> pa, DmaRowMajor<Cfg::BN, Cfg::WAVES> pb, int K,
               const float* __restrict__ dphi, int R, int N, FastDiv fOD, FastDiv fD, float* __restrict__ out,
               int tiles_n, ImageMax mx) {
  extern __shared__ float smem[];
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  gemm_mainloop_dma_ops<Cfg, NS>(pa, pb, m0, n0, 0, K, smem, acc);
  store_pixel_rows<Cfg>(acc, m0, n0, dphi, out, R, N, fOD, fD, mx);
}

// The same on pairs.  A tile's rows are a run of BM pixels of the stacked cotangent images, and the
// pixels its nine taps read are that run widened by W + 1 on both sides, so the workgroup keeps
// 32 channels of those BM + 2 (W + 1) pixels in LDS as pairs: each cotangent is read from memory
// and split once per tile (with the exponent of its image) instead of once per tap, the nine taps
// are row shifts of the LDS reads, and a tap outside the image reads a row of zeros.  The kernel
// (pair rows) streams through two LDS stages, 32 k at a time.  1280 images of 32 x 32 x 64:
// 788 us with the fp32 MFMA, 408 us with the cotangents gathered and split per tap (VALU beside
// the MFMAs), this form 327 us; 346 with the channels' balancing factors and the maxima of the images
// it writes.  Any number of channels: they are padded with zeros to a multiple
// of 32 on the way into LDS (and in the kernel's pair rows); VEC: Cg % 4 == 0, 16-byte loads.
constexpr int kHaloMaxW = 63;
template <class Cfg>
constexpr int halo_rows(int W) {
  return Cfg::BM + 2 * (W + 1);
}
// tasks (8 channels of a pixel) per thread of the staging: widest images
template <class Cfg>
constexpr int halo_tasks() {
  return (halo_rows<Cfg>(kHaloMaxW) * 4 + Cfg::THREADS - 1) / Cfg::THREADS;
}
template <class Cfg>
static int halo_smem_bytes(int W) {
  return ((halo_rows<Cfg>(W) + 1) * 32 + 2 * Cfg::BN * 32) * 4;
}
template <class Cfg, bool VEC>
__global__ void __launch_bounds__(Cfg::THREADS, 2 * Cfg::THREADS / 256)
k_conv_bwd_pair(const float* __restrict__ G, int H, int W, int Cg, FastDiv fW, DmaRowMajor<Cfg::BN, Cfg::WAVES> pb,
                ConvPairBwd pr, const float* __restrict__ dphi, int R, int N, FastDiv fOD, FastDiv fD,
                float* __restrict__ out, int tiles_n, ImageMax mx) {
  extern __shared__ f32x4 halo_lds[];   // 16-byte aligned
  float* smem = reinterpret_cast<float*>(halo_lds);
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm0 = (wave / Cfg::WAVES_N) * Cfg::WM, wn0 = (wave % Cfg::WAVES_N) * Cfg::WN;
  const int lr = lane & 31, lc = (lane >> 5) * 2;
  const int HR = halo_rows<Cfg>(W);
  float* Bs = smem + (HR + 1) * 32;
  constexpr int NT = halo_tasks<Cfg>();
  const int ncb = (Cg + 31) / 32, nk = 9 * ncb;
  // staging: task t = row t / 4 of the widened run, channels 8 (t % 4) .. + 7 of the block.  Rows
  // outside the batch are read from a clamped address; no tap inside an image reaches them.
  const float* src[NT];
  float sf[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int t = threadIdx.x + i * Cfg::THREADS;
    const int q = min(max(m0 - (W + 1) + min(t >> 2, HR - 1), 0), R - 1);
    src[i] = G + (long long)q * Cg;
    sf[i] = pair_factor(pair_row_exp(pr.gbal[fD.div(q)]));
  }
  f32x4 st[NT][2], kf[2];   // kf: the balancing factors of the thread's channels (padded to whole blocks)
  auto fetch = [&](int cb) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      kf[u] = *reinterpret_cast<const f32x4*>(pr.kfac + cb * 32 + 8 * (threadIdx.x & 3) + 4 * u);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int c0 = cb * 32 + 8 * (threadIdx.x & 3);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = c0 + 4 * u;
        if (VEC) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(src[i] + min(c, Cg - 4));
          st[i][u] = c < Cg ? v : f32x4{0.f, 0.f, 0.f, 0.f};
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float v = src[i][min(c + k, Cg - 1)];
            st[i][u][k] = c + k < Cg ? v : 0.f;
          }
        }
      }
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int t = threadIdx.x + i * Cfg::THREADS, row = t >> 2, c = 2 * (t & 3);
      if (row < HR) {
        f16x8 hi, lo;
        pair_split8(st[i][0] * kf[0], st[i][1] * kf[1], sf[i], hi, lo);
        *reinterpret_cast<f16x8*>(&smem[row * 32 + (DmaTile<32>::swz(row, c) << 2)]) = hi;
        *reinterpret_cast<f16x8*>(&smem[row * 32 + (DmaTile<32>::swz(row, c + 1) << 2)]) = lo;
      }
    }
  };
  // this lane's rows: the row of the pixel itself in LDS and the taps outside its image
  int rb[Cfg::FM];
  unsigned om[Cfg::FM];
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
    const int l = wm0 + i * 32 + lr, r = m0 + l;
    const int rc = min(r, R - 1), p = rc - (int)fD.div(rc) * (int)fD.d;
    const int y = (int)fW.div(p), x = p - y * W;
    rb[i] = l + W + 1;
    unsigned m = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int ky = y + t / 3 - 1, kx = x + t % 3 - 1;
      m |= ((unsigned)ky < (unsigned)H && (unsigned)kx < (unsigned)W) ? 0u : (1u << t);
    }
    om[i] = r < R ? m : 0x1FFu;
  }
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  pb.prepare(n0, wave, lane);
  if (threadIdx.x < 32) smem[HR * 32 + threadIdx.x] = 0.f;
  pb.template issue<Cfg::WAVES>(0, Bs, wave, lane);
  fetch(0);
  stage();
  wait_vmcnt_lgkm0<0>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  f16x8 a[2][2], b[2][Cfg::FN][2];
  int row[Cfg::FM];
  auto rows_of = [&](int tap) {
    const int shift = (tap / 3 - 1) * W + tap % 3 - 1;
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) row[i] = ((om[i] >> tap) & 1u) ? HR : rb[i] + shift;
  };
  auto load_a = [&](int half, int i, f16x8 (&x)[2]) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
      x[p] = *reinterpret_cast<const f16x8*>(&smem[row[i] * 32 + (DmaTile<32>::swz(row[i], half * 4 + lc + p) << 2)]);
  };
  auto load_b = [&](const float* bs, int half, f16x8 (&x)[Cfg::FN][2]) {
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int r = wn0 + j * 32 + lr;
        x[j][p] = *reinterpret_cast<const f16x8*>(&bs[r * 32 + (DmaTile<32>::swz(r, half * 4 + lc + p) << 2)]);
      }
  };
  auto mma = [&](int i, const f16x8 (&x)[2], const f16x8 (&y)[Cfg::FN][2]) {
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
  rows_of(0);
  load_b(Bs, 0, b[0]);
  load_a(0, 0, a[0]);
  int tap = 0, cb = 0;
  auto step = [&](int kt, auto stage_tag) {
    constexpr int S = decltype(stage_tag)::value;
    const float* bs = Bs + S * Cfg::BN * 32;
    int tap1 = tap + 1, cb1 = cb;
    if (tap1 == 9) {
      tap1 = 0;
      ++cb1;
    }
    if (kt + 1 < nk) pb.template issue<Cfg::WAVES>((tap1 * ncb + cb1) * 32, Bs + (S ^ 1) * Cfg::BN * 32, wave, lane);
    if (tap == 0 && cb + 1 < ncb) fetch(cb + 1);
#pragma unroll
    for (int q = 0; q + 1 < 2 * Cfg::FM; ++q) {
      const int half = q / Cfg::FM, next = (q + 1) / Cfg::FM;
      if (next != half) load_b(bs, next, b[1]);
      load_a(next, (q + 1) % Cfg::FM, a[(q + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      mma(q % Cfg::FM, a[q & 1], b[half]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (kt + 1 < nk) {
      if (tap1 == 0) {   // every wave has read the block's last fragments: the next block's pixels
        wait_vmcnt_lgkm0<0>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        stage();
      }
      wait_vmcnt_lgkm0<0>();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      rows_of(tap1);
      load_b(Bs + (S ^ 1) * Cfg::BN * 32, 0, b[0]);
      load_a(0, 0, a[0]);
      __builtin_amdgcn_sched_barrier(0);
    }
    mma(Cfg::FM - 1, a[1], b[1]);
    __builtin_amdgcn_sched_barrier(0);
    tap = tap1;
    cb = cb1;
  };
  int kb = 0;
  for (; kb + 2 <= nk; kb += 2) {
    step(kb, std::integral_constant<int, 0>{});
    step(kb + 1, std::integral_constant<int, 1>{});
  }
  if (kb < nk) step(kb, std::integral_constant<int, 0>{});
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
    const int r0 = min(m0 + wm0 + i * 32, R - 1), t0 = (int)fD.div(r0);
    const bool one = (int)fD.div(min(r0 + 31, R - 1)) == t0;
    const int e0 = pair_row_exp(pr.gbal[t0]);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int e = one ? e0 : pair_row_exp(pr.gbal[fD.div(min(r0 + frag_row(v, lane), R - 1))]);
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j)
        acc[i][j][v] = ldexpf(acc[i][j][v], e + pr.kexps[min(n0 + wn0 + j * 32 + lr, N - 1)]);
    }
  }
  store_pixel_rows<Cfg>(acc, m0, n0, dphi, out, R, N, fOD, fD, mx);
}

template <bool VEC>
static hipError_t conv_bwd_vec(hipStream_t s, const float* G, int images, int O, int H, int W, int Cg,
                               const float* Kt, int Cin, const float* dphi, float* out, const ImageMax& mx) {
  using Cfg = CfgConv;
  using LA = LoadPatchesKInnerT<VEC>;
  using LB = LoadKInnerT<VEC>;
  const int D = H * W;
  LA la = patches_kinner<VEC>(G, images * O, H, W, Cg);
  LB lb{Kt, Cin, 9 * Cg, 9 * Cg};
  int R;
  if (!to_int((long long)images * O * D, R)) return hipErrorInvalidValue;
  const int tn = cdiv(Cin, Cfg::BN), tm = cdiv(R, Cfg::BM);
  hipError_t e = set_smem<Cfg, LA, LB>((const void*)k_conv_bwd<Cfg, VEC>);
  if (e != hipSuccess) return e;
  k_conv_bwd<Cfg, VEC><<<dim3(tm * tn), dim3(Cfg::THREADS), gemm_smem_bytes<Cfg, LA, LB>(), s>>>(
      la, lb, dphi, R, Cin, FastDiv((uint32_t)(O * D)), FastDiv((uint32_t)D), out, tn, mx);
  return hipGetLastError();
}

template <class Cfg>
static hipError_t conv_bwd_dma_cfg(hipStream_t s, const float* G, int images, int O, int H, int W, int Cg,
                                   const float* Kt, int Cin, const float* dphi, float* out, const ImageMax& mx) {
  constexpr int NS = kConvBwdStages;
  const int D = H * W, Kd = 9 * Cg;
  int R;
  if (!to_int((long long)images * O * D, R)) return hipErrorInvalidValue;
  const int tn = cdiv(Cin, Cfg::BN), tm = cdiv(R, Cfg::BM);
  auto pa = dma_patches<Cfg::BM, Cfg::WAVES>(G, images * O, H, W, Cg);
  DmaRowMajor<Cfg::BN, Cfg::WAVES> pb{Kt, Kd, Cin};
  constexpr int bytes = gemm_dma_smem_bytes<Cfg, NS>();
  hipError_t e = hipFuncSetAttribute((const void*)k_conv_bwd_dma<Cfg, NS>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  k_conv_bwd_dma<Cfg, NS><<<dim3(tm * tn), dim3(Cfg::THREADS), bytes, s>>>(
      pa, pb, Kd, dphi, R, Cin, FastDiv((uint32_t)(O * D)), FastDiv((uint32_t)D), out, tn, mx);
  return hipGetLastError();
}

template <class Cfg, bool VEC>
static hipError_t conv_bwd_pair_cfg(hipStream_t s, const float* G, int images, int O, int H, int W, int Cg,
                                    const ConvPairBwd& pr, int Cin, const float* dphi, float* out, const ImageMax& mx) {
  const int D = H * W, Kd = 9 * (int)pair_stride(Cg);
  int R;
  if (!to_int((long long)images * O * D, R)) return hipErrorInvalidValue;
  const int tn = cdiv(Cin, Cfg::BN), tm = cdiv(R, Cfg::BM);
  DmaRowMajor<Cfg::BN, Cfg::WAVES> pb{pr.Kp, Kd, Cin};
  hipError_t e = hipFuncSetAttribute((const void*)k_conv_bwd_pair<Cfg, VEC>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, halo_smem_bytes<Cfg>(kHaloMaxW));
  if (e != hipSuccess) return e;
  k_conv_bwd_pair<Cfg, VEC><<<dim3(tm * tn), dim3(Cfg::THREADS), halo_smem_bytes<Cfg>(W), s>>>(
      G, H, W, Cg, FastDiv((uint32_t)W), pb, pr, dphi, R, Cin, FastDiv((uint32_t)(O * D)), FastDiv((uint32_t)D), out, tn,
      mx);
  return hipGetLastError();
}

// whether the cotangent backward of a layer takes the pair form
bool conv_bwd_pair_ok(int W, int Cg) {
  const long long Kd = 9 * pair_stride(Cg);
  return W <= kHaloMaxW && dma_span_ok(Kd, Kd, 256);
}

static hipError_t conv_bwd_pair(hipStream_t s, const float* G, int images, int O, int H, int W, int Cg,
                                const ConvPairBwd& pr, int Cin, const float* dphi, float* out, const ImageMax& mx) {
  const bool vec = Cg % 4 == 0 && aligned16(G);
  auto go = [&](auto cfg_tag) {
    using Cfg = decltype(cfg_tag);
    return vec ? conv_bwd_pair_cfg<Cfg, true>(s, G, images, O, H, W, Cg, pr, Cin, dphi, out, mx)
               : conv_bwd_pair_cfg<Cfg, false>(s, G, images, O, H, W, Cg, pr, Cin, dphi, out, mx);
  };
  // few rows: 128-row tiles, for more workgroups; few channels: 32 columns
  const bool few = (long long)cdiv((long long)images * O * H * W, 256) * cdiv(Cin, 64) < kConvFewTiles;
  if (Cin <= 32) return few ? go(CfgConvBwdPairSmallN{}) : go(CfgConvBwdPairN{});
  return few ? go(CfgConvBwdPairSmall{}) : go(CfgConvBwdPair{});
}

hipError_t launch_conv_bwd(hipStream_t s, const float* G, int images, int O, int H, int W, int Cg,
                           const float* Kt, int Cin, const float* dphi, float* out, const ConvPairBwd* pair,
                           const ImageMax& mx) {
  if (pair) return conv_bwd_pair(s, G, images, O, H, W, Cg, *pair, Cin, dphi, out, mx);
  if (conv_dma_ok(G, (long long)images * O * H * W * Cg, W, Cg, Kt)) {
    const long long tiles = (long long)cdiv((long long)images * O * H * W, CfgConvBwd::BM) * cdiv(Cin, CfgConvBwd::BN);
    if (tiles < kConvFewTiles) return conv_bwd_dma_cfg<CfgConv>(s, G, images, O, H, W, Cg, Kt, Cin, dphi, out, mx);
    return conv_bwd_dma_cfg<CfgConvBwd>(s, G, images, O, H, W, Cg, Kt, Cin, dphi, out, mx);
  }
  if (Cg % 4 == 0 && aligned16(G) && vec_ok(Kt, 9 * Cg, 9 * Cg))
    return conv_bwd_vec<true>(s, G, images, O, H, W, Cg, Kt, Cin, dphi, out, mx);
  return conv_bwd_vec<false>(s, G, images, O, H, W, Cg, Kt, Cin, dphi, out, mx);
}

// ------------------------------------------------------------------------------ weight-space cotangent
// For sample s = blockIdx.y:  J[s*O + o][off + c*KC + k] = sum_p G[s,o,p,c] patch[s,p,k]
// (VA / VB: float4 loads of the cotangent / patch operand)
template <class Cfg, bool VA, bool VB, bool PW>
__global__ void __launch_bounds__(Cfg::THREADS)
k_conv_wgrad(const float* __restrict__ G, const float* __restrict__ h, int O, int H, int W, int C,
             int Cin, FastDiv fC, FastDiv fW, FastDiv fCin, float* __restrict__ J, long long ldJ,
             long long off, int tiles_m, int tiles_n, int samples) {
  extern __shared__ float smem[];
  int s, t;
  if (!xcd_sample_tile(blockIdx.x, tiles_m * tiles_n, samples, s, t)) return;
  const int D = H * W;
  const int KC = PW ? Cin : 9 * Cin;
  const int tm = t / tiles_n, tn = t - tm * tiles_n;
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  LoadCotangentKOuterT<VA> la;
  la.g = G + (long long)s * O * D * C;
  la.rows = O * C;
  la.K = D;
  la.C = C;
  la.D = D;
  la.fC = fC;
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  if constexpr (PW) {
    // pointwise: the columns are the input channels themselves, [D, Cin] of the sample
    LoadCotangentKOuterT<VB> lb;
    lb.g = h + (long long)s * D * Cin;
    lb.rows = Cin;
    lb.K = D;
    lb.C = Cin;
    lb.D = D;
    lb.fC = fCin;
    gemm_mainloop<Cfg>(la, lb, m0, n0, 0, D, smem, acc);
  } else {
    LoadPatchesKOuterT<VB> lb;
    lb.x = h + (long long)s * D * Cin;
    lb.rows = KC;
    lb.K = D;
    lb.H = H;
    lb.W = W;
    lb.C = Cin;
    lb.fW = fW;
    lb.fC = fCin;
    gemm_mainloop<Cfg>(la, lb, m0, n0, 0, D, smem, acc);
  }
  conv_wgrad_store<Cfg>(acc, m0, n0, s, O, fC, KC, fCin, Cin, J, ldJ, off);
}

// direct-to-LDS form (C % 4 == 0 and Cin % 4 == 0): both operands K-outer, NS LDS stages
// AL: every K tile of 32 pixels is whole (D % 32 == 0) and, for the 3x3 patches, lies in one
// image row (W % 32 == 0)
template <class Cfg, int NS, bool PW, bool AL>
__global__ void __launch_bounds__(Cfg::THREADS)
k_conv_wgrad_dma(const float* __restrict__ G, const float* __restrict__ h, int O, int H, int W, int C, int Cin, FastDiv fC, FastDiv fW, FastDiv fCin,
                 int Cst, float* __restrict__ J, long long ldJ, long long off, int tiles_m, int tiles_n, int samples) {
  extern __shared__ float smem[];
  int s, t;
  if (!xcd_sample_tile(blockIdx.x, tiles_m * tiles_n, samples, s, t)) return;
  const int D = H * W;
  const int KC = PW ? Cin : 9 * Cin;
  const int tm = t / tiles_n, tn = t - tm * tiles_n;
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  DmaCotangentKOuter<Cfg::BM, Cfg::WAVES, AL> ia;
  ia.g = G + (long long)s * O * D * C;
  ia.rows = O * C;
  ia.D = D;
  ia.C = C;
  ia.fC = fC;
  // two MFMA chains per fragment (DualAcc), added after the K loop
  DualAcc dacc[Cfg::FM][Cfg::FN];
#pragma unroll
  for (int fm = 0; fm < Cfg::FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < Cfg::FN; ++fn)
#pragma unroll
      for (int v = 0; v < 16; ++v) dacc[fm][fn].v[0][v] = dacc[fm][fn].v[1][v] = 0.f;
  if constexpr (PW) {
    // pointwise: the columns are the input channels themselves, [D, Cin] of the sample
    DmaCotangentKOuter<Cfg::BN, Cfg::WAVES, AL> ib;
    ib.g = h + (long long)s * D * Cin;
    ib.rows = Cin;
    ib.D = D;
    ib.C = Cin;
    ib.fC = fCin;
    gemm_mainloop_dma_ops<Cfg, NS>(ia, ib, m0, n0, 0, D, smem, dacc);
  } else {
    DmaPatchesKOuter<Cfg::BN, Cfg::WAVES, AL> ib;
    ib.x = h + (long long)s * D * Cin;
    ib.rows = KC;
    ib.K = D;
    ib.H = H;
    ib.W = W;
    ib.C = Cin;
    ib.fW = fW;
    ib.fC = fCin;
    gemm_mainloop_dma_ops<Cfg, NS>(ia, ib, m0, n0, 0, D, smem, dacc);
  }
  f32x16 acc[Cfg::FM][Cfg::FN];
#pragma unroll
  for (int fm = 0; fm < Cfg::FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < Cfg::FN; ++fn) acc[fm][fn] = dacc[fm][fn].v[0] + dacc[fm][fn].v[1];
  conv_wgrad_store<Cfg>(acc, m0, n0, s, O, fC, KC, fCin, Cst, J, ldJ, off);
}

// The same on pairs.  Both operands are K-outer in memory (4 consecutive rows at one pixel per 16
// bytes), so a thread loads 4 rows x 8 pixels, splits them with the row's exponent (the cotangent
// image (s, o), or the sample's input) and writes them as pair rows [row][32 pixels] into LDS:
// each value is split once per tile, and the waves read whole MFMA operands (16 bytes) instead of
// eight floats each.  The next K tile's loads are in flight during a tile's MFMAs; two LDS stages.
// 64 -> 64 channels, 128 x 10 cotangent images of 32 x 32: 555 us with the fp32 MFMA, 415 us with
// every wave splitting its own fragments, this form 384 us.
// The first column tile also adds up the bias columns: a pass of their own over 1280 cotangent images of
// 32 x 32 x 64 took 70 us (1689 us for the biased network of five convolutions, 1830 us with it).
// Position of 16-byte chunk c of row r: eight consecutive rows (a fragment read) and every fourth
// row (the writes of eight threads) both fall in eight distinct bank groups.
__device__ __forceinline__ int wg_swz(int r, int c) { return c ^ ((r >> 2) & 7) ^ (((r >> 1) & 1) << 2); }

// VA, VB: C % 4 == 0, Cin % 4 == 0 with aligned operands, one 16-byte load per pixel; otherwise the
// four rows of a task have addresses (and taps) of their own.
template <class Cfg, bool PW, bool AL, bool VA, bool VB>
__global__ void __launch_bounds__(Cfg::THREADS, 2 * Cfg::THREADS / 256)
k_conv_wgrad_pair(const float* __restrict__ G, const float* __restrict__ h, ConvPairWgrad pr, int O, int H, int W, int C,
                  int Cin, FastDiv fC, FastDiv fW, FastDiv fCin, int Cst, float* __restrict__ J, long long ldJ,
                  long long off, int tiles_m, int tiles_n, int samples) {
  static_assert(Cfg::BM + Cfg::BN <= Cfg::THREADS && Cfg::BM % 64 == 0, "one staging task per thread, per wave one operand");
  static_assert(!AL || (VA && VB), "the aligned form loads vectors");
  extern __shared__ f32x4 wg_lds[];   // 16-byte aligned
  float* smem = reinterpret_cast<float*>(wg_lds);
  constexpr int AF = Cfg::BM * 32, STAGE = (Cfg::BM + Cfg::BN) * 32;
  constexpr int NR = VA && VB ? 1 : 4;       // addresses per task
  int s, t;
  if (!xcd_sample_tile(blockIdx.x, tiles_m * tiles_n, samples, s, t)) return;
  const int D = H * W, nk = (D + 31) / 32;
  const int KC = PW ? Cin : 9 * Cin;
  const int tm = t / tiles_n, tn = t - tm * tiles_n;
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm0 = (wave / Cfg::WAVES_N) * Cfg::WM, wn0 = (wave % Cfg::WAVES_N) * Cfg::WN;
  const int lr = lane & 31, lc = (lane >> 5) * 2;
  auto row_exp = [&](int r) { return pair_row_exp(pr.gmax[s * O + (int)fC.div(min(r, O * C - 1))]); };
  const int eh = pair_row_exp(pr.hmax[s]);
  // staging task of this thread: 4 rows (quad q) x 8 pixels (group g) of operand A (the first BM
  // threads) or B.  Byte offsets through a buffer resource that starts W + 1 pixels before the
  // sample for the patches; a pixel outside the sample or the image, or a row past the operand,
  // takes an offset past its end, which reads zeros.
  const bool is_b = __builtin_amdgcn_readfirstlane(threadIdx.x >= Cfg::BM ? 1 : 0) != 0;
  const int task = threadIdx.x - (is_b ? Cfg::BM : 0);
  const int nq = (is_b ? Cfg::BN : Cfg::BM) / 4;
  const int q = task % nq, g = task / nq;
  const bool active = g < 4;
  const int row = 4 * q;                       // in the tile
  const int Ct = is_b ? Cin : C;               // floats between two pixels
  const bool vec = is_b ? VB : VA;
  int base[NR], dy[NR], dx[NR];
  bool in_rows[NR];
  float sf[4];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    dy[i] = dx[i] = 0;
    if (!is_b) {
      const int r = m0 + row + i, rc = min(r, O * C - (vec ? 4 : 1)), o = (int)fC.div(rc);
      base[i] = (o * D * C + (rc - o * C)) * 4;
      in_rows[i] = r < O * C;
    } else {
      const int r = n0 + row + i, rc = min(r, KC - (vec ? 4 : 1));
      const int tap = PW ? 0 : (int)fCin.div(rc), ci = rc - tap * Cin;
      if (!PW) {
        const int kh = (tap * 11) >> 5;
        dy[i] = kh - 1;
        dx[i] = tap - 3 * kh - 1;
      }
      base[i] = ((PW ? 0 : dy[i] * W + dx[i] + W + 1) * Cin + ci) * 4;
      in_rows[i] = r < KC;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) sf[i] = pair_factor(is_b ? eh : row_exp(m0 + row + (vec ? 0 : i)));
  const float* p0 = is_b ? h + (long long)s * D * Cin - (PW ? 0 : (long long)(W + 1) * Cin) : G + (long long)s * O * D * C;
  const uint32_t span = (uint32_t)((is_b ? (long long)(D + (PW ? 0 : W + 1)) * Cin : (long long)O * D * C) * 4);
  const __amdgpu_buffer_rsrc_t rsrc = buffer_rsrc(p0, span);   // wave-uniform: is_b is
  // the lambdas are forced inline: called as functions they would keep the arrays in scratch memory
  float st[4][8];   // [row][pixel]
  // the pixels of this thread's group that a row with tap (dyr, dxr) reads as zeros
  auto outside = [&](bool in_row, int dyr, int dxr, int p, int y, int x) __attribute__((always_inline)) {
    unsigned bad = (in_row && active) ? 0u : 0xFFu;
    if (AL) {   // the K tile is whole and (patches) a run of one image row
      if (is_b && !PW) {
        if ((unsigned)(y + dyr) >= (unsigned)H) bad = 0xFFu;
        if (x == 0 && dxr < 0) bad |= 1u;
        if (x + 8 == W && dxr > 0) bad |= 0x80u;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        bool ok = p + j < D;
        if (is_b && !PW) {
          ok = ok && (unsigned)(y + dyr) < (unsigned)H && (unsigned)(x + dxr) < (unsigned)W;
          if (++x == W) {
            x = 0;
            ++y;
          }
        }
        bad |= ok ? 0u : (1u << j);
      }
    }
    return bad;
  };
  auto fetch = [&](int kt) __attribute__((always_inline)) {
    const int p = kt * 32 + 8 * g;
    int y = 0, x = 0;
    if (is_b && !PW) {
      y = (int)fW.div(AL ? kt * 32 : min(p, D - 1));
      x = p - y * W;
    }
    if (vec) {
      const unsigned bad = outside(in_rows[0], dy[0], dx[0], p, y, x);
      const uint32_t voff = (uint32_t)base[0] + (uint32_t)(p * Ct) * 4u;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                      rsrc, ((bad >> j) & 1u) ? kDmaPastEnd : voff + (uint32_t)(j * Ct) * 4u,
                                                      0, 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) st[i][j] = v[i];
      }
    } else {
      static_for<0, NR>([&](auto it) __attribute__((always_inline)) {
        constexpr int i = decltype(it)::value;
        const unsigned bad = outside(in_rows[i], dy[i], dx[i], p, y, x);
        const uint32_t voff = (uint32_t)base[i] + (uint32_t)(p * Ct) * 4u;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          st[i][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                   rsrc, ((bad >> j) & 1u) ? kDmaPastEnd : voff + (uint32_t)(j * Ct) * 4u, 0, 0));
      });
    }
  };
  // the row tile's first column tile also sums its cotangents over the pixels (the bias columns):
  // they pass through these registers anyway
  const bool sums = !is_b && tn == 0 && pr.bias >= 0;
  float rs[4] = {};
  auto stage = [&](float* dst) __attribute__((always_inline)) {
    if (!active) return;
    if (sums)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        rs[i] += ((st[i][0] + st[i][1]) + (st[i][2] + st[i][3])) + ((st[i][4] + st[i][5]) + (st[i][6] + st[i][7]));
    float* d = dst + (is_b ? AF : 0);
    static_for<0, 4>([&](auto it) __attribute__((always_inline)) {
      constexpr int i = decltype(it)::value;
      const f32x4 x = {st[i][0], st[i][1], st[i][2], st[i][3]}, y = {st[i][4], st[i][5], st[i][6], st[i][7]};
      f16x8 hi, lo;
      pair_split8(x, y, sf[i], hi, lo);
      const int r = row + i;
      *reinterpret_cast<f16x8*>(&d[r * 32 + (wg_swz(r, 2 * g) << 2)]) = hi;
      *reinterpret_cast<f16x8*>(&d[r * 32 + (wg_swz(r, 2 * g + 1) << 2)]) = lo;
    });
  };
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  fetch(0);
  stage(smem);
  __syncthreads();
  f16x8 a[2][2], b[2][Cfg::FN][2];
  auto frag = [&](const float* st_, int r, int c) {
    return *reinterpret_cast<const f16x8*>(&st_[r * 32 + (wg_swz(r, c) << 2)]);
  };
  auto load_a = [&](const float* st_, int half, int i, f16x8 (&x)[2]) {
#pragma unroll
    for (int p = 0; p < 2; ++p) x[p] = frag(st_, wm0 + i * 32 + lr, half * 4 + lc + p);
  };
  auto load_b = [&](const float* st_, int half, f16x8 (&x)[Cfg::FN][2]) {
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p) x[j][p] = frag(st_ + AF, wn0 + j * 32 + lr, half * 4 + lc + p);
  };
  auto mma = [&](int i, const f16x8 (&x)[2], const f16x8 (&y)[Cfg::FN][2]) {
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
  auto tile = [&](int kt, auto stage_tag) {
    constexpr int S = decltype(stage_tag)::value;
    const float* cur = smem + S * STAGE;
    if (kt + 1 < nk) fetch(kt + 1);
    load_b(cur, 0, b[0]);
    load_a(cur, 0, 0, a[0]);
#pragma unroll
    for (int z = 0; z < 2 * Cfg::FM; ++z) {
      const int half = z / Cfg::FM, next = (z + 1) / Cfg::FM;
      if (z + 1 < 2 * Cfg::FM) {
        if (next != half) load_b(cur, next, b[1]);
        load_a(cur, next, (z + 1) % Cfg::FM, a[(z + 1) & 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      mma(z % Cfg::FM, a[z & 1], b[half]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the other stage was last read in tile kt - 1, which every wave has left
    if (kt + 1 < nk) stage(smem + (S ^ 1) * STAGE);
    __syncthreads();
  };
  int kb = 0;
  for (; kb + 2 <= nk; kb += 2) {
    tile(kb, std::integral_constant<int, 0>{});
    tile(kb + 1, std::integral_constant<int, 1>{});
  }
  if (kb < nk) tile(kb, std::integral_constant<int, 0>{});
  if (tn == 0 && pr.bias >= 0) {   // every wave has left the stages
    if (sums)
#pragma unroll
      for (int i = 0; i < 4; ++i) smem[g * Cfg::BM + row + i] = rs[i];
    __syncthreads();
    const int r = m0 + threadIdx.x;
    if (threadIdx.x < Cfg::BM && r < O * C) {
      const int o = (int)fC.div(r);
      J[((long long)s * O + o) * ldJ + pr.bias + (r - o * C)] =
          (smem[threadIdx.x] + smem[Cfg::BM + threadIdx.x]) + (smem[2 * Cfg::BM + threadIdx.x] + smem[3 * Cfg::BM + threadIdx.x]);
    }
  }
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int e = row_exp(m0 + wm0 + i * 32 + frag_row(v, lane)) + eh;
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j) acc[i][j][v] = ldexpf(acc[i][j][v], e);
    }
  conv_wgrad_store<Cfg>(acc, m0, n0, s, O, fC, KC, fCin, Cst, J, ldJ, off);
}

// Grid of the per-sample weight-space products: the tiles of one sample on one XCD, so the
// column tiles that share a block of cotangent rows (and the row tiles that share the patch
// columns) read them through one L2 (xcd_sample_tile).
static unsigned wgrad_grid(int tiles, int images) { return (unsigned)(8 * ((images + 7) / 8) * tiles); }

// Pairs need a workgroup per compute unit: a K tile's loads and splits are one serial chain, which
// other workgroups have to hide.  38 workgroups of 23 K tiles: 72 us, 51 with the fp32 form; 152:
// 31 and 20; 294: 66 and 106.
constexpr long long kConvWgPairMinGroups = 256;
bool conv_wgrad_takes_pairs(int images, int O, int H, int W, int C, int Cin, bool pw) {
  const int KC = (pw ? 1 : 9) * Cin;
  const bool spans = (long long)O * H * W * C * 4 < (1LL << 31) && ((long long)H * W + W + 1) * Cin * 4 < (1LL << 31);
  const long long tiles = KC <= 64 ? (long long)cdiv(O * C, CfgConvWgPairN::BM)
                          : O * C <= 64 ? (long long)cdiv(KC, CfgConvWgPairM::BN)
                                        : (long long)cdiv(O * C, CfgConvWgPair::BM) * cdiv(KC, CfgConvWgPair::BN);
  return spans && tiles * images >= kConvWgPairMinGroups;
}

template <bool VA, bool VB, bool PW>
static hipError_t conv_wgrad_vec(hipStream_t s, const float* G, const float* h, int images, int O,
                                 int H, int W, int C, int Cin, float* J, long long ldJ, long long off) {
  using Cfg = CfgConv;
  using LA = LoadCotangentKOuterT<VA>;
  using LB = std::conditional_t<PW, LoadCotangentKOuterT<VB>, LoadPatchesKOuterT<VB>>;
  const int tn = cdiv((PW ? 1 : 9) * Cin, Cfg::BN), tm = cdiv(O * C, Cfg::BM);
  hipError_t e = set_smem<Cfg, LA, LB>((const void*)k_conv_wgrad<Cfg, VA, VB, PW>);
  if (e != hipSuccess) return e;
  k_conv_wgrad<Cfg, VA, VB, PW><<<dim3(wgrad_grid(tm * tn, images)), dim3(Cfg::THREADS),
                                  gemm_smem_bytes<Cfg, LA, LB>(), s>>>(
      G, h, O, H, W, C, Cin, FastDiv((uint32_t)C), FastDiv((uint32_t)W), FastDiv((uint32_t)Cin), J,
      ldJ, off, tm, tn, images);
  return hipGetLastError();
}

// Per-sample weight-space product of a 3x3 (PW = false: columns (tap, ci) of the patches) or a
// pointwise (PW = true: columns ci of the layer input) convolution.
template <bool PW>
static hipError_t conv_wgrad_any(hipStream_t s, const float* G, const float* h, int images, int O, int H,
                                 int W, int C, int Cin, float* J, long long ldJ, long long off, int Cst,
                                 const ConvPairWgrad* pair, bool* bias_done) {
  const int KC = (PW ? 1 : 9) * Cin;
  if ((long long)8 * ((images + 7) / 8) * cdiv(KC, CfgConv::BN) * cdiv((long long)O * C, CfgConv::BM) >=
      (1LL << 31))
    return hipErrorInvalidValue;
  if (pair && conv_wgrad_takes_pairs(images, O, H, W, C, Cin, PW)) {
    if (bias_done) *bias_done = pair->bias >= 0;
    const bool va = C % 4 == 0 && aligned16(G), vb = Cin % 4 == 0 && aligned16(h);
    const bool al = va && vb && (PW ? (H * W) % 32 == 0 : W % 32 == 0);
    auto go = [&](auto cfg_tag, auto al_tag, auto va_tag, auto vb_tag) -> hipError_t {
      using Cfg = decltype(cfg_tag);
      constexpr bool AL = decltype(al_tag)::value, VA = decltype(va_tag)::value, VB = decltype(vb_tag)::value;
      const int tn = cdiv(KC, Cfg::BN), tm = cdiv(O * C, Cfg::BM);
      constexpr int bytes = gemm_dma_smem_bytes<Cfg, 2>();
      hipError_t e = hipFuncSetAttribute((const void*)k_conv_wgrad_pair<Cfg, PW, AL, VA, VB>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
      if (e != hipSuccess) return e;
      k_conv_wgrad_pair<Cfg, PW, AL, VA, VB><<<dim3(wgrad_grid(tm * tn, images)), dim3(Cfg::THREADS), bytes, s>>>(
          G, h, *pair, O, H, W, C, Cin, FastDiv((uint32_t)C), FastDiv((uint32_t)W), FastDiv((uint32_t)Cin), Cst, J, ldJ,
          off, tm, tn, images);
      return hipGetLastError();
    };
    auto gov = [&](auto cfg_tag) -> hipError_t {
      using T = std::true_type;
      using F = std::false_type;
      if (al) return go(cfg_tag, T{}, T{}, T{});
      if (va) return vb ? go(cfg_tag, F{}, T{}, T{}) : go(cfg_tag, F{}, T{}, F{});
      return vb ? go(cfg_tag, F{}, F{}, T{}) : go(cfg_tag, F{}, F{}, F{});
    };
    // few columns (the 3-channel first layer, a pointwise layer): half-width tiles; few rows (one
    // output, as for the folded last convolution): 64 x 64, for enough workgroups
    if (KC <= 64) return gov(CfgConvWgPairN{});
    if (O * C <= 64) return gov(CfgConvWgPairM{});
    return gov(CfgConvWgPair{});
  }
  // direct-to-LDS: one sample's cotangents and layer input each within a buffer resource
  if (C % 4 == 0 && Cin % 4 == 0 && aligned16(G) && aligned16(h) && (long long)O * H * W * C * 4 < (1LL << 31) &&
      (long long)H * W * Cin * 4 < (1LL << 31)) {
    constexpr int NS = kConvWgStages;
    auto go = [&](auto cfg_tag, auto al_tag) -> hipError_t {
      using Cfg = decltype(cfg_tag);
      constexpr bool AL = decltype(al_tag)::value;
      const int tn = cdiv(KC, Cfg::BN), tm = cdiv(O * C, Cfg::BM);
      constexpr int bytes = gemm_dma_smem_bytes<Cfg, NS>();
      hipError_t e = hipFuncSetAttribute((const void*)k_conv_wgrad_dma<Cfg, NS, PW, AL>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
      if (e != hipSuccess) return e;
      k_conv_wgrad_dma<Cfg, NS, PW, AL><<<dim3(wgrad_grid(tm * tn, images)), dim3(Cfg::THREADS), bytes, s>>>(
          G, h, O, H, W, C, Cin, FastDiv((uint32_t)C), FastDiv((uint32_t)W), FastDiv((uint32_t)Cin), Cst, J,
          ldJ, off, tm, tn, images);
      return hipGetLastError();
    };
    const bool al = PW ? (H * W) % 32 == 0 : W % 32 == 0;
    // at most 64 rows (O C: one output, as for the folded last convolution): 64 x 64 tiles
    if (O * C <= 64)
      return al ? go(CfgConvWgSmall{}, std::true_type{}) : go(CfgConvWgSmall{}, std::false_type{});
    return al ? go(CfgConvWg{}, std::true_type{}) : go(CfgConvWg{}, std::false_type{});
  }
  if (Cst != Cin) return hipErrorInvalidValue;   // padded inputs take the direct-to-LDS form only
  const bool va = C % 4 == 0 && aligned16(G), vb = Cin % 4 == 0 && aligned16(h);
  if (va && vb) return conv_wgrad_vec<true, true, PW>(s, G, h, images, O, H, W, C, Cin, J, ldJ, off);
  if (va) return conv_wgrad_vec<true, false, PW>(s, G, h, images, O, H, W, C, Cin, J, ldJ, off);
  return conv_wgrad_vec<false, false, PW>(s, G, h, images, O, H, W, C, Cin, J, ldJ, off);
}

hipError_t launch_conv_wgrad(hipStream_t s, const float* G, const float* h, int images, int O, int H,
                             int W, int C, int Cin, float* J, long long ldJ, long long off,
                             const ConvPairWgrad* pair, bool* bias_done) {
  return conv_wgrad_any<false>(s, G, h, images, O, H, W, C, Cin, J, ldJ, off, Cin, pair, bias_done);
}

hipError_t launch_pw_wgrad(hipStream_t s, const float* G, const float* h, int images, int O, int H, int W,
                           int C, int Cin, float* J, long long ldJ, long long off, const ConvPairWgrad* pair, bool* bias_done) {
  return conv_wgrad_any<true>(s, G, h, images, O, H, W, C, Cin, J, ldJ, off, Cin, pair, bias_done);
}

// xp [rows, Cp] = x [rows, Cin] with zero channels Cin .. Cp - 1.
__global__ void __launch_bounds__(256)
k_pad_channels(const float* __restrict__ x, long long rows, int Cin, int Cp, float* __restrict__ xp) {
  const long long total = rows * Cp;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
    const long long r = i / Cp;
    const int c = (int)(i - r * Cp);
    xp[i] = c < Cin ? x[r * Cin + c] : 0.f;
  }
}

// (images of fewer than kPadMinPixels pixels keep the register-staged form: a few K tiles per
// sample do not repay the copy; 4x4 images measured slower padded)
constexpr int kPadMinPixels = 256;
bool conv_wgrad_pad_ok(int images, int O, int H, int W, int C, int Cin, const float* G, const float* xp) {
  const int Cp = (Cin + 3) & ~3;
  return Cin % 4 != 0 && C % 4 == 0 && H * W >= kPadMinPixels && aligned16(G) && aligned16(xp) &&
         (long long)O * H * W * C * 4 < (1LL << 31) && (long long)H * W * Cp * 4 < (1LL << 31) &&
         (long long)images * H * W * Cp < (1LL << 40);
}

hipError_t launch_conv_wgrad_padded(hipStream_t s, const float* G, const float* h, float* xp, int images, int O,
                                    int H, int W, int C, int Cin, float* J, long long ldJ, long long off, bool pw,
                                    const ConvPairWgrad* pair, bool* bias_done) {
  const int Cp = (Cin + 3) & ~3;
  if (!conv_wgrad_pad_ok(images, O, H, W, C, Cin, G, xp)) return hipErrorInvalidValue;
  const long long rows = (long long)images * H * W;
  k_pad_channels<<<dim3((unsigned)std::min<long long>((rows * Cp + 255) / 256, 16384)), dim3(256), 0, s>>>(
      h, rows, Cin, Cp, xp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return pw ? conv_wgrad_any<true>(s, G, xp, images, O, H, W, C, Cp, J, ldJ, off, Cin, pair, bias_done)
            : conv_wgrad_any<false>(s, G, xp, images, O, H, W, C, Cp, J, ldJ, off, Cin, pair, bias_done);
}

// ------------------------------------------------------------------------------ split-K J1 J2^T
__device__ __forceinline__ void tri_index_c(int t, int nt, int& tm, int& tn) {
  int r = 0, base = 0;
  while (base + (nt - r) <= t) {
    base += nt - r;
    ++r;
  }
  tm = r;
  tn = r + (t - base);
}

// part[z][r1][r2] = sum_{k in chunk z} J1[r1, k] J2[r2, k]
template <class Cfg, bool VEC>
__global__ void __launch_bounds__(Cfg::THREADS)
k_ntk_splitk(LoadKInnerT<VEC> la, LoadKInnerT<VEC> lb, int chunk, int symmetric, float* __restrict__ part,
             int tiles_n) {
  extern __shared__ float smem[];
  const int z = blockIdx.y;
  int tm, tn;
  if (symmetric) {
    tri_index_c(blockIdx.x, tiles_n, tm, tn);
  } else {
    tm = blockIdx.x / tiles_n;
    tn = blockIdx.x % tiles_n;
  }
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  const int k0 = z * chunk;
  const int k1 = min(la.K, k0 + chunk);
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  gemm_mainloop<Cfg>(la, lb, m0, n0, k0, k1, smem, acc);
  const int R1 = la.rows, R2 = lb.rows;
  float* P = part + (long long)z * R1 * R2;
  for_each_acc<Cfg>(acc, m0, n0, [&](int r, int c, float v) {
    if (r < R1 && c < R2) P[(long long)r * R2 + c] = v;
  });
}

// Direct-to-LDS form (K-contiguous 16-byte aligned rows, K % 32 == 0): the same products, with
// the work items ordered per XCD.  The items (chunk z, tile t) are numbered chunk by chunk,
// i = z * tiles + t, and cut into 8 equal contiguous ranges, one per XCD.  Workgroup b runs on
// XCD x = b % 8 (the hardware hands out workgroup ids round robin over the 8 XCDs) and takes
// the (b / 8)-th item of range x, so the tiles of a chunk run together on one XCD and share its
// L2 for the rows of J1 and J2 they read.
template <class Cfg>
__global__ void __launch_bounds__(Cfg::THREADS)
k_ntk_splitk_dma(const float* __restrict__ J1, const float* __restrict__ J2, int R1, int R2, int K,
                 long long ld, int chunk, int splits, int tiles, int symmetric, float* __restrict__ part,
                 int tiles_n) {
  extern __shared__ float smem[];
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  const long long items = (long long)tiles * splits;
  const long long i = x * items / 8 + j;
  if (i >= (x + 1) * items / 8) return;
  const int z = (int)(i / tiles), t = (int)(i - (long long)z * tiles);
  int tm, tn;
  if (symmetric) {
    tri_index_c(t, tiles_n, tm, tn);
  } else {
    tm = t / tiles_n;
    tn = t % tiles_n;
  }
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  const int k0 = z * chunk;
  const int k1 = min(K, k0 + chunk);
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  gemm_mainloop_dma<Cfg, 2>(J1, ld, R1, J2, ld, R2, m0, n0, k0, k1, smem, acc);
  float* P = part + (long long)z * R1 * R2;
  for_each_acc<Cfg>(acc, m0, n0, [&](int r, int c, float v) {
    if (r < R1 && c < R2) P[(long long)r * R2 + c] = v;
  });
}

// The same products on pairs, split into f16 values on the way through registers into LDS (a thread:
// 8 k of a row, four threads a row's K tile; two LDS stages, the next tile's loads in flight during the
// MFMAs).  No row maxima are known before, so a row's exponent follows what has been read: it starts
// from its first K tile with two bits to spare, and a K tile that passes the top raises it, which
// scales the row's (column's) sums so far by the power of two in between.  The decision is per K
// tile and workgroup, through flags and exponent steps in LDS beside the stage; past the first tiles
// of a chunk it is rare.  Bound by the MFMAs and the splits: 640 x 640 x 75 456: 553 us
// with the fp32 MFMA (112 TF/s), 313 here (197 TF/s).
template <class Cfg, bool VEC>
__global__ void __launch_bounds__(Cfg::THREADS, 2)
k_ntk_splitk_pair(const float* __restrict__ J1, const float* __restrict__ J2, int R1, int R2, int K, long long ld,
                  int chunk, int splits, int tiles, int symmetric, float* __restrict__ part, int tiles_n) {
  constexpr int ROWS = Cfg::BM + Cfg::BN, STAGE = ROWS * 32, NT = ROWS * 4 / Cfg::THREADS;
  static_assert(Cfg::THREADS == 256 && Cfg::BM % 64 == 0 && Cfg::BN % 64 == 0, "64 rows of one operand per task");
  extern __shared__ f32x4 sk_lds[];   // 16-byte aligned
  float* smem = reinterpret_cast<float*>(sk_lds);
  int* steps = reinterpret_cast<int*>(smem + 2 * STAGE);   // [2][ROWS]
  int* flags = steps + 2 * ROWS;                           // [2][4], per wave
  const int x = blockIdx.x & 7, jb = blockIdx.x >> 3;
  const long long items = (long long)tiles * splits;
  const long long item = x * items / 8 + jb;
  if (item >= (x + 1) * items / 8) return;
  const int z = (int)(item / tiles), t = (int)(item - (long long)z * tiles);
  int tm, tn;
  if (symmetric) {
    tri_index_c(t, tiles_n, tm, tn);
  } else {
    tm = t / tiles_n;
    tn = t % tiles_n;
  }
  const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
  const int k0 = z * chunk, k1 = min(K, k0 + chunk), nk = (k1 - k0 + 31) / 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm0 = (wave / Cfg::WAVES_N) * Cfg::WM, wn0 = (wave % Cfg::WAVES_N) * Cfg::WN;
  const int lr = lane & 31, lc = (lane >> 5) * 2;
  const int g = threadIdx.x & 3, trow = threadIdx.x >> 2;
  // rows of a tile through buffer resources; a row past the operand or a k past the chunk reads zeros
  const int rows_a = min(Cfg::BM, R1 - m0), rows_b = min(Cfg::BN, R2 - n0);
  const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(J1 + m0 * ld, (uint32_t)(((rows_a - 1) * ld + K) * 4));
  const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(J2 + n0 * ld, (uint32_t)(((rows_b - 1) * ld + K) * 4));
  int exps[NT];
  static_for<0, NT>([&](auto it) __attribute__((always_inline)) { exps[decltype(it)::value] = -126; });
  f32x4 st[NT][2];
  auto fetch = [&](int kt) __attribute__((always_inline)) {
    const int k = k0 + kt * 32 + 8 * g;
    static_for<0, NT>([&](auto it) __attribute__((always_inline)) {
      constexpr int i = decltype(it)::value;
      constexpr bool is_b = i * 64 >= Cfg::BM;
      const int r = i * 64 - (is_b ? Cfg::BM : 0) + trow;
      const bool in = r < (is_b ? rows_b : rows_a);
      const uint32_t voff = ((uint32_t)r * (uint32_t)ld + (uint32_t)k) * 4u;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (VEC) {
          st[i][h] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                   is_b ? rb : ra, in && k + 4 * h < k1 ? voff + 16u * h : kDmaPastEnd, 0, 0));
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            st[i][h][j] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(
                           is_b ? rb : ra, in && k + 4 * h + j < k1 ? voff + 16u * h + 4u * j : kDmaPastEnd, 0, 0));
        }
      }
    });
  };
  auto swz = [](int r, int c) { return c ^ (r & 7); };
  auto stage = [&](int sidx) __attribute__((always_inline)) {
    float* d = smem + sidx * STAGE;
    bool raised = false;
    static_for<0, NT>([&](auto it) __attribute__((always_inline)) {
      constexpr int i = decltype(it)::value;
      const f32x4 u = st[i][0], v = st[i][1];
      float m = fmaxf(fmaxf(fmaxf(fabsf(u[0]), fabsf(u[1])), fmaxf(fabsf(u[2]), fabsf(u[3]))),
                      fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
      m = fmaxf(m, __shfl_xor(m, 1));
      m = fmaxf(m, __shfl_xor(m, 2));
      const int e = m > 0.f ? pair_row_exp(m) : -126, step = e > exps[i] ? exps[i] - (e + 2) : 0;
      exps[i] -= step;
      raised = raised || step != 0;
      const int r = i * 64 + trow;
      if (g == 0) steps[sidx * ROWS + r] = step;
      f16x8 hi, lo;
      pair_split8(u, v, pair_factor(exps[i]), hi, lo);
      *reinterpret_cast<f16x8*>(&d[r * 32 + (swz(r, 2 * g) << 2)]) = hi;
      *reinterpret_cast<f16x8*>(&d[r * 32 + (swz(r, 2 * g + 1) << 2)]) = lo;
    });
    const int any = __any(raised) ? 1 : 0;
    if (lane == 0) flags[sidx * 4 + wave] = any;
  };
  f32x16 acc[Cfg::FM][Cfg::FN];
  zero_acc<Cfg>(acc);
  // acc[r][c] times 2^(v[r] + v[BM + c]), v in LDS
  auto scale = [&](const int* v) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) {
      const int ec = v[Cfg::BM + wn0 + j * 32 + lr];
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
        for (int q = 0; q < 16; ++q)
          acc[i][j][q] = ldexpf(acc[i][j][q], v[wm0 + i * 32 + frag_row(q, lane)] + ec);
    }
  };
  auto frag = [&](const float* p, int r, int c) __attribute__((always_inline)) {
    return *reinterpret_cast<const f16x8*>(&p[r * 32 + (swz(r, c) << 2)]);
  };
  auto tile = [&](int kt, auto stage_tag) __attribute__((always_inline)) {
    constexpr int S = decltype(stage_tag)::value;
    const float* cur = smem + S * STAGE;
    if (kt + 1 < nk) fetch(kt + 1);
    if (__builtin_amdgcn_readfirstlane(flags[S * 4] | flags[S * 4 + 1] | flags[S * 4 + 2] | flags[S * 4 + 3]))
      scale(steps + S * ROWS);
    f16x8 a[2][2], b[Cfg::FN][2];
    static_for<0, 2>([&](auto ht) __attribute__((always_inline)) {
      constexpr int half = decltype(ht)::value;
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
        for (int p = 0; p < 2; ++p) b[j][p] = frag(cur, Cfg::BM + wn0 + j * 32 + lr, half * 4 + lc + p);
      static_for<0, Cfg::FM>([&](auto it) __attribute__((always_inline)) {
        constexpr int i = decltype(it)::value;
#pragma unroll
        for (int p = 0; p < 2; ++p) a[i & 1][p] = frag(cur, wm0 + i * 32 + lr, half * 4 + lc + p);
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i & 1][1], b[j][0], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i & 1][0], b[j][1], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i & 1][0], b[j][0], acc[i][j], 0, 0, 0);
      });
    });
    // the other stage, its steps and flags were last read in tile kt - 1, which every wave has left
    if (kt + 1 < nk) stage(S ^ 1);
    __syncthreads();
  };
  fetch(0);
  stage(0);
  __syncthreads();
  int kb = 0;
  for (; kb + 2 <= nk; kb += 2) {
    tile(kb, std::integral_constant<int, 0>{});
    tile(kb + 1, std::integral_constant<int, 1>{});
  }
  if (kb < nk) tile(kb, std::integral_constant<int, 0>{});
  static_for<0, NT>([&](auto it) __attribute__((always_inline)) {
    constexpr int i = decltype(it)::value;
    if (g == 0) steps[i * 64 + trow] = exps[i];
  });
  __syncthreads();
  scale(steps);
  float* P = part + (long long)z * R1 * R2;
  for_each_acc<Cfg>(acc, m0, n0, [&](int r, int c, float v) {
    if (r < R1 && c < R2) P[(long long)r * R2 + c] = v;
  });
}

// theta[n1][n2][o1][o2] = w[n1, n2] sum_z part[z][r1][r2] + (o1 == o2) rscale gram[n1, n2], or,
// with accumulate, theta += w[n1, n2] sum_z part[z][r1][r2] (the readout summand is then
// already in theta).  w = null means 1; gram = null means no readout summand.
// ZG threads per entry, each a contiguous range of the partials, added in order through LDS: with few
// entries and many partials (64 x 64 entries, 295 partials: 35 us with ZG = 1, 9 with 8) one thread's
// chain of loads would be all there is.
template <int ZG>
__global__ void __launch_bounds__(256)
k_ntk_reduce(const float* __restrict__ part, int splits, int N1, int N2, int O,
             int symmetric, const float* __restrict__ w,
             const float* __restrict__ gram, float rscale, int accumulate,
             float* __restrict__ theta) {
  constexpr int EB = 256 / ZG;   // entries per workgroup and pass
  __shared__ float sums[ZG > 1 ? 256 : 1];
  const int R1 = N1 * O, R2 = N2 * O;   // below 2^31: the launcher checked them
  const long long total = (long long)R1 * R2;
  const int zg = ZG > 1 ? threadIdx.x / EB : 0, te = ZG > 1 ? threadIdx.x % EB : threadIdx.x;
  const int z0 = ZG > 1 ? (int)((long long)splits * zg / ZG) : 0;
  const int z1 = ZG > 1 ? (int)((long long)splits * (zg + 1) / ZG) : splits;
  for (long long i0 = blockIdx.x * (long long)EB; i0 < total; i0 += (long long)gridDim.x * EB) {
    const long long i = i0 + te;
    if (ZG == 1 && i >= total) return;   // later passes of this thread lie further on
    const int r1 = (int)(min(i, total - 1) / R2), r2 = (int)(min(i, total - 1) - (long long)r1 * R2);
    bool direct, mirror;
    sym_writes(symmetric, r1, r2, direct, mirror);
    const bool in = i < total && direct;
    float v = 0.f;
    if (in) {
      const long long src = i;
      float a[4] = {0.f, 0.f, 0.f, 0.f};   // four independent chains keep several loads in flight
      int z = z0;
      for (; z + 4 <= z1; z += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] += part[(long long)(z + u) * total + src];
      }
      for (; z < z1; ++z) a[0] += part[(long long)z * total + src];
      v = (a[0] + a[1]) + (a[2] + a[3]);
    }
    if (ZG > 1) {
      sums[threadIdx.x] = v;
      __syncthreads();
      if (zg == 0) {
        v = 0.f;
#pragma unroll
        for (int u = 0; u < ZG; ++u) v += sums[u * EB + te];
      }
      __syncthreads();
    }
    if (!in || zg) continue;
    const int n1 = r1 / O, o1 = r1 - n1 * O, n2 = r2 / O, o2 = r2 - n2 * O;
    if (w) v *= w[(long long)n1 * N2 + n2];
    if (!accumulate && o1 == o2 && gram) v += rscale * gram[(long long)n1 * N2 + n2];
    float* dst = theta + (((long long)n1 * N2 + n2) * O + o1) * O + o2;
    *dst = accumulate ? *dst + v : v;
    if (mirror) {
      float* dst2 = theta + (((long long)n2 * N1 + n1) * O + o2) * O + o1;
      *dst2 = accumulate ? *dst2 + v : v;
    }
  }
}

int splitk_tile() { return CfgSplitK::BM; }

int splitk_plan(int R1, int R2, long long K, int symmetric, long long part_capacity, int* chunk_out) {
  using Cfg = CfgSplitK;
  const int tm = cdiv(R1, Cfg::BM), tn = cdiv(R2, Cfg::BN);
  const int tiles = symmetric ? tn * (tn + 1) / 2 : tm * tn;
  // aim for about 4 workgroups per compute unit, with chunks that are whole K tiles, and
  // never more partial [R1, R2] products than the workspace holds
  long long want = std::min<long long>(1024 / std::max(tiles, 1), cdiv(K, 256));
  want = std::min<long long>(want, part_capacity / ((long long)R1 * R2));
  int splits = (int)std::max<long long>(1, want);
  long long chunk = (K + splits - 1) / splits;
  chunk = ((chunk + Cfg::BK - 1) / Cfg::BK) * Cfg::BK;
  splits = (int)((K + chunk - 1) / chunk);
  *chunk_out = (int)chunk;
  return splits;
}

template <bool VEC>
static hipError_t splitk_vec(hipStream_t s, const float* J1, const float* J2, int R1, int R2,
                             long long K, long long ld, int symmetric, int chunk, int splits,
                             float* part) {
  using Cfg = CfgSplitK;
  using L = LoadKInnerT<VEC>;
  L la{J1, R1, (int)K, ld};
  L lb{J2, R2, (int)K, ld};
  const int tm = cdiv(R1, Cfg::BM), tn = cdiv(R2, Cfg::BN);
  const int tiles = symmetric ? tn * (tn + 1) / 2 : tm * tn;
  hipError_t e = set_smem<Cfg, L, L>((const void*)k_ntk_splitk<Cfg, VEC>);
  if (e != hipSuccess) return e;
  k_ntk_splitk<Cfg, VEC><<<dim3(tiles, splits), dim3(Cfg::THREADS), gemm_smem_bytes<Cfg, L, L>(), s>>>(
      la, lb, chunk, symmetric, part, tn);
  return hipGetLastError();
}

// Pairs from 0.3 GFLOP and 4096 columns on: 64 x 64 x 75 000, 38 us with the fp32 MFMA, 25 with pairs;
// 217 x 126 x 10 700, 24 and 21.  640 x 640 x 1728 (chunks of eight K tiles, the first of which sets the
// exponents): 22 us either way, the evaluation around it 315 and 318.
constexpr double kSplitKPairMinFlops = 3e8;
constexpr long long kSplitKPairMinK = 4096;
hipError_t launch_ntk_splitk(hipStream_t s, const float* J1, const float* J2, int R1, int R2,
                             long long K, long long ld, int symmetric, int chunk, int splits,
                             float* part, bool pairs) {
  if (pairs && K >= kSplitKPairMinK && 2.0 * R1 * R2 * K >= kSplitKPairMinFlops && dma_span_ok(ld, K, 128)) {
    using Cfg = CfgSplitK;
    const int tm = cdiv(R1, Cfg::BM), tn = cdiv(R2, Cfg::BN);
    const int tiles = symmetric ? tn * (tn + 1) / 2 : tm * tn;
    constexpr int rows = Cfg::BM + Cfg::BN, bytes = 2 * rows * 128 + 2 * rows * 4 + 32;
    const unsigned blocks = (unsigned)(8 * (((long long)tiles * splits + 7) / 8));
    auto go = [&](auto vec_tag) -> hipError_t {
      constexpr bool VEC = decltype(vec_tag)::value;
      hipError_t e = hipFuncSetAttribute((const void*)k_ntk_splitk_pair<Cfg, VEC>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
      if (e != hipSuccess) return e;
      k_ntk_splitk_pair<Cfg, VEC><<<dim3(blocks), dim3(Cfg::THREADS), bytes, s>>>(
          J1, J2, R1, R2, (int)K, ld, chunk, splits, tiles, symmetric, part, tn);
      return hipGetLastError();
    };
    return vec_ok(J1, ld, K) && vec_ok(J2, ld, K) ? go(std::true_type{}) : go(std::false_type{});
  }
  if (vec_ok(J1, ld, K) && vec_ok(J2, ld, K) && K % 32 == 0 && chunk % 32 == 0 && dma_span_ok(ld, K, 128)) {
    using Cfg = CfgSplitKDma;
    static_assert(Cfg::BM == CfgSplitK::BM && Cfg::BN == CfgSplitK::BN, "the reduction's tile grid");
    const int tm = cdiv(R1, Cfg::BM), tn = cdiv(R2, Cfg::BN);
    const int tiles = symmetric ? tn * (tn + 1) / 2 : tm * tn;
    constexpr int bytes = gemm_dma_smem_bytes<Cfg, 2>();
    hipError_t e = hipFuncSetAttribute((const void*)k_ntk_splitk_dma<Cfg>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    const long long blocks = 8 * (((long long)tiles * splits + 7) / 8);
    k_ntk_splitk_dma<Cfg><<<dim3((unsigned)blocks), dim3(Cfg::THREADS), bytes, s>>>(
        J1, J2, R1, R2, (int)K, ld, chunk, splits, tiles, symmetric, part, tn);
    return hipGetLastError();
  }
  if (vec_ok(J1, ld, K) && vec_ok(J2, ld, K))
    return splitk_vec<true>(s, J1, J2, R1, R2, K, ld, symmetric, chunk, splits, part);
  return splitk_vec<false>(s, J1, J2, R1, R2, K, ld, symmetric, chunk, splits, part);
}

hipError_t launch_ntk_reduce(hipStream_t s, const float* part, int splits, int N1, int N2, int O,
                             int symmetric, const float* w, const float* gram, float rscale,
                             int accumulate, float* theta) {
  int R1, R2;
  if (!to_int((long long)N1 * O, R1) || !to_int((long long)N2 * O, R2)) return hipErrorInvalidValue;
  const long long total = (long long)R1 * R2;
  auto go = [&](auto zg_tag) {
    constexpr int ZG = decltype(zg_tag)::value, EB = 256 / ZG;
    k_ntk_reduce<ZG><<<dim3((unsigned)std::min<long long>((total + EB - 1) / EB, 256 * 64)), dim3(256), 0, s>>>(
        part, splits, N1, N2, O, symmetric, w, gram, rscale, accumulate, theta);
  };
  // one thread per entry from two workgroups a compute unit on, or for a few partials
  if (total < 512 * 256 && splits >= 16)
    go(std::integral_constant<int, 8>{});
  else
    go(std::integral_constant<int, 1>{});
  return hipGetLastError();
}

}  // namespace ntk
