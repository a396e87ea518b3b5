// cnn.hip -- BF16 MFMA kernels of the corrector network (see cnn.hpp).
#include "cnn.hpp"

#include <cstring>

#include "common.hpp"

namespace le {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
// wide loads from a caller's arrays, which need only their elements' alignment
typedef unsigned short u16x8_any __attribute__((ext_vector_type(8), aligned(2)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));
typedef unsigned u32_any __attribute__((aligned(2)));

constexpr int kOffW[kCnnLayers] = {0, 608, 9856, 19104};
constexpr int kOffB[kCnnLayers] = {576, 9824, 19072, 19680};

// A training step takes as many samples at once as hold kGroupPixels pixels
// (850 to 1010 B each; 16 of 256^2: 655 us per step, in groups of 8 705, of 4 830).
// Blocks over the tiles of a batch: three per CU, as many as are resident, of
// the 32-channel forward (1024 blocks: 66 -> 64 us, last layer 38 -> 32), four
// of the others; of the weight gradient as many as are resident, so that its
// partials (37 KB per block in the middle layers) are few.
constexpr int kGroupPixels = 1 << 20;
constexpr int kFwdBlocks = 768, kConvBlocks = 1024;
constexpr int kDwBlocks[kCnnLayers] = {1024, 512, 512, 1024};

constexpr int pad16(int k) { return (k + 15) / 16 * 16; }
constexpr int pad32(int k) { return (k + 31) / 32 * 32; }

// FP32 -> BF16, round to nearest even (the hardware conversion).
__device__ __forceinline__ uint16_t f2bf(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// c += a b for one 32x32x16 tile.  Lane l holds A[l % 32][8 (l / 32) + e],
// B[8 (l / 32) + e][l % 32] (e < 8) and C[8 (r / 4) + 4 (l / 32) + r % 4][l % 32]
// in register r < 16.
__device__ __forceinline__ f32x16 mfma(u16x8 a, u16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ int c_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// Logistic function from the hardware base-2 exponential and reciprocal
// (about 1 ulp each: far below the BF16 rounding of the activations).
__device__ __forceinline__ float sigmoid(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}
__device__ __forceinline__ float silu(float z) { return z * sigmoid(z); }
__device__ __forceinline__ float silu_grad(float z) {
  const float s = sigmoid(z);
  return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------- tiles
//
// The per-layer kernels take tiles of 16 x 16 pixels in turn (ntiles over all
// samples) and stage each tile's operands, with one pixel of halo, once in LDS
// as BF16: every pixel is then read about once from memory instead of once per
// tap, and a batch is one launch per layer.

constexpr int kFT = 16, kFS = 40;   // LDS pixel stride of 32 channels: the 80 bytes
                                    // put 16-byte reads of consecutive pixels on
                                    // distinct banks
constexpr int kHR = kFT + 2;

struct TileAt {
  int y0, x0;
  size_t base;   // the sample's first pixel
};
__device__ __forceinline__ TileAt tile_at(int tile, int H, int W, int lgW) {
  const int tiles_x = W / kFT, tps = tiles_x * (H / kFT);
  const int smp = tile / tps, k = tile - smp * tps;
  return {k / tiles_x * kFT, k % tiles_x * kFT, (size_t)smp * ((size_t)H << lgW)};
}
// Pixel q of the tile with its halo, row by row.
__device__ __forceinline__ size_t halo_px(const TileAt& at, int q, int H, int W, int lgW) {
  const int y = (at.y0 - 1 + q / kHR) & (H - 1), x = (at.x0 - 1 + q % kHR) & (W - 1);
  return at.base + (size_t)((y << lgW) + x);
}
// Pixel pp of the tile's 256.
__device__ __forceinline__ size_t tile_px(const TileAt& at, int pp, int lgW) {
  return at.base + (size_t)(((at.y0 + (pp >> 4)) << lgW) + at.x0 + (pp & 15));
}

// Eight k values, k = tap C + channel, of output pixel (oy, ox) for MFMA step
// ks from the staged tile; FLIP reads the taps mirrored (the input gradient).
template <int C, bool FLIP>
__device__ __forceinline__ u16x8 tile_operand(const uint16_t* in, int oy, int ox, int ks,
                                              int half) {
  auto off = [](int tap) {
    return FLIP ? (2 - tap / 3) * kHR + 2 - tap % 3 : tap / 3 * kHR + tap % 3;
  };
  u16x8 av;
  if constexpr (C == 2) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int ta = ks * 8 + e, tb = ta + 4;   // the tap of each half
      const int oa = ta < 9 ? off(ta) : 0, ob = tb < 9 ? off(tb) : 0;
      unsigned v = 0;
      if (half ? tb < 9 : ta < 9)
        v = *reinterpret_cast<const unsigned*>(in + 2 * (oy * kHR + ox + (half ? ob : oa)));
      av[2 * e] = (uint16_t)(v & 0xffffu);
      av[2 * e + 1] = (uint16_t)(v >> 16);
    }
  } else {
    av = *reinterpret_cast<const u16x8*>(in + (oy * kHR + ox + off(ks / 2)) * kFS +
                                         (ks & 1) * 16 + half * 8);
  }
  return av;
}

// ---------------------------------------------------------------- forward

// z[p][co] = b[co] + sum_{tap, ci} W[co][ci][tap] a[p + tap - (1,1)][ci];
// a_out = bf16(silu(z)) when ACT.  Four wavefronts, each two 32-pixel products
// per tile.  Bound by memory, mostly its writes: 2^20 pixels take 36 us (2 -> 32
// channels, 200 B per pixel), 64 us (32 -> 32, 270 B) and 32 us (32 -> 2).
template <int CIN, int COUT, bool ACT>
__global__ __launch_bounds__(256) void k_conv_fwd(const uint16_t* __restrict__ a_in,
                                                  const uint16_t* __restrict__ wt,
                                                  const float* __restrict__ bias,
                                                  float* __restrict__ z_out,
                                                  uint16_t* __restrict__ a_out, int ntiles,
                                                  int H, int W, int lgW) {
  constexpr int KP = pad16(9 * CIN), NKS = KP / 16;
  __shared__ __align__(16) uint16_t in[kHR * kHR * (CIN == 2 ? 2 : kFS)];
  const int lane = threadIdx.x & 63, half = lane >> 5, i = lane & 31;
  u16x8 bv[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    bv[ks] = *reinterpret_cast<const u16x8*>(wt + (size_t)i * KP + ks * 16 + half * 8);
  const float bc = i < COUT ? bias[i] : 0.f;
  constexpr int G = CIN == 2 ? 1 : 4, NI = kHR * kHR * G, NT = (NI + 255) / 256;
  for (int tile = (int)blockIdx.x; tile < ntiles; tile += (int)gridDim.x) {
    const TileAt at = tile_at(tile, H, W, lgW);
    if constexpr (CIN == 2) {
      unsigned v[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const int q = (int)threadIdx.x + u * 256;
        if (q < NI) v[u] = *reinterpret_cast<const u32_any*>(a_in + halo_px(at, q, H, W, lgW) * 2);
      }
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const int q = (int)threadIdx.x + u * 256;
        if (q < NI) *reinterpret_cast<unsigned*>(in + 2 * q) = v[u];
      }
    } else {
      u16x8 v[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const int it = (int)threadIdx.x + u * 256;
        if (it < NI)
          v[u] = *reinterpret_cast<const u16x8*>(a_in + halo_px(at, it / G, H, W, lgW) * CIN +
                                                 it % G * 8);
      }
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const int it = (int)threadIdx.x + u * 256;
        if (it < NI) *reinterpret_cast<u16x8*>(in + it / G * kFS + it % G * 8) = v[u];
      }
    }
    __syncthreads();
    for (int mt = (int)(threadIdx.x >> 6); mt < kFT * kFT / 32; mt += 4) {
      const int t = mt * 32 + i;
      f32x16 acc = {};
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
        acc = mfma(tile_operand<CIN, false>(in, t >> 4, t & 15, ks, half), bv[ks], acc);
      if (i < COUT) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const size_t e = tile_px(at, mt * 32 + c_row(r, half), lgW) * COUT + i;
          const float z = acc[r] + bc;
          z_out[e] = z;
          if constexpr (ACT) a_out[e] = f2bf(silu(z));
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- fused inference

// The corrected step runs the whole network over one 16 x 16 output tile per
// block.  The state planes of the tile and a 4-pixel halo (one pixel per 3x3
// layer) are read once; every intermediate activation stays in LDS as
// [pixel][kFS] BF16 (32 channels and 8 of padding: an 80-byte pixel stride
// puts the 16-byte reads of consecutive pixels on distinct banks).  Layer l
// computes the (22 - 2l)^2 pixels the next layer needs.  Each value is formed
// with the k order, products and roundings of the per-layer kernel above, so
// it equals the per-layer result bit for bit.
constexpr int kFH = 4, kFR = kFT + 2 * kFH, kFWaves = 8;

// One layer on the tile: input region SIN x SIN (LDS), output region
// (SIN - 2)^2, weights wt in LDS as [COUT][KP + 8] (the 8 of padding spread
// the rows over the banks).  Hidden layers write bf16(silu(z)) to LDS, whole
// 32-pixel tiles of it (a mask per value kept the exponentials of different
// values apart: 256^2 14.0 us per call, without 12.8); the last writes z of both
// channels to z_out at the global pixels (tile origin gy0, gx0) and adds channel
// 0 into zs (FP64, lanes 0 and 32 of each wavefront).
template <int CIN, int SIN, bool LAST>
__device__ __forceinline__ void fused_layer(const uint16_t* __restrict__ in,
                                            uint16_t* __restrict__ out,
                                            const uint16_t* __restrict__ wt,
                                            const float* __restrict__ bias,
                                            float* __restrict__ z_out, int gy0, int gx0, int lgW,
                                            double& zs) {
  constexpr int COUT = LAST ? 2 : 32;
  constexpr int SOUT = SIN - 2, NP = SOUT * SOUT, NT = (NP + 31) / 32;
  constexpr int K = 9 * CIN, KP = pad16(K), NKS = KP / 16;
  const int lane = threadIdx.x & 63, half = lane >> 5, i = lane & 31;
  u16x8 bv[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    bv[ks] = i < COUT ? *reinterpret_cast<const u16x8*>(wt + i * (KP + 8) + ks * 16 + half * 8)
                      : u16x8{};
  const float bc = i < COUT ? bias[i] : 0.f;
  for (int tile = (int)(threadIdx.x >> 6); tile < NT; tile += kFWaves) {
    // rows past the region repeat its last pixel; their results are dropped
    const int t = min(tile * 32 + i, NP - 1);
    const int oy = t / SOUT, ox = t - oy * SOUT;
    u16x8 av[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int k0 = ks * 16 + half * 8;
      if constexpr (CIN == 2) {
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const int k = k0 + e, tap = k / 2;
          unsigned v = 0;
          if (k < K) {
            const int q = (oy + tap / 3) * SIN + ox + tap % 3;
            v = *reinterpret_cast<const unsigned*>(in + 2 * q);
          }
          av[ks][e] = (uint16_t)(v & 0xffffu);
          av[ks][e + 1] = (uint16_t)(v >> 16);
        }
      } else {
        const int tap = k0 / CIN, ci0 = k0 % CIN;
        const int q = (oy + tap / 3) * SIN + ox + tap % 3;
        av[ks] = *reinterpret_cast<const u16x8*>(in + q * kFS + ci0);
      }
    }
    f32x16 acc = {};
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) acc = mfma(av[ks], bv[ks], acc);
    if constexpr (!LAST) {
      // rows past the region land in the buffer's padding
#pragma unroll
      for (int r = 0; r < 16; ++r)
        out[(tile * 32 + c_row(r, half)) * kFS + i] = f2bf(silu(acc[r] + bc));
    } else if (i < COUT) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int tt = tile * 32 + c_row(r, half);
        const float z = acc[r] + bc;
        z_out[(size_t)(((gy0 + tt / kFT) << lgW) + gx0 + tt % kFT) * 2 + i] = z;
        if (i == 0) zs += (double)z;
      }
    }
  }
}

// Grid: (H / 16) (W / 16) blocks of 512 threads, tile b at rows
// 16 (b / (W / 16)), columns 16 (b % (W / 16)).  part[b] = the tile's FP64 sum
// of z[.][0] (fixed order).
template <typename T>
__global__ __launch_bounds__(kFWaves * 64) void k_net_fused(
    const T* __restrict__ phi, const T* __restrict__ om, float s0, float s1,
    const uint16_t* __restrict__ w0, const uint16_t* __restrict__ w1,
    const uint16_t* __restrict__ w2, const uint16_t* __restrict__ w3,
    const float* __restrict__ params, float* __restrict__ z3, double* __restrict__ part, int H,
    int W, int lgW) {
  __shared__ __align__(16) uint16_t in0[kFR * kFR * 2];
  __shared__ __align__(16) uint16_t buf_a[pad32((kFR - 2) * (kFR - 2)) * kFS];
  __shared__ __align__(16) uint16_t buf_b[pad32((kFR - 4) * (kFR - 4)) * kFS];
  constexpr int KP0 = pad16(18), KP = pad16(288);
  __shared__ __align__(16) uint16_t wl0[32 * (KP0 + 8)];
  __shared__ __align__(16) uint16_t wl1[32 * (KP + 8)];
  __shared__ __align__(16) uint16_t wl2[32 * (KP + 8)];
  __shared__ __align__(16) uint16_t wl3[2 * (KP + 8)];
  __shared__ double wsum[2 * kFWaves];
  const int tiles_x = W / kFT;
  const int ty0 = (int)(blockIdx.x / tiles_x) * kFT, tx0 = (int)(blockIdx.x % tiles_x) * kFT;
  // every global read of the block is issued before the first is used: the
  // 16-byte chunks of the four weight matrices (rows past the last layer's
  // two outputs are not needed) and the state planes of the region
  constexpr int C0 = 32 * KP0 / 8, C1 = 32 * KP / 8, C3 = 2 * KP / 8;
  constexpr int NCH = C0 + 2 * C1 + C3, NCH_T = (NCH + kFWaves * 64 - 1) / (kFWaves * 64);
  u16x8 wv[NCH_T];
#pragma unroll
  for (int u = 0; u < NCH_T; ++u) {
    int c = (int)threadIdx.x + u * kFWaves * 64;
    const uint16_t* src = nullptr;
    if (c < C0) {
      src = w0 + c * 8;
    } else if ((c -= C0) < C1) {
      src = w1 + c * 8;
    } else if ((c -= C1) < C1) {
      src = w2 + c * 8;
    } else if ((c -= C1) < C3) {
      src = w3 + c * 8;
    }
    wv[u] = src ? *reinterpret_cast<const u16x8*>(src) : u16x8{};
  }
  constexpr int NPX = kFR * kFR, NPX_T = (NPX + kFWaves * 64 - 1) / (kFWaves * 64);
  T xv[NPX_T][2];
#pragma unroll
  for (int u = 0; u < NPX_T; ++u) {
    const int q = (int)threadIdx.x + u * kFWaves * 64;
    const int ry = q / kFR, rx = q - ry * kFR;
    const int gp = (((ty0 - kFH + ry) & (H - 1)) << lgW) | ((tx0 - kFH + rx) & (W - 1));
    xv[u][0] = q < NPX ? phi[gp] : T(0);
    xv[u][1] = q < NPX ? om[gp] : T(0);
  }
#pragma unroll
  for (int u = 0; u < NCH_T; ++u) {
    int c = (int)threadIdx.x + u * kFWaves * 64;
    uint16_t* dst = nullptr;
    if (c < C0) {
      dst = wl0 + (c / (KP0 / 8)) * (KP0 + 8) + (c % (KP0 / 8)) * 8;
    } else if ((c -= C0) < C1) {
      dst = wl1 + (c / (KP / 8)) * (KP + 8) + (c % (KP / 8)) * 8;
    } else if ((c -= C1) < C1) {
      dst = wl2 + (c / (KP / 8)) * (KP + 8) + (c % (KP / 8)) * 8;
    } else if ((c -= C1) < C3) {
      dst = wl3 + (c / (KP / 8)) * (KP + 8) + (c % (KP / 8)) * 8;
    }
    if (dst) *reinterpret_cast<u16x8*>(dst) = wv[u];
  }
#pragma unroll
  for (int u = 0; u < NPX_T; ++u) {
    const int q = (int)threadIdx.x + u * kFWaves * 64;
    if (q < NPX) {
      in0[2 * q] = f2bf((float)xv[u][0] * s0);
      in0[2 * q + 1] = f2bf((float)xv[u][1] * s1);
    }
  }
  __syncthreads();
  double zs = 0.0;
  fused_layer<2, kFR, false>(in0, buf_a, wl0, params + kOffB[0], nullptr, 0, 0, lgW, zs);
  __syncthreads();
  fused_layer<32, kFR - 2, false>(buf_a, buf_b, wl1, params + kOffB[1], nullptr, 0, 0, lgW,
                                  zs);
  __syncthreads();
  fused_layer<32, kFR - 4, false>(buf_b, buf_a, wl2, params + kOffB[2], nullptr, 0, 0, lgW,
                                  zs);
  __syncthreads();
  fused_layer<32, kFR - 6, true>(buf_a, nullptr, wl3, params + kOffB[3], z3, ty0, tx0, lgW,
                                 zs);
  const int lane = threadIdx.x & 63;
  if ((lane & 31) == 0) wsum[(threadIdx.x >> 6) * 2 + (lane >> 5)] = zs;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int k = 0; k < 2 * kFWaves; ++k) t += wsum[k];
    part[blockIdx.x] = t;
  }
}

// ---------------------------------------------------------------- input grad

// da[p][ci] = sum_{tap, co} W[co][ci][tap] dz[p + (1,1) - tap][co], then
// dzprev = da * silu'(zprev).  CIN = 32 (every layer with an input grad).
// Bound by memory: 2^20 pixels take 71 us (COUT = 32, 420 B per pixel, 6.1 TB/s)
// and 59 us (COUT = 2, 330 B); reading dz once per tap instead of once per tile
// and halo, 65536 pixels took 21 and 10 us.  Held to three wavefronts per SIMD
// the registers spill (114 us).
template <int COUT>
__global__ __launch_bounds__(256) void k_conv_dx(const float* __restrict__ dz,
                                                 const uint16_t* __restrict__ wx,
                                                 const float* __restrict__ zprev,
                                                 float* __restrict__ dzprev, int ntiles, int H,
                                                 int W, int lgW) {
  constexpr int CIN = 32, K = 9 * COUT, KP = pad16(K), NKS = KP / 16;
  constexpr int PS = COUT == 2 ? 2 : kFS;   // LDS pixel stride
  __shared__ __align__(16) uint16_t in[kHR * kHR * PS];
  const int lane = threadIdx.x & 63, half = lane >> 5, i = lane & 31;
  u16x8 bv[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    bv[ks] = *reinterpret_cast<const u16x8*>(wx + i * KP + ks * 16 + half * 8);
  for (int tile = (int)blockIdx.x; tile < ntiles; tile += (int)gridDim.x) {
    const TileAt at = tile_at(tile, H, W, lgW);
    auto pixel = [&](int q) { return halo_px(at, q, H, W, lgW); };
    if constexpr (COUT == 2) {
      f32x2_any v[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = (int)threadIdx.x + u * 256;
        if (q < kHR * kHR) v[u] = *reinterpret_cast<const f32x2_any*>(dz + pixel(q) * 2);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = (int)threadIdx.x + u * 256;
        if (q < kHR * kHR)
          *reinterpret_cast<unsigned*>(in + 2 * q) =
              (unsigned)f2bf(v[u].x) | ((unsigned)f2bf(v[u].y) << 16);
      }
    } else {
      constexpr int NI = kHR * kHR * 8, NT = (NI + 255) / 256;
      float4 v[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const int it = (int)threadIdx.x + u * 256;
        if (it < NI)
          v[u] = *reinterpret_cast<const float4*>(dz + pixel(it >> 3) * 32 + (it & 7) * 4);
      }
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const int it = (int)threadIdx.x + u * 256;
        if (it < NI) {
          const uint2 w = {(unsigned)f2bf(v[u].x) | ((unsigned)f2bf(v[u].y) << 16),
                           (unsigned)f2bf(v[u].z) | ((unsigned)f2bf(v[u].w) << 16)};
          *reinterpret_cast<uint2*>(in + (it >> 3) * PS + (it & 7) * 4) = w;
        }
      }
    }
    __syncthreads();
    for (int mt = (int)(threadIdx.x >> 6); mt < kFT * kFT / 32; mt += 4) {
      const int t = mt * 32 + i;
      auto elem = [&](int r) { return tile_px(at, mt * 32 + c_row(r, half), lgW) * CIN + i; };
      float zp[16];
      if (zprev) {
#pragma unroll
        for (int r = 0; r < 16; ++r) zp[r] = zprev[elem(r)];
      }
      f32x16 acc = {};
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
        acc = mfma(tile_operand<COUT, true>(in, t >> 4, t & 15, ks, half), bv[ks], acc);
#pragma unroll
      for (int r = 0; r < 16; ++r) dzprev[elem(r)] = zprev ? acc[r] * silu_grad(zp[r]) : acc[r];
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- weight grad

// part[block] = { dW[co][kcol], db[co] } of the block's tiles, with
// dW[co][kcol] = sum_p dz[p][co] a[p + tap - (1,1)][ci], kcol = tap CIN + ci,
// db[co] = sum_p dz[p][co].  Staging transposes both operands to
// [channel][pixel pair]: eight pixels of a row are then one 16-byte read, and
// the three taps of a tap row are the same five pairs, shifted by half a pair
// at a time.  CIN = 32: wavefront w takes tap row w; CIN = 2: one 32-column
// product covers the 18 columns, and the wavefronts take rows in turn.  The
// next tile is read into registers while one is multiplied; partials are per
// block, not per 256 pixels.  Bound by memory (CIN = COUT = 32: 200 B per pixel).
constexpr int kDwTpb = 192;
constexpr int kDwRow = 12;                       // dwords per staged row of a (9 pairs)
constexpr int kDwAs = kHR * kDwRow + 4;          // per channel of a: 28 mod 32 banks
constexpr int kDwDs = kFT * kFT / 2 + 4;         // per channel of dz: 4 mod 32 banks

template <int CIN, int COUT>
__global__ __launch_bounds__(kDwTpb) void k_conv_dw(const float* __restrict__ dz,
                                                    const uint16_t* __restrict__ a,
                                                    float* __restrict__ part, int ntiles, int H,
                                                    int W, int lgW) {
  constexpr int NK = 9 * CIN, REC = COUT * NK + COUT;
  __shared__ __align__(16) unsigned as[CIN * kDwAs];
  __shared__ __align__(16) unsigned ds[COUT * kDwDs];
  __shared__ float dbs[kDwTpb * 4];
  const int tid = (int)threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63, half = lane >> 5, i = lane & 31;

  constexpr int GA = CIN == 32 ? 4 : 1, NA = kHR * (kHR / 2) * GA, NAT = (NA + kDwTpb - 1) / kDwTpb;
  constexpr int GD = COUT == 32 ? 8 : 1, ND = kFT * kFT / 2 * GD, NDT = (ND + kDwTpb - 1) / kDwTpb;
  u16x8 ra[NAT][CIN == 32 ? 2 : 1];
  f32x4_any rd[NDT][COUT == 32 ? 2 : 1];
  auto fetch = [&](int tile) {
    const TileAt at = tile_at(tile, H, W, lgW);
#pragma unroll
    for (int u = 0; u < NAT; ++u) {
      const int it = tid + u * kDwTpb;
      if (it < NA) {
        const int pr = it / GA, row = pr / (kHR / 2), j = pr % (kHR / 2);
        const size_t line = at.base + (size_t)(((at.y0 - 1 + row) & (H - 1)) << lgW);
        const size_t q0 = line + ((at.x0 - 1 + 2 * j) & (W - 1));
        const size_t q1 = line + ((at.x0 + 2 * j) & (W - 1));
        if constexpr (CIN == 32) {
          ra[u][0] = *reinterpret_cast<const u16x8_any*>(a + q0 * 32 + (it % GA) * 8);
          ra[u][1] = *reinterpret_cast<const u16x8_any*>(a + q1 * 32 + (it % GA) * 8);
        } else {
          const unsigned v0 = *reinterpret_cast<const u32_any*>(a + q0 * 2);
          const unsigned v1 = *reinterpret_cast<const u32_any*>(a + q1 * 2);
          ra[u][0][0] = (uint16_t)v0;
          ra[u][0][1] = (uint16_t)(v0 >> 16);
          ra[u][0][2] = (uint16_t)v1;
          ra[u][0][3] = (uint16_t)(v1 >> 16);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < NDT; ++u) {
      const int it = tid + u * kDwTpb;
      if (it < ND) {
        const int pr = it / GD, row = pr / (kFT / 2), j = pr % (kFT / 2);
        const size_t q = at.base + (size_t)(((at.y0 + row) << lgW) + at.x0 + 2 * j);
        if constexpr (COUT == 32) {
          rd[u][0] = *reinterpret_cast<const f32x4_any*>(dz + q * 32 + (it % GD) * 4);
          rd[u][1] = *reinterpret_cast<const f32x4_any*>(dz + q * 32 + 32 + (it % GD) * 4);
        } else {
          rd[u][0] = *reinterpret_cast<const f32x4_any*>(dz + q * 2);
        }
      }
    }
  };
  float db[4] = {0.f, 0.f, 0.f, 0.f};   // channels 4 (tid % 8) + c, or c
  auto put = [&] {
    auto pair = [](uint16_t lo, uint16_t hi) { return (unsigned)lo | ((unsigned)hi << 16); };
#pragma unroll
    for (int u = 0; u < NAT; ++u) {
      const int it = tid + u * kDwTpb;
      if (it < NA) {
        const int pr = it / GA;
        unsigned* o = as + pr / (kHR / 2) * kDwRow + pr % (kHR / 2);
        if constexpr (CIN == 32) {
#pragma unroll
          for (int c = 0; c < 8; ++c)
            o[((it % GA) * 8 + c) * kDwAs] = pair(ra[u][0][c], ra[u][1][c]);
        } else {
          o[0] = pair(ra[u][0][0], ra[u][0][2]);
          o[kDwAs] = pair(ra[u][0][1], ra[u][0][3]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < NDT; ++u) {
      const int it = tid + u * kDwTpb;
      if (it < ND) {
        const int pr = it / GD;
        if constexpr (COUT == 32) {
          const f32x4_any x0 = rd[u][0], x1 = rd[u][1];
          unsigned* o = ds + (it % GD) * 4 * kDwDs + pr;
          o[0] = pair(f2bf(x0.x), f2bf(x1.x));
          o[kDwDs] = pair(f2bf(x0.y), f2bf(x1.y));
          o[2 * kDwDs] = pair(f2bf(x0.z), f2bf(x1.z));
          o[3 * kDwDs] = pair(f2bf(x0.w), f2bf(x1.w));
          db[0] += x0.x + x1.x;
          db[1] += x0.y + x1.y;
          db[2] += x0.z + x1.z;
          db[3] += x0.w + x1.w;
        } else {
          const f32x4_any x = rd[u][0];
          ds[pr] = pair(f2bf(x.x), f2bf(x.z));
          ds[kDwDs + pr] = pair(f2bf(x.y), f2bf(x.w));
          db[0] += x.x + x.z;
          db[1] += x.y + x.w;
        }
      }
    }
  };

  constexpr int NACC = CIN == 32 ? 3 : 1;
  f32x16 acc[NACC] = {};
  const int tap = i < NK ? i / 2 : 0, tx = tap % 3;   // CIN = 2: this lane's column
  fetch((int)blockIdx.x);
  for (int tile = (int)blockIdx.x; tile < ntiles; tile += (int)gridDim.x) {
    put();
    __syncthreads();
    if (tile + (int)gridDim.x < ntiles) fetch(tile + (int)gridDim.x);
    for (int ks = CIN == 32 ? 0 : wave; ks < kFT; ks += CIN == 32 ? 1 : 3) {
      uint4 av = {0u, 0u, 0u, 0u};
      if (i < COUT)
        av = *reinterpret_cast<const uint4*>(ds + i * kDwDs + ks * (kFT / 2) + 4 * half);
      const u16x8 A = __builtin_bit_cast(u16x8, av);
      auto shifted = [](uint4 p, unsigned p4, unsigned by) {
        const uint4 v = {
            __builtin_amdgcn_alignbit(p.y, p.x, by), __builtin_amdgcn_alignbit(p.z, p.y, by),
            __builtin_amdgcn_alignbit(p.w, p.z, by), __builtin_amdgcn_alignbit(p4, p.w, by)};
        return __builtin_bit_cast(u16x8, v);
      };
      if constexpr (CIN == 32) {
        const unsigned* b = as + i * kDwAs + (ks + wave) * kDwRow + 4 * half;
        const uint4 p = *reinterpret_cast<const uint4*>(b);
        const unsigned p4 = b[4];
        const uint4 p1 = {p.y, p.z, p.w, p4};
        acc[0] = mfma(A, __builtin_bit_cast(u16x8, p), acc[0]);
        acc[1] = mfma(A, shifted(p, p4, 16), acc[1]);
        acc[2] = mfma(A, __builtin_bit_cast(u16x8, p1), acc[2]);
      } else {
        const unsigned* b = as + (i & 1) * kDwAs + (ks + tap / 3) * kDwRow + 4 * half + (tx == 2);
        const uint4 p = {b[0], b[1], b[2], b[3]};
        const u16x8 B = shifted(p, b[4], tx == 1 ? 16u : 0u);
        acc[0] = mfma(A, i < NK ? B : u16x8{}, acc[0]);
      }
    }
    __syncthreads();
  }

  float* out = part + (size_t)blockIdx.x * REC;
  if constexpr (CIN == 32) {
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = c_row(r, half);
        if (row < COUT) out[row * NK + (wave * 3 + x) * 32 + i] = acc[x][r];
      }
  } else {
    static_assert(CIN == 32 || COUT * kDwDs >= 3 * 32 * 32, "the three wavefronts' sums");
    float* red = reinterpret_cast<float*>(ds);
#pragma unroll
    for (int r = 0; r < 16; ++r) red[(wave * 32 + c_row(r, half)) * 32 + i] = acc[0][r];
    __syncthreads();
    for (int e = tid; e < COUT * NK; e += kDwTpb) {
      const int row = e / NK, col = e % NK;
      out[e] = red[row * 32 + col] + red[(32 + row) * 32 + col] + red[(64 + row) * 32 + col];
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) dbs[tid * 4 + c] = db[c];
  __syncthreads();
  if (tid < COUT) {
    double s = 0.0;
    for (int t = COUT == 32 ? tid / 4 : 0; t < kDwTpb; t += GD) s += (double)dbs[t * 4 + tid % 4];
    out[COUT * NK + tid] = (float)s;
  }
}

struct GradParts {
  const float* part[kCnnLayers];   // nb[l] records { dW, db } of layer l
  int nb[kCnnLayers];
};

// grad[e] += the sum of the partials of parameter e, e0 <= e < e1.  64
// parameters per block, their records over 16 wavefronts (fixed order, FP64).
__global__ __launch_bounds__(1024) void k_grad_reduce(GradParts parts, float* __restrict__ grad,
                                                      int e0, int e1) {
  __shared__ double red[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int e = e0 + (int)blockIdx.x * 64 + lane;
  const int l = e >= kOffW[3] ? 3 : e >= kOffW[2] ? 2 : e >= kOffW[1] ? 1 : 0;
  const int cin = l ? 32 : 2, cout = l < 3 ? 32 : 2, nk = 9 * cin, rec = cout * (nk + 1);
  const int off = l == 3 ? kOffW[3] : l == 2 ? kOffW[2] : l == 1 ? kOffW[1] : kOffW[0];
  const float* part = l == 3   ? parts.part[3]
                      : l == 2 ? parts.part[2]
                      : l == 1 ? parts.part[1]
                               : parts.part[0];
  const int nb = l == 3 ? parts.nb[3] : l == 2 ? parts.nb[2] : l == 1 ? parts.nb[1] : parts.nb[0];
  double s = 0.0;
  if (e < e1) {
    const float* p = part + (e - off);
#pragma unroll 8
    for (int b = w; b < nb; b += 16) s += (double)p[(size_t)b * rec];
  }
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && e < e1) {
    for (int k = 1; k < 16; ++k) s += red[k][lane];
    int d = e - off;
    if (d < cout * nk) {
      const int co = d / nk, kcol = d % nk;
      d = (co * cin + kcol % cin) * 9 + kcol / cin;
    }
    grad[off + d] += (float)s;
  }
}

// ---------------------------------------------------------------- loss, I/O

// r = z4 * s_out; e = r - t; dz4 = scale * e * s_out; per-block sum of e^2.
// n pixels over samples of P = 2^lgP (t: two planes per sample).
__global__ __launch_bounds__(256) void k_loss(const float* __restrict__ z4,
                                              const float* __restrict__ t, int n, int lgP,
                                              float s2, float s3, float scale,
                                              float* __restrict__ dz4,
                                              double* __restrict__ part) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int p = blockIdx.x * 256 + threadIdx.x; p < n; p += gridDim.x * 256) {
    const float* tp = t + p + ((size_t)(p >> lgP) << lgP);
    const float2 z = *reinterpret_cast<const float2*>(z4 + 2 * (size_t)p);
    const float e0 = z.x * s2 - tp[0];
    const float e1 = z.y * s3 - tp[(size_t)1 << lgP];
    *reinterpret_cast<float2*>(dz4 + 2 * (size_t)p) = {scale * e0 * s2, scale * e1 * s3};
    acc += (double)e0 * e0 + (double)e1 * e1;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = 128; h >= 1; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// out[0] (+)= sum of part[0 .. n) as one block's fixed-order
// tree; acc = 0 overwrites (no clearing launch needed, so the call may sit
// in a captured graph).  Launch with 256 threads.
__global__ __launch_bounds__(256) void k_sum_into(const double* __restrict__ part, int n,
                                                  double* __restrict__ out, int acc) {
  __shared__ double red[256];
  double s = 0.0;
  for (int k = threadIdx.x; k < n; k += 256) s += part[k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h >= 1; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (acc ? out[0] : 0.0) + red[0];
}

// Layer 0's input of n pixels over samples of P = 2^lgP (x: two planes each).
__global__ void k_pack_input(const float* __restrict__ x, int n, int lgP, float s0, float s1,
                             uint16_t* __restrict__ a0) {
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < n; p += gridDim.x * blockDim.x) {
    const float* xp = x + p + ((size_t)(p >> lgP) << lgP);
    reinterpret_cast<unsigned*>(a0)[p] =
        (unsigned)f2bf(xp[0] * s0) | ((unsigned)f2bf(xp[(size_t)1 << lgP] * s1) << 16);
  }
}

__global__ void k_unpack_out(const float* __restrict__ z4, int P, float s2, float s3,
                             float* __restrict__ r) {
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < P; p += gridDim.x * blockDim.x) {
    r[p] = z4[2 * (size_t)p] * s2;
    r[(size_t)P + p] = z4[2 * (size_t)p + 1] * s3;
  }
}

// BF16 GEMM operands of every layer from the FP32 master weights.
__global__ void k_pack_weights(const float* __restrict__ params, uint16_t* wt0, uint16_t* wt1,
                               uint16_t* wt2, uint16_t* wt3, uint16_t* wx1, uint16_t* wx2,
                               uint16_t* wx3) {
  uint16_t* wt[4] = {wt0, wt1, wt2, wt3};
  uint16_t* wx[4] = {nullptr, wx1, wx2, wx3};
  const int l = blockIdx.y;
  const int cin = kCnnCin[l], cout = kCnnCout[l];
  const int kp = pad16(9 * cin), kpx = pad16(9 * cout);
  const float* Wl = params + kOffW[l];
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < 32 * kp; e += gridDim.x * blockDim.x) {
    const int j = e / kp, k = e % kp;
    float v = 0.f;
    if (j < cout && k < 9 * cin) v = Wl[(j * cin + k % cin) * 9 + k / cin];
    wt[l][e] = f2bf(v);
  }
  if (l == 0) return;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < 32 * kpx;
       e += gridDim.x * blockDim.x) {
    const int ci = e / kpx, k = e % kpx;
    float v = 0.f;
    if (ci < cin && k < 9 * cout) v = Wl[((k % cout) * cin + ci) * 9 + k / cout];
    wx[l][e] = f2bf(v);
  }
}

// Adam with bias correction; the gradient is cleared for the next batch.
__global__ void k_adam(float* __restrict__ p, float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
    const float gg = g[e];
    const float mm = b1 * m[e] + (1.f - b1) * gg;
    const float vv = b2 * v[e] + (1.f - b2) * gg * gg;
    m[e] = mm;
    v[e] = vv;
    p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    g[e] = 0.f;
  }
}

__global__ void k_mfma_probe(const uint16_t* __restrict__ a, const uint16_t* __restrict__ b,
                             float* __restrict__ c) {
  const int lane = threadIdx.x, half = lane >> 5, i = lane & 31;
  u16x8 av, bv;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    av[e] = a[i * 16 + 8 * half + e];
    bv[e] = b[(8 * half + e) * 32 + i];
  }
  f32x16 acc = {};
  acc = mfma(av, bv, acc);
#pragma unroll
  for (int r = 0; r < 16; ++r) c[c_row(r, half) * 32 + i] = acc[r];
}

#define CNN_TRY(x)                          \
  do {                                      \
    if ((x) != hipSuccess) return -3;       \
  } while (0)

int alloc_dev(void** p, size_t bytes) { return hipMalloc(p, bytes) == hipSuccess ? 0 : -2; }

// The pixel kernels' grid over n pixels (four blocks per CU at most).
int px_blocks(int n) { return n / 256 < 1024 ? n / 256 : 1024; }

// Tiles of `samples` samples.
int tiles_of(const Net* n, int samples) { return samples * (n->P / (kFT * kFT)); }

void launch_fwd(const Net* n, int li, int samples, const uint16_t* a_in, float* z,
                uint16_t* a_out, hipStream_t st) {
  const int nt = tiles_of(n, samples);
  const int cap = li ? kFwdBlocks : kConvBlocks;
  const dim3 g(nt < cap ? nt : cap), b(256);
  const float* bias = n->params + kOffB[li];
  if (li == 0)
    hipLaunchKernelGGL((k_conv_fwd<2, 32, true>), g, b, 0, st, a_in, n->wt[0], bias, z, a_out, nt,
                       n->H, n->W, n->lgW);
  else if (li < 3)
    hipLaunchKernelGGL((k_conv_fwd<32, 32, true>), g, b, 0, st, a_in, n->wt[li], bias, z, a_out,
                       nt, n->H, n->W, n->lgW);
  else
    hipLaunchKernelGGL((k_conv_fwd<32, 2, false>), g, b, 0, st, a_in, n->wt[3], bias, z, a_out,
                       nt, n->H, n->W, n->lgW);
}

// The weight gradient's partials over at most `tiles` tiles: layer l's
// dw_blocks(l, tiles) records at part + dw_part(l, tiles), layers 1 and 2 in turn
// in one place (layer 2's are added up before layer 1's are written).
int dw_blocks(int li, int ntiles) { return ntiles < kDwBlocks[li] ? ntiles : kDwBlocks[li]; }
int dw_rec(int li) { return kOffB[li] + kCnnCout[li] - kOffW[li]; }
size_t dw_part(int li, int tiles) {
  auto len = [&](int l) { return (size_t)dw_blocks(l, tiles) * dw_rec(l); };
  return li == 0 ? 0 : li == 3 ? len(0) : len(0) + len(3);
}
size_t dw_floats(int tiles) { return dw_part(1, tiles) + (size_t)dw_blocks(1, tiles) * dw_rec(1); }
static_assert(kDwBlocks[1] == kDwBlocks[2], "layers 1 and 2 share their place");

// Weight and bias gradient partials of layer li over `samples` samples; the
// input gradient (times silu' of zprev, when given) into dzprev for li > 0.
void launch_bwd(const Net* n, int li, int samples, const float* dz, const uint16_t* a_in,
                const float* zprev, float* dzprev, hipStream_t st) {
  const int nt = tiles_of(n, samples), nb = dw_blocks(li, nt);
  const dim3 b(kDwTpb), g(nb);
  float* part = n->work.part + dw_part(li, tiles_of(n, n->work.samples));
  if (li == 0)
    hipLaunchKernelGGL((k_conv_dw<2, 32>), g, b, 0, st, dz, a_in, part, nt, n->H, n->W, n->lgW);
  else if (li < 3)
    hipLaunchKernelGGL((k_conv_dw<32, 32>), g, b, 0, st, dz, a_in, part, nt, n->H, n->W, n->lgW);
  else
    hipLaunchKernelGGL((k_conv_dw<32, 2>), g, b, 0, st, dz, a_in, part, nt, n->H, n->W, n->lgW);
  if (li > 0 && dzprev) {
    const dim3 gx(nt < kConvBlocks ? nt : kConvBlocks);
    if (li < 3)
      hipLaunchKernelGGL((k_conv_dx<32>), gx, dim3(256), 0, st, dz, n->wx[li], zprev, dzprev, nt,
                         n->H, n->W, n->lgW);
    else
      hipLaunchKernelGGL((k_conv_dx<2>), gx, dim3(256), 0, st, dz, n->wx[li], zprev, dzprev, nt,
                         n->H, n->W, n->lgW);
  }
}

// The gradient of layers l0 .. l1 += the partials of launch_bwd.
void launch_reduce(const Net* n, int samples, int l0, int l1, hipStream_t st) {
  GradParts p;
  for (int l = 0; l < kCnnLayers; ++l) {
    p.part[l] = n->work.part + dw_part(l, tiles_of(n, n->work.samples));
    p.nb[l] = dw_blocks(l, tiles_of(n, samples));
  }
  const int e0 = kOffW[l0], e1 = kOffB[l1] + kCnnCout[l1];
  hipLaunchKernelGGL(k_grad_reduce, dim3((e1 - e0 + 63) / 64), dim3(1024), 0, st, p, n->grad, e0,
                     e1);
}

void launch_pack_weights(Net* n, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_weights, dim3(16, 4), dim3(256), 0, st, n->params, n->wt[0],
                     n->wt[1], n->wt[2], n->wt[3], n->wx[1], n->wx[2], n->wx[3]);
}

}  // namespace

// The calling thread's current device is `dev` while this lives.
struct OnDevice {
  int was = -1;
  explicit OnDevice(int dev) {
    if (hipGetDevice(&was) != hipSuccess || was == dev || hipSetDevice(dev) != hipSuccess) was = -1;
  }
  ~OnDevice() {
    if (was >= 0) (void)hipSetDevice(was);
  }
};

// Buffers of `samples` samples at once for the training step.
int train_alloc(TrainWork* w, const Net* n, int samples) {
  const size_t px = (size_t)n->P * samples;
  int rc = 0;
  for (int l = 0; l < kCnnLayers; ++l)
    rc = rc ? rc : alloc_dev((void**)&w->act[l], px * kCnnCin[l] * 2);
  for (int l = 0; l < kCnnLayers; ++l)
    rc = rc ? rc : alloc_dev((void**)&w->z[l], px * kCnnCout[l] * sizeof(float));
  for (int k = 0; k < 2; ++k) rc = rc ? rc : alloc_dev((void**)&w->dz[k], px * 32 * sizeof(float));
  rc = rc ? rc : alloc_dev((void**)&w->part, dw_floats(tiles_of(n, samples)) * sizeof(float));
  if (!rc) w->samples = samples;
  return rc;
}

void train_free(TrainWork* w) {
  void* ps[] = {w->act[0], w->act[1], w->act[2], w->act[3], w->z[0], w->z[1],
                w->z[2],   w->z[3],   w->dz[0],  w->dz[1],  w->part};
  for (void* p : ps)
    if (p) (void)hipFree(p);
  *w = TrainWork();
}

// Room for B samples at once, at most kGroupPixels pixels, on the network's
// device; with less memory than that, for as many as fit beside what is there,
// which stays where none do.
int train_reserve(Net* n, int B) {
  TrainWork* w = &n->work;
  int want = kGroupPixels / n->P;
  want = want < 1 ? 1 : want > B ? B : want;
  if (w->asked >= want) return 0;
  const OnDevice on(n->dev);
  for (int k = want; k > w->samples; k /= 2) {
    TrainWork more;
    if (!train_alloc(&more, n, k)) {
      train_free(w);
      *w = more;
      break;
    }
    train_free(&more);
    (void)hipGetLastError();
  }
  if (!w->samples) return -2;
  w->asked = want;
  return 0;
}

int net_create(Net* n, int H, int W, bool training) {
  if (H < 16 || W < 16 || (H & (H - 1)) || (W & (W - 1))) return -1;
  if (hipGetDevice(&n->dev) != hipSuccess) return -3;
  n->H = H;
  n->W = W;
  n->lgW = 0;
  while ((1 << n->lgW) < W) ++n->lgW;
  n->P = H * W;
  n->lgP = n->lgW;
  while ((1 << n->lgP) < n->P) ++n->lgP;
  const size_t P = (size_t)n->P;
  int rc = 0;
  rc = rc ? rc : alloc_dev((void**)&n->params, kCnnParams * sizeof(float));
  for (int l = 0; l < kCnnLayers; ++l) {
    rc = rc ? rc : alloc_dev((void**)&n->wt[l], 32 * (size_t)pad16(9 * kCnnCin[l]) * 2);
    if (l > 0) rc = rc ? rc : alloc_dev((void**)&n->wx[l], 32 * (size_t)pad16(9 * kCnnCout[l]) * 2);
    if (training) continue;
    rc = rc ? rc : alloc_dev((void**)&n->act[l], P * kCnnCin[l] * 2);
    rc = rc ? rc : alloc_dev((void**)&n->z[l], P * kCnnCout[l] * sizeof(float));
  }
  // the corrected step's per-tile partials; the loss and its partials
  const size_t nred = P / (kFT * kFT) > 1025 ? P / (kFT * kFT) : 1025;
  rc = rc ? rc : alloc_dev((void**)&n->red, nred * sizeof(double));
  if (training) {
    rc = rc ? rc : alloc_dev((void**)&n->grad, kCnnParams * sizeof(float));
    rc = rc ? rc : alloc_dev((void**)&n->m, kCnnParams * sizeof(float));
    rc = rc ? rc : alloc_dev((void**)&n->v, kCnnParams * sizeof(float));
    rc = rc ? rc : train_reserve(n, 1);
    if (!rc && (hipMemset(n->grad, 0, kCnnParams * 4) || hipMemset(n->m, 0, kCnnParams * 4) ||
                hipMemset(n->v, 0, kCnnParams * 4)))
      rc = -3;
  }
  if (rc) net_destroy(n);
  return rc;
}

void net_destroy(Net* n) {
  void* ps[] = {n->params, n->grad, n->m, n->v, n->red};
  for (void* p : ps)
    if (p) (void)hipFree(p);
  train_free(&n->work);
  for (int l = 0; l < kCnnLayers; ++l) {
    if (n->wt[l]) (void)hipFree(n->wt[l]);
    if (n->wx[l]) (void)hipFree(n->wx[l]);
    if (n->act[l]) (void)hipFree(n->act[l]);
    if (n->z[l]) (void)hipFree(n->z[l]);
  }
  *n = Net();
}

int net_set_params(Net* n, const float* host, hipStream_t st) {
  CNN_TRY(hipMemcpyAsync(n->params, host, kCnnParams * sizeof(float), hipMemcpyHostToDevice, st));
  launch_pack_weights(n, st);
  CNN_TRY(hipGetLastError());
  n->adam_t = 0;
  return 0;
}

int net_forward_planes(Net* n, const float* x, float* r, hipStream_t st) {
  const int P = n->P;
  const bool training = n->grad != nullptr;
  uint16_t* const* act = training ? n->work.act : n->act;
  float* const* z = training ? n->work.z : n->z;
  hipLaunchKernelGGL(k_pack_input, dim3(px_blocks(P)), dim3(256), 0, st, x, P, n->lgP,
                     n->scales[0], n->scales[1], act[0]);
  for (int l = 0; l < kCnnLayers; ++l)
    launch_fwd(n, l, 1, act[l], z[l], l < 3 ? act[l + 1] : nullptr, st);
  hipLaunchKernelGGL(k_unpack_out, dim3(256), dim3(256), 0, st, z[3], P, n->scales[2],
                     n->scales[3], r);
  CNN_TRY(hipGetLastError());
  return 0;
}

int net_grad(Net* n, const float* xs, const float* ts, int B, double* loss, hipStream_t st) {
  if (!n->grad || B < 1) return -1;
  if (const int rc = train_reserve(n, B)) return rc;
  const int P = n->P;
  const float scale = 2.0f / ((float)B * 2.0f * (float)P);
  const TrainWork& w = n->work;
  for (int s = 0; s < B; s += w.samples) {
    const int ns = B - s < w.samples ? B - s : w.samples, px = ns * P, nbl = px_blocks(px);
    hipLaunchKernelGGL(k_pack_input, dim3(nbl), dim3(256), 0, st, xs + (size_t)s * 2 * P, px,
                       n->lgP, n->scales[0], n->scales[1], w.act[0]);
    for (int l = 0; l < kCnnLayers; ++l)
      launch_fwd(n, l, ns, w.act[l], w.z[l], l < 3 ? w.act[l + 1] : nullptr, st);
    hipLaunchKernelGGL(k_loss, dim3(nbl), dim3(256), 0, st, w.z[3], ts + (size_t)s * 2 * P, px,
                       n->lgP, n->scales[2], n->scales[3], scale, w.dz[0], n->red + 1);
    hipLaunchKernelGGL(k_sum_into, dim3(1), dim3(256), 0, st, n->red + 1, nbl, n->red, s > 0);
    int cur = 0;
    for (int l = kCnnLayers - 1; l >= 0; --l) {
      launch_bwd(n, l, ns, w.dz[cur], w.act[l], l > 0 ? w.z[l - 1] : nullptr,
                 l > 0 ? w.dz[cur ^ 1] : nullptr, st);
      if (l == 2) launch_reduce(n, ns, 2, 3, st);
      cur ^= 1;
    }
    launch_reduce(n, ns, 0, 1, st);
  }
  CNN_TRY(hipGetLastError());
  double h = 0.0;
  CNN_TRY(hipMemcpyAsync(&h, n->red, sizeof(double), hipMemcpyDeviceToHost, st));
  CNN_TRY(hipStreamSynchronize(st));
  if (loss) *loss = h / ((double)B * 2.0 * P);
  return 0;
}

int net_adam(Net* n, float lr, float b1, float b2, float eps, hipStream_t st) {
  if (!n->grad) return -1;
  n->adam_t += 1;
  const float c1 = 1.f - powf(b1, (float)n->adam_t);
  const float c2 = 1.f - powf(b2, (float)n->adam_t);
  hipLaunchKernelGGL(k_adam, dim3(80), dim3(256), 0, st, n->params, n->grad, n->m, n->v,
                     kCnnParams, lr, b1, b2, eps, c1, c2);
  launch_pack_weights(n, st);
  CNN_TRY(hipGetLastError());
  return 0;
}

int net_layer_fwd(Net* n, int li, const uint16_t* a_in, float* z_out, uint16_t* a_out,
                  hipStream_t st) {
  if (li < 0 || li >= kCnnLayers) return -1;
  launch_fwd(n, li, 1, a_in, z_out, li < 3 ? a_out : nullptr, st);
  CNN_TRY(hipGetLastError());
  return 0;
}

int net_layer_bwd(Net* n, int li, const float* dz, const uint16_t* a_in, const float* zprev,
                  float* dzprev, float* dw, hipStream_t st) {
  if (li < 0 || li >= kCnnLayers || !n->grad) return -1;
  CNN_TRY(hipMemsetAsync(n->grad, 0, kCnnParams * sizeof(float), st));
  launch_bwd(n, li, 1, dz, a_in, zprev, dzprev, st);
  launch_reduce(n, 1, li, li, st);
  CNN_TRY(hipGetLastError());
  if (dw) {
    const int len = kOffB[li] + kCnnCout[li] - kOffW[li];
    CNN_TRY(hipMemcpyAsync(dw, n->grad + kOffW[li], len * sizeof(float), hipMemcpyDeviceToDevice,
                           st));
  }
  return 0;
}

int net_tiles(const Net* n) { return (n->H / kFT) * (n->W / kFT); }

template <typename T>
int net_residual(Net* n, const T* phi, const T* omega, hipStream_t st) {
  hipLaunchKernelGGL((k_net_fused<T>), dim3(net_tiles(n)), dim3(kFWaves * 64), 0, st, phi, omega,
                     n->scales[0], n->scales[1], n->wt[0], n->wt[1], n->wt[2], n->wt[3],
                     n->params, n->z[3], n->red, n->H, n->W, n->lgW);
  CNN_TRY(hipGetLastError());
  return 0;
}
template int net_residual<double>(Net*, const double*, const double*, hipStream_t);
template int net_residual<float>(Net*, const float*, const float*, hipStream_t);

int mfma_probe(const uint16_t* a, const uint16_t* b, float* c, hipStream_t st) {
  uint16_t *da = nullptr, *db = nullptr;
  float* dc = nullptr;
  int rc = 0;
  rc = rc ? rc : alloc_dev((void**)&da, 32 * 16 * 2);
  rc = rc ? rc : alloc_dev((void**)&db, 16 * 32 * 2);
  rc = rc ? rc : alloc_dev((void**)&dc, 32 * 32 * 4);
  if (!rc && (hipMemcpyAsync(da, a, 32 * 16 * 2, hipMemcpyHostToDevice, st) ||
              hipMemcpyAsync(db, b, 16 * 32 * 2, hipMemcpyHostToDevice, st)))
    rc = -3;
  if (!rc) {
    hipLaunchKernelGGL(k_mfma_probe, dim3(1), dim3(64), 0, st, da, db, dc);
    if (hipGetLastError() || hipMemcpyAsync(c, dc, 32 * 32 * 4, hipMemcpyDeviceToHost, st) ||
        hipStreamSynchronize(st))
      rc = -3;
  }
  if (da) (void)hipFree(da);
  if (db) (void)hipFree(db);
  if (dc) (void)hipFree(dc);
  return rc;
}

}  // namespace le
