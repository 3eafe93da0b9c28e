// Learned cardinality estimator beside the HyperLogLog estimate of Alg. 5:
// a 67 -> 64 -> 64 -> 1 GELU MLP over a host's register histogram, the pool's
// register histogram and ln(g/m), predicting ln(1 + n).
//   - inference: bf16 weights and inputs on the matrix cores
//     (v_mfma_f32_16x16x32_bf16, fp32 accumulation), 16 hosts per wave, with
//     the plain estimate as fallback outside the training envelope;
//   - training: fp32 backpropagation on the fp32 matrix cores, gradients
//     added with atomics, then an Adam update.
// Parameter vector (fp32, 8577): W1 (64 x 67), b1, W2 (64 x 64), b2, w3, b3.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstring>
#include <new>
#include <vector>

#include "vbdr_internal.h"

using namespace vbdr;

namespace {

constexpr int kIn = 67, kHid = 64, kInPad = 96;
constexpr int kOffW1 = 0, kOffB1 = kHid * kIn, kOffW2 = kOffB1 + kHid, kOffB2 = kOffW2 + kHid * kHid;
constexpr int kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kHid, kParams = kOffB3 + 1;
static_assert(kParams == 8577, "parameter layout");

typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct MlpDev {
  uint16_t w1[kHid * kInPad];  // bf16, K zero-padded to 96
  uint16_t w2p[kHid * kHid];   // bf16, W2 with its columns in layer 2's K order (l2_unit)
  float b1[kHid], b2[kHid], w3[kHid], b3;  // w3 holds bf16-rounded values
  float env_lo[kIn], env_hi[kIn];
  int has_env;
  float plain_above;  // hosts whose plain estimate is at least this keep it (+inf: none)
};

// float -> bf16 bits, round to nearest even (host and device).
__host__ __device__ inline uint16_t f2bf(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x7FFFFFu)) return 0x7FC0;  // NaN
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__host__ __device__ inline float bf2f(uint16_t b) {
  uint32_t u = (uint32_t)b << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

// GELU of the inference kernel: erf by Abramowitz & Stegun 7.1.26 (absolute
// error <= 1.5e-7, below one fp32 ulp of the GELU's 1 + erf term), without
// the branches of erff, so that a lane's 16 activations need few registers.
__device__ __forceinline__ float gelu_inf(float x) {
  const float z = fabsf(x) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * z);
  const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  const float e = 1.0f - poly * __expf(-z * z);  // erf(|x| / sqrt 2)
  return 0.5f * x * (1.0f + (x < 0.0f ? -e : e));
}

// ------------------------------------------------------------ features
// fp32 features of nh hosts from the histogram pass: [h][67], a thread per value.
__global__ __launch_bounds__(256) void k_features(uint32_t nh, uint32_t parts, uint32_t hstride,
                                                  const uint32_t* __restrict__ hws,
                                                  const unsigned long long* __restrict__ hist, uint32_t g, uint32_t m,
                                                  float* __restrict__ feats) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (uint64_t)nh * kIn) return;
  const uint32_t h = (uint32_t)(i / kIn), c = (uint32_t)(i - (uint64_t)h * kIn);
  if (c < kBins) {
    uint32_t n = 0;
    for (uint32_t x = 0; x < parts; ++x) n += hws[((uint64_t)x * hstride + h) * kBins + c];
    feats[i] = (float)((double)n / (double)g);
  } else if (c < 2 * kBins) {
    feats[i] = (float)((double)hist[c - kBins] / (double)m);
  } else {
    feats[i] = (float)log((double)g / (double)m);
  }
}

// ----------------------------------------------------------- inference
// A wave estimates a tile of 16 hosts.  Both layers run transposed on the
// matrix cores, hidden units as rows and hosts as columns, so that the
// accumulator of layer 1 (lane l: units 16 nt + 4 (l/16) + i of host l%16) is
// already the B operand of layer 2 once the K order of layer 2 is permuted to
// match (W2's columns are stored permuted, w2p).  Layer 2's outputs meet w3 in
// the same lanes; three lane exchanges give the tile's 16 sums.  The plain
// estimate is computed (in parallel over the tile's hosts) only for hosts that
// fall back.
constexpr int kInfBlock = 256;
constexpr int kInfWaves = kInfBlock / 64;
constexpr int kHistStride = 36;  // words per histogram row (16-byte aligned rows)

// Unit of layer 1 held in K slot (ks, q, i) of layer 2's operands.
__host__ __device__ inline int l2_unit(int ks, int q, int i) { return 16 * (2 * ks + (i >> 2)) + 4 * q + (i & 3); }

// bf16x8 of eight fp32 values.
__device__ __forceinline__ bf16x8 pack8(const float* v) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (short)f2bf(v[i]);
  return r;
}

// DIRECT: each wave gathers its 16 hosts' registers itself (pools whose
// registers are cache resident) into an LDS histogram per host; otherwise
// the histograms come from a histogram pass (hws, summed over parts).
// SPREAD, for few hosts: a workgroup of 16 waves gathers one tile, a wave a host,
// and its first wave goes on; four rounds of four hosts by one wave left the
// chip idle behind a chain of gathers (64 hosts, host path included: g = 64
// 13.8 -> 10.9 us, g = 1024 42.8 -> 15.4, g = 2048 70.3 -> 22.8; 8192 hosts and
// g = 1024: 50.4 -> 46.3, but g = 256: 21.7 -> 22.2).  At most 128 registers a
// thread: 96 (five waves a SIMD) spilled, 50000 hosts and g = 64 26.4 -> 22.3 us.
constexpr int kSpreadBlock = 16 * 64;
constexpr uint32_t kSpreadWideG = 1024;  // from which two workgroups a CU still pay
template <bool DIRECT, bool SPREAD = false>
__global__ __launch_bounds__(SPREAD ? kSpreadBlock : kInfBlock) __attribute__((amdgpu_waves_per_eu(4)))
void k_learned(uint32_t nh, uint32_t parts, uint32_t hstride, const uint32_t* __restrict__ hws,
               const uint32_t* __restrict__ hosts, const uint32_t* __restrict__ s1g, const uint8_t* __restrict__ reg,
               const uint8_t* __restrict__ reg4, const unsigned long long* __restrict__ hist, uint32_t g, uint32_t m,
               const MlpDev* __restrict__ mlp, float* __restrict__ out, uint8_t* __restrict__ used_fallback) {
  constexpr int kBlock = SPREAD ? kSpreadBlock : kInfBlock, kTiles = SPREAD ? 1 : kInfWaves;
  extern __shared__ uint32_t s1_lds[];
  __shared__ __attribute__((aligned(16))) uint16_t sw1[kHid * kInPad];
  __shared__ __attribute__((aligned(16))) uint16_t sw2[kHid * kHid];
  __shared__ __attribute__((aligned(16))) uint32_t lh[kTiles][16 * kHistStride];
  __shared__ __attribute__((aligned(16))) uint16_t sconst[kInPad];  // bf16 features 33..95 (pool, ln(g/m), 0)
  __shared__ float sb1[kHid], sb2[kHid], sw3[kHid], senv_lo[kBins], senv_hi[kBins];
  __shared__ int spool_bad;
  __shared__ double sem;
  for (int i = threadIdx.x; i < kHid * kInPad / 8; i += kBlock)
    reinterpret_cast<uint4*>(sw1)[i] = reinterpret_cast<const uint4*>(mlp->w1)[i];
  for (int i = threadIdx.x; i < kHid * kHid / 8; i += kBlock)
    reinterpret_cast<uint4*>(sw2)[i] = reinterpret_cast<const uint4*>(mlp->w2p)[i];
  for (int i = threadIdx.x; i < kTiles * 16 * kHistStride; i += kBlock) (&lh[0][0])[i] = 0;
  if (threadIdx.x < kHid) {
    sb1[threadIdx.x] = mlp->b1[threadIdx.x];
    sb2[threadIdx.x] = mlp->b2[threadIdx.x];
    sw3[threadIdx.x] = mlp->w3[threadIdx.x];
  }
  if (threadIdx.x < kBins) {
    senv_lo[threadIdx.x] = mlp->has_env ? mlp->env_lo[threadIdx.x] : -INFINITY;
    senv_hi[threadIdx.x] = mlp->has_env ? mlp->env_hi[threadIdx.x] : INFINITY;
  }
  if (threadIdx.x == 0) {
    sem = stat_em(hist);
    spool_bad = 0;
  }
  if constexpr (DIRECT)
    for (uint32_t i = threadIdx.x; i < g; i += kBlock) s1_lds[i] = s1g[i];
  __syncthreads();
  if (threadIdx.x < kInPad) {
    const int c = threadIdx.x;
    float v = 0.0f;
    if (c >= kBins && c < 2 * kBins) v = (float)((double)hist[c - kBins] / (double)m);
    if (c == 2 * kBins) v = (float)log((double)g / (double)m);
    sconst[c] = f2bf(v);
    if (c >= kBins && c < kIn && mlp->has_env && !(v >= mlp->env_lo[c] && v <= mlp->env_hi[c])) atomicOr(&spool_bad, 1);
  }
  __syncthreads();
  const double Em = sem;
  const int pool_bad = spool_bad;
  const bool bytes = DIRECT && gather_bytes<kWideHist>(hist, m);
  const float inv_g = 1.0f / (float)g;  // g is a power of two: c * inv_g == c / g exactly
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, q = lane >> 4;
  uint32_t* H = lh[SPREAD ? 0 : wave];
  const uint32_t ntiles = (nh + 15) / 16;
  for (uint32_t tile = blockIdx.x * kTiles + (SPREAD ? 0 : wave); tile < ntiles; tile += gridDim.x * kTiles) {
    // An offset opaque to the compiler: the weights, biases and envelope are
    // read from LDS per tile instead of being pinned in ~150 registers across
    // the loop, which would cut the waves available to hide gather latency.
    uint32_t woff = 0;
    asm volatile("" : "+v"(woff));
    // 1. register histograms of the tile's hosts
    if constexpr (DIRECT) {
      const uint32_t last = nh - 1;  // rows past it repeat its host and are not used
      if constexpr (SPREAD) {
        const uint32_t h = tile * 16 + wave;
        hist_hosts<64, false>(mm3_key(hosts[h < last ? h : last]), s1_lds, g, m, reg, reg4, 0u, 0u, bytes,
                              H + wave * kHistStride);
        __syncthreads();
        if (wave != 0) continue;  // one tile a workgroup
      } else if (g <= 2048) {
        for (int r0 = 0; r0 < 16; r0 += 4) {
          const uint32_t h = tile * 16 + r0 + q;
          hist_hosts<16, false>(mm3_key(hosts[h < last ? h : last]), s1_lds, g, m, reg, reg4, 0u, 0u, bytes,
                                H + (r0 + q) * kHistStride);
        }
      } else {
        for (int row = 0; row < 16; ++row) {
          const uint32_t h = tile * 16 + row;
          hist_hosts<64, false>(mm3_key(hosts[h < last ? h : last]), s1_lds, g, m, reg, reg4, 0u, 0u, bytes,
                                H + row * kHistStride);
        }
      }
    } else {
      for (int e = lane; e < 16 * kBins; e += 64) {
        const int row = e / kBins, r = e - row * kBins;
        const uint32_t h = tile * 16 + row;
        uint32_t v[8], c = 0;  // all loads before their sum (8 ranges, 20 hosts: 28.7 us one after the other, 24)
#pragma unroll
        for (uint32_t x = 0; x < 8; ++x) v[x] = h < nh && x < parts ? hws[((uint64_t)x * hstride + h) * kBins + r] : 0u;
#pragma unroll
        for (uint32_t x = 0; x < 8; ++x) c += v[x];
        H[row * kHistStride + r] = c;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // 2. features of host `col`: this lane's bins 8q..8q+7 (and bin 32 for q = 0)
    uint32_t c8[8];
    {
      const uint4 lo = *reinterpret_cast<const uint4*>(H + col * kHistStride + 8 * q);
      const uint4 hi = *reinterpret_cast<const uint4*>(H + col * kHistStride + 8 * q + 4);
      c8[0] = lo.x, c8[1] = lo.y, c8[2] = lo.z, c8[3] = lo.w, c8[4] = hi.x, c8[5] = hi.y, c8[6] = hi.z, c8[7] = hi.w;
    }
    const uint32_t c32 = q == 0 ? H[col * kHistStride + 32] : 0u;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 8; ++i) H[col * kHistStride + 8 * q + i] = 0;  // clean for the next tile
    if (q == 0) H[col * kHistStride + 32] = 0;
    float f[8];
    int bad = 0;
    uint64_t U = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = 8 * q + i;
      f[i] = (float)c8[i] * inv_g;
      bad |= !(f[i] >= senv_lo[woff + r] && f[i] <= senv_hi[woff + r]);
      U += (uint64_t)c8[i] << (32 - r);
    }
    const float f32 = (float)c32 * inv_g;
    if (q == 0) {
      bad |= !(f32 >= senv_lo[woff + 32] && f32 <= senv_hi[woff + 32]);
      U += (uint64_t)c32;
    }
    const bf16x8 x0 = pack8(f);
    bf16x8 x1 = *reinterpret_cast<const bf16x8*>(sconst + woff + 32 + 8 * q);
    if (q == 0) x1[0] = (short)f2bf(f32);
    const bf16x8 x2 = *reinterpret_cast<const bf16x8*>(sconst + woff + 64 + 8 * q);
    // 3. layer 1, transposed: Z1^T (64 x 16) = W1 (64 x 96) X^T
    f32x4 z1[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const uint16_t* wr = sw1 + woff + (nt * 16 + col) * kInPad + 8 * q;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(wr), x0, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(wr + 32), x1, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(wr + 64), x2, acc, 0, 0, 0);
      z1[nt] = acc;
    }
    // 4. H1 = bf16(gelu(Z1 + b1)) in place as layer 2's B operand
    bf16x8 hb[2];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int i = 0; i < 4; ++i) hb[nt >> 1][4 * (nt & 1) + i] = (short)f2bf(gelu_inf(z1[nt][i] + sb1[woff + 16 * nt + 4 * q + i]));
    // 5. layer 2, transposed, and the output unit
    float part = 0.f;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const uint16_t* wr = sw2 + woff + (nt * 16 + col) * kHid + 8 * q;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(wr), hb[0], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(wr + 32), hb[1], acc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int u = woff + 16 * nt + 4 * q + i;
        part += gelu_inf(acc[i] + sb2[u]) * sw3[u];
      }
    }
    part += __shfl_xor(part, 16);
    part += __shfl_xor(part, 32);
    U += __shfl_xor(U, 16);
    U += __shfl_xor(U, 32);
    bad |= __shfl_xor(bad, 16);
    bad |= __shfl_xor(bad, 32);
    // 6. outputs of the tile, lane col of the first row group
    const uint32_t h = tile * 16 + col;
    if (q == 0 && h < nh) {
      float est = expf(part + mlp->b3) - 1.0f;
      int fb = bad | pool_bad;
      if (!isfinite(est)) fb = 1;
      const float above = mlp->plain_above;
      if (fb || above < INFINITY) {
        const double Es = hll_estimate(U, c8[0], (double)g);
        const double n = noise_removed(Es, Em, (double)m, (double)g);
        const float plain = (float)(n > 0.0 ? n : 0.0);
        if (!fb && plain >= above) fb = 2;  // a large count: the plain estimate is kept
        if (fb) est = plain;
      }
      out[h] = est > 0.0f ? est : 0.0f;
      if (used_fallback) used_fallback[h] = (uint8_t)fb;
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------ training
// A group of four waves takes a tile of 16 samples; wave w of it owns hidden
// units 16w..16w+15 of both layers.  All five products run on the fp32
// matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands and accumulation), units
// as rows and samples as columns, so that the activations of layer 1, their
// derivatives and dL/dh1 meet in the same lanes; the waves exchange h1 and
// dL/dz2 through LDS, sample-major.  W1 and the wave's share of the gradient stay in registers over all
// tiles of the group; a workgroup's four groups add their gradients pairwise through LDS,
// then once to memory (8577 atomics).  A chain of small dependent products
// bounds a tile (about 4 us), the atomics the rest: 4096 samples 246 us ->
// 29 us (one wave per 32 samples with serial fp32 dot products before).
// Few workgroups, each adding much: every fp32 atomic rounds, and the
// gradient's relative error against 64 bits is 2.4e-7 with 256 workgroups of
// one group, 1.1e-7 with 64 of four (1.6e-7 before).
constexpr int kTrainGroup = 256;              // threads of a tile's group
constexpr int kTrainGroups = 4;               // groups per workgroup
constexpr int kTrainBlock = kTrainGroup * kTrainGroups;
constexpr int kTrainTile = 16;                // samples per tile
constexpr int kTrainGrid = 128;               // workgroups at most
constexpr int kK1 = (kIn + 3) / 4;            // K steps of layer 1 (inputs 67 padded to 68)
constexpr int kC1 = (kIn + 15) / 16;          // column tiles of dW1
// LDS row stride of all matrices, 17 mod 64: lanes (col, q) reading [col][4t + q] hit 64 banks, [4t + q][col] nearly so
constexpr int kTStride = 16 * kC1 + 1;
static_assert(kTrainGroup / 64 * 16 == kHid, "one 16-unit row tile per wave");
constexpr int kTrainLds = 4 * kTrainTile * kTStride + kTrainGroup / 64 * kTrainTile;  // floats of a group
static_assert(kTrainGroups * kTrainLds >= 2 * kParams, "two groups' gradients fit the tiles' LDS");

// GELU and its derivative.
__device__ __forceinline__ void gelu_both(float x, float& y, float& dy) {
  const float c = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
  y = x * c;
  dy = c + x * expf(-0.5f * x * x) * 0.39894228040143268f;
}

__global__ __launch_bounds__(kTrainBlock) void k_train_grad(const float* __restrict__ params,
                                                            const float* __restrict__ feats,
                                                            const float* __restrict__ targets, uint32_t B,
                                                            float* __restrict__ grads, float* __restrict__ loss) {
  extern __shared__ float train_lds[];
  const int grp = threadIdx.x / kTrainGroup, tg = threadIdx.x % kTrainGroup, wave = tg >> 6, lane = tg & 63;
  float* xs = train_lds + grp * kTrainLds;
  float* h1s = xs + kTrainTile * kTStride;
  float* dz2s = h1s + kTrainTile * kTStride;
  float* dz1s = dz2s + kTrainTile * kTStride;
  float* ys = dz1s + kTrainTile * kTStride;
  const int col = lane & 15, q = lane >> 4;  // operands: row or column col, K index 4t + q; results: row 4q + i, column col
  const int row0 = 16 * wave;
  // weights: W1 as A operand of z1 = W1 x in registers; W2, read by rows for z2 = W2 h1 and by columns for
  // dh1 = W2^T dz2, in LDS (in registers too it would spill)
  float* w2s = train_lds + kTrainGroups * kTrainLds;
  for (int i = threadIdx.x; i < kHid * kHid; i += kTrainBlock) w2s[(i / kHid) * kTStride + i % kHid] = params[kOffW2 + i];
  float w1a[kK1], b1[4], b2[4], w3[4];
#pragma unroll
  for (int t = 0; t < kK1; ++t)
    w1a[t] = 4 * t + q < kIn ? params[kOffW1 + (row0 + col) * kIn + 4 * t + q] : 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    b1[i] = params[kOffB1 + row0 + 4 * q + i];
    b2[i] = params[kOffB2 + row0 + 4 * q + i];
    w3[i] = params[kOffW3 + row0 + 4 * q + i];
  }
  const float b3 = params[kOffB3];
  f32x4 g1[kC1], g2[kHid / 16];
#pragma unroll
  for (int c = 0; c < kC1; ++c) g1[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < kHid / 16; ++c) g2[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float gb1[4] = {}, gb2[4] = {}, gw3[4] = {}, gb3 = 0.f, lsum = 0.f;
  const float inv_b = 1.0f / (float)B;
  for (int i = tg; i < kTrainTile * kTStride; i += kTrainGroup) xs[i] = 0.f;  // columns 67.. stay 0
  const uint32_t tiles = (B + kTrainTile - 1) / kTrainTile;
  for (uint32_t tile0 = blockIdx.x * kTrainGroups; tile0 < tiles; tile0 += gridDim.x * kTrainGroups) {
    const uint32_t tile = tile0 + grp, s0 = tile * kTrainTile;
    // samples of this group's tile; 0 past the last tile
    const uint32_t ns = tile >= tiles ? 0u : B - s0 < (uint32_t)kTrainTile ? B - s0 : (uint32_t)kTrainTile;
    __syncthreads();  // the previous tile's readers of xs are done
    for (uint32_t i = tg; i < kTrainTile * kIn; i += kTrainGroup) {
      const uint32_t s = i / kIn, k = i - s * kIn;
      xs[s * kTStride + k] = s < ns ? feats[(uint64_t)s0 * kIn + i] : 0.f;
    }
    const bool live = (uint32_t)col < ns;  // a column past the batch adds nothing, whatever its activations
    const float target = live ? targets[s0 + col] : 0.f;
    __syncthreads();
    f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < kK1; ++t)
      z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1a[t], xs[col * kTStride + 4 * t + q], z, 0, 0, 0);
    float d1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float h;
      gelu_both(z[i] + b1[i], h, d1[i]);
      h1s[col * kTStride + row0 + 4 * q + i] = live ? h : 0.f;
    }
    __syncthreads();
    z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < kHid / 4; ++t)
      z = __builtin_amdgcn_mfma_f32_16x16x4f32(w2s[(row0 + col) * kTStride + 4 * t + q], h1s[col * kTStride + 4 * t + q], z, 0, 0, 0);
    float h2[4], d2[4], part = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      gelu_both(z[i] + b2[i], h2[i], d2[i]);
      part += w3[i] * h2[i];
    }
    part += __shfl_xor(part, 16);
    part += __shfl_xor(part, 32);
    if (q == 0) ys[wave * kTrainTile + col] = part;
    __syncthreads();
    float y = b3;
#pragma unroll
    for (int w = 0; w < kTrainGroup / 64; ++w) y += ys[w * kTrainTile + col];
    const float r = live ? y - target : 0.f;
    const float dy = 2.0f * r * inv_b;
    if (wave == 0 && q == 0) {
      lsum += r * r * inv_b;
      gb3 += dy;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      gw3[i] += live ? dy * h2[i] : 0.f;
      const float dz2 = live ? dy * w3[i] * d2[i] : 0.f;
      gb2[i] += dz2;
      dz2s[col * kTStride + row0 + 4 * q + i] = dz2;
    }
    __syncthreads();
    z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < kHid / 4; ++t)
      z = __builtin_amdgcn_mfma_f32_16x16x4f32(w2s[(4 * t + q) * kTStride + row0 + col], dz2s[col * kTStride + 4 * t + q], z, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float dz1 = live ? z[i] * d1[i] : 0.f;
      gb1[i] += dz1;
      dz1s[col * kTStride + row0 + 4 * q + i] = dz1;  // read by this wave only
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll 2
    for (int t = 0; t < kTrainTile / 4; ++t) {
      const int s = 4 * t + q;
      const float a2 = dz2s[s * kTStride + row0 + col], a1 = dz1s[s * kTStride + row0 + col];
#pragma unroll
      for (int c = 0; c < kHid / 16; ++c)
        g2[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a2, h1s[s * kTStride + 16 * c + col], g2[c], 0, 0, 0);
#pragma unroll
      for (int c = 0; c < kC1; ++c)
        g1[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, xs[s * kTStride + 16 * c + col], g1[c], 0, 0, 0);
    }
  }
  // sums over the samples (the 16 columns) of the unit gradients
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      gb1[i] += __shfl_xor(gb1[i], d);
      gb2[i] += __shfl_xor(gb2[i], d);
      gw3[i] += __shfl_xor(gw3[i], d);
    }
    gb3 += __shfl_xor(gb3, d);
    lsum += __shfl_xor(lsum, d);
  }
  // v = f(parameter index, v) for every gradient v this lane holds
  auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = row0 + 4 * q + i;
#pragma unroll
      for (int c = 0; c < kC1; ++c)
        if (16 * c + col < kIn) g1[c][i] = f(kOffW1 + u * kIn + 16 * c + col, g1[c][i]);
#pragma unroll
      for (int c = 0; c < kHid / 16; ++c) g2[c][i] = f(kOffW2 + u * kHid + 16 * c + col, g2[c][i]);
      if (col == 0) {
        gb1[i] = f(kOffB1 + u, gb1[i]);
        gb2[i] = f(kOffB2 + u, gb2[i]);
        gw3[i] = f(kOffW3 + u, gw3[i]);
      }
    }
    if (tg == 0) gb3 = f(kOffB3, gb3);
  };
  __shared__ float lsums[kTrainGroups];
  if (tg == 0) lsums[grp] = lsum;
  // groups 1 and 3 to 0 and 2, then 2 to 0
  float* half = train_lds + (grp >> 1) * kParams;
  __syncthreads();
  if (grp & 1) each([&](int at, float v) { return half[at] = v; });
  __syncthreads();
  if (!(grp & 1)) each([&](int at, float v) { return v + half[at]; });
  if (grp == 2) each([&](int at, float v) { return half[at] = v; });  // each lane's own places, read above
  __syncthreads();
  if (grp == 0) {
    const float* other = train_lds + kParams;
    each([&](int at, float v) { return atomicAdd(&grads[at], v + other[at]), v; });
    if (tg == 0 && loss) atomicAdd(loss, (lsums[0] + lsums[1]) + (lsums[2] + lsums[3]));
  }
}

__global__ void k_adam(float* __restrict__ params, float* __restrict__ grads, float* __restrict__ m1,
                       float* __restrict__ m2, float lr, float beta1, float beta2, float eps, float bc1, float bc2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kParams) return;
  const float gr = grads[i];
  const float a = beta1 * m1[i] + (1.0f - beta1) * gr;
  const float v = beta2 * m2[i] + (1.0f - beta2) * gr * gr;
  m1[i] = a;
  m2[i] = v;
  params[i] -= lr * (a / bc1) / (sqrtf(v / bc2) + eps);
  grads[i] = 0.f;
}

__global__ void k_zero_f32(float* __restrict__ p, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

}  // namespace

struct vbdr_mlp {
  int device;
  MlpDev* dev;
};

struct vbdr_trainer {
  int device;
  float *params, *grads, *m1, *m2;
  uint64_t step;
  float lr, beta1, beta2, eps;
};

extern "C" {

int vbdr_mlp_create(const float* params_host, const float* env_lo, const float* env_hi, vbdr_mlp** out) {
  if (!params_host || !out) return vbdr_fail(VBDR_EINVAL, "NULL argument");
  if ((env_lo == nullptr) != (env_hi == nullptr)) return vbdr_fail(VBDR_EINVAL, "give both envelope bounds or none");
  *out = nullptr;
  std::vector<uint8_t> buf(sizeof(MlpDev), 0);
  MlpDev* h = reinterpret_cast<MlpDev*>(buf.data());
  for (int j = 0; j < kHid; ++j) {
    for (int k = 0; k < kIn; ++k) h->w1[j * kInPad + k] = f2bf(params_host[kOffW1 + j * kIn + k]);
    for (int ks = 0; ks < 2; ++ks)
      for (int q = 0; q < 4; ++q)
        for (int i = 0; i < 8; ++i)
          h->w2p[j * kHid + 32 * ks + 8 * q + i] = f2bf(params_host[kOffW2 + j * kHid + l2_unit(ks, q, i)]);
    h->b1[j] = params_host[kOffB1 + j];
    h->b2[j] = params_host[kOffB2 + j];
    h->w3[j] = bf2f(f2bf(params_host[kOffW3 + j]));
  }
  h->b3 = params_host[kOffB3];
  h->has_env = env_lo != nullptr;
  h->plain_above = INFINITY;
  for (int k = 0; k < kIn; ++k) {
    h->env_lo[k] = env_lo ? env_lo[k] : 0.f;
    h->env_hi[k] = env_hi ? env_hi[k] : 0.f;
  }
  vbdr_mlp* mlp = new (std::nothrow) vbdr_mlp();
  if (!mlp) return vbdr_fail(VBDR_ENOMEM, "host allocation failed");
  if (hipGetDevice(&mlp->device) != hipSuccess || vbdr_malloc(&mlp->dev, sizeof(MlpDev)) != hipSuccess) {
    delete mlp;
    return vbdr_fail(VBDR_ENOMEM, "device allocation of the MLP failed");
  }
  if (hipMemcpy(mlp->dev, h, sizeof(MlpDev), hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipFree(mlp->dev);
    delete mlp;
    return vbdr_fail(VBDR_EHIP, "upload of the MLP failed");
  }
  *out = mlp;
  return VBDR_OK;
}

int vbdr_mlp_set_plain_above(vbdr_mlp* mlp, float threshold) {
  if (!mlp) return vbdr_fail(VBDR_EINVAL, "mlp is NULL");
  if (!(threshold > 0.0f)) return vbdr_fail(VBDR_EINVAL, "threshold must be positive (INFINITY: never)");
  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess || cur != mlp->device)
    return vbdr_fail(VBDR_EINVAL, "the network lives on device %d, not the current one", mlp->device);
  if (hipMemcpy(reinterpret_cast<uint8_t*>(mlp->dev) + offsetof(MlpDev, plain_above), &threshold, sizeof(float),
                hipMemcpyHostToDevice) != hipSuccess)
    return vbdr_fail(VBDR_EHIP, "upload of the threshold failed");
  return VBDR_OK;
}

void vbdr_mlp_destroy(vbdr_mlp* mlp) {
  if (!mlp) return;
  (void)hipDeviceSynchronize();
  (void)hipFree(mlp->dev);
  delete mlp;
}

int vbdr_features(vbdr_sketch* sk, const uint32_t* hosts_dev, uint64_t n_hosts, float* feats_dev, void* stream) {
  if (!sk) return vbdr_fail(VBDR_EINVAL, "sketch is NULL");
  if (n_hosts == 0) return VBDR_OK;
  if (!hosts_dev || !feats_dev) return vbdr_fail(VBDR_EINVAL, "hosts_dev and feats_dev must not be NULL");
  if (int rc = vbdr_check_device(sk)) return rc;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const uint32_t chunk = vbdr_hist_chunk(sk), parts = vbdr_gather_parts(sk);
  for (uint64_t c = 0; c < n_hosts; c += chunk) {
    const uint32_t nh = (uint32_t)(n_hosts - c < chunk ? n_hosts - c : chunk);
    if (int rc = vbdr_hist_pass(sk, hosts_dev + c, nh, st)) return rc;
    hipLaunchKernelGGL(k_features, dim3((uint32_t)(((uint64_t)nh * kIn + 255) / 256)), dim3(256), 0, st, nh, parts, chunk,
                       sk->hist_ws, sk->hist, sk->g, (uint32_t)sk->m, feats_dev + c * kIn);
    VBDR_LAUNCHED("k_features");
  }
  return VBDR_OK;
}

int vbdr_estimate_learned(vbdr_sketch* sk, const vbdr_mlp* mlp, const uint32_t* hosts_dev, uint64_t n_hosts,
                          float* out_dev, uint8_t* used_fallback_dev, void* stream) {
  if (!sk || !mlp) return vbdr_fail(VBDR_EINVAL, "sketch and mlp must not be NULL");
  if (n_hosts == 0) return VBDR_OK;
  if (!hosts_dev || !out_dev) return vbdr_fail(VBDR_EINVAL, "hosts_dev and out_dev must not be NULL");
  if (mlp->device != sk->device) return vbdr_fail(VBDR_EINVAL, "mlp and sketch live on different devices");
  if (int rc = vbdr_check_device(sk)) return rc;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const uint32_t parts = vbdr_gather_parts(sk), chunk = vbdr_hist_chunk(sk);
  // Few hosts of large g on a pool that fills the L2s: a workgroup that gathers 16 of them waits for its CU's misses, so
  // the histogram pass spreads them wider (2^23 BDRs: g = 8192, 64 hosts 120 us in one launch, 48 in two; g = 2048,
  // 600 hosts 35 and 26).  Smaller pools, which have always used no workspace here, stay with one launch.
  const bool pass = sk->g >= 2048 && sk->m >= kPartMinM && n_hosts <= 4 * (uint64_t)sk->n_cu;
  if (parts == 1 && sk->g <= kStageMaxG && n_hosts < (1ull << 32) && !pass) {
    // registers cache resident: one fused launch, gathers feed the MLP tile directly
    const uint32_t nh = (uint32_t)n_hosts;
    const uint32_t tiles = (uint32_t)((n_hosts + 15) / 16);
    const uint32_t want = (tiles + kInfWaves - 1) / kInfWaves;
    const uint32_t cap = (uint32_t)sk->n_cu * 8;
    const bool spread = tiles <= (uint32_t)sk->n_cu * (sk->g >= kSpreadWideG ? 2 : 1);
    hipLaunchKernelGGL((spread ? k_learned<true, true> : k_learned<true>), dim3(spread ? tiles : want < cap ? want : cap),
                       dim3(spread ? kSpreadBlock : kInfBlock), (size_t)sk->g * 4, st, nh, 1u, 0u,
                       (const uint32_t*)nullptr, hosts_dev, sk->s1, sk->reg, sk->reg4, sk->hist, sk->g, (uint32_t)sk->m,
                       mlp->dev, out_dev, used_fallback_dev);
    VBDR_LAUNCHED("k_learned(direct)");
    return VBDR_OK;
  }
  for (uint64_t c = 0; c < n_hosts; c += chunk) {
    const uint32_t nh = (uint32_t)(n_hosts - c < chunk ? n_hosts - c : chunk);
    if (int rc = vbdr_hist_pass(sk, hosts_dev + c, nh, st)) return rc;
    const uint32_t tiles = (nh + 15) / 16;
    const uint32_t want = (tiles + kInfWaves - 1) / kInfWaves;
    const uint32_t cap = (uint32_t)sk->n_cu * 4;
    hipLaunchKernelGGL(k_learned<false>, dim3(want < cap ? want : cap), dim3(kInfBlock), 0, st, nh,
                       parts, chunk, sk->hist_ws, (const uint32_t*)nullptr, (const uint32_t*)nullptr,
                       (const uint8_t*)nullptr, (const uint8_t*)nullptr, sk->hist, sk->g, (uint32_t)sk->m, mlp->dev, out_dev + c,
                       used_fallback_dev ? used_fallback_dev + c : nullptr);
    VBDR_LAUNCHED("k_learned");
  }
  return VBDR_OK;
}

int vbdr_trainer_create(const float* params_host, float lr, vbdr_trainer** out) {
  if (!params_host || !out) return vbdr_fail(VBDR_EINVAL, "NULL argument");
  if (!(lr > 0.f)) return vbdr_fail(VBDR_EINVAL, "learning rate must be positive");
  *out = nullptr;
  vbdr_trainer* tr = new (std::nothrow) vbdr_trainer();
  if (!tr) return vbdr_fail(VBDR_ENOMEM, "host allocation failed");
  std::memset(tr, 0, sizeof(*tr));
  tr->lr = lr, tr->beta1 = 0.9f, tr->beta2 = 0.999f, tr->eps = 1e-8f;
  const size_t bytes = kParams * sizeof(float);
  if (hipGetDevice(&tr->device) != hipSuccess || vbdr_malloc(&tr->params, bytes) != hipSuccess ||
      vbdr_malloc(&tr->grads, bytes) != hipSuccess || vbdr_malloc(&tr->m1, bytes) != hipSuccess ||
      vbdr_malloc(&tr->m2, bytes) != hipSuccess) {
    vbdr_trainer_destroy(tr);
    return vbdr_fail(VBDR_ENOMEM, "device allocation of the trainer failed");
  }
  const uint32_t grid = (kParams + 255) / 256;
  hipLaunchKernelGGL(k_zero_f32, dim3(grid), dim3(256), 0, nullptr, tr->grads, (uint32_t)kParams);
  hipLaunchKernelGGL(k_zero_f32, dim3(grid), dim3(256), 0, nullptr, tr->m1, (uint32_t)kParams);
  hipLaunchKernelGGL(k_zero_f32, dim3(grid), dim3(256), 0, nullptr, tr->m2, (uint32_t)kParams);
  if (hipGetLastError() != hipSuccess || hipMemcpy(tr->params, params_host, bytes, hipMemcpyHostToDevice) != hipSuccess) {
    vbdr_trainer_destroy(tr);
    return vbdr_fail(VBDR_EHIP, "trainer initialisation failed");
  }
  *out = tr;
  return VBDR_OK;
}

void vbdr_trainer_destroy(vbdr_trainer* tr) {
  if (!tr) return;
  (void)hipDeviceSynchronize();
  if (tr->params) (void)hipFree(tr->params);
  if (tr->grads) (void)hipFree(tr->grads);
  if (tr->m1) (void)hipFree(tr->m1);
  if (tr->m2) (void)hipFree(tr->m2);
  delete tr;
}

int vbdr_trainer_set_lr(vbdr_trainer* tr, float lr) {
  if (!tr || !(lr > 0.f)) return vbdr_fail(VBDR_EINVAL, "bad trainer or learning rate");
  tr->lr = lr;
  return VBDR_OK;
}

int vbdr_trainer_grad(vbdr_trainer* tr, const float* feats_dev, const float* targets_dev, uint64_t n, float* grads_out_dev,
                      float* loss_dev, void* stream) {
  if (!tr || !feats_dev || !targets_dev || !grads_out_dev) return vbdr_fail(VBDR_EINVAL, "NULL argument");
  if (n == 0 || n >= (1ull << 31)) return vbdr_fail(VBDR_EINVAL, "batch size out of range");
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const uint32_t tiles = (uint32_t)((n + kTrainTile - 1) / kTrainTile);
  const uint32_t want = (tiles + kTrainGroups - 1) / kTrainGroups;
  hipLaunchKernelGGL(k_train_grad, dim3(want < kTrainGrid ? want : kTrainGrid), dim3(kTrainBlock),
                     sizeof(float) * (kTrainGroups * kTrainLds + kHid * kTStride), st, tr->params, feats_dev, targets_dev, (uint32_t)n,
                     grads_out_dev, loss_dev);
  VBDR_LAUNCHED("k_train_grad");
  return VBDR_OK;
}

int vbdr_trainer_step(vbdr_trainer* tr, const float* feats_dev, const float* targets_dev, uint64_t n, float* loss_dev,
                      void* stream) {
  if (int rc = vbdr_trainer_grad(tr, feats_dev, targets_dev, n, tr ? tr->grads : nullptr, loss_dev, stream)) return rc;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  tr->step++;
  const float bc1 = 1.0f - powf(tr->beta1, (float)tr->step), bc2 = 1.0f - powf(tr->beta2, (float)tr->step);
  hipLaunchKernelGGL(k_adam, dim3((kParams + 255) / 256), dim3(256), 0, st, tr->params, tr->grads, tr->m1, tr->m2,
                     tr->lr, tr->beta1, tr->beta2, tr->eps, bc1, bc2);
  VBDR_LAUNCHED("k_adam");
  return VBDR_OK;
}

int vbdr_trainer_params(vbdr_trainer* tr, float* params_host, void* stream) {
  if (!tr || !params_host) return vbdr_fail(VBDR_EINVAL, "NULL argument");
  VBDR_HIP(hipStreamSynchronize(reinterpret_cast<hipStream_t>(stream)));
  VBDR_HIP(hipMemcpy(params_host, tr->params, kParams * sizeof(float), hipMemcpyDeviceToHost));
  return VBDR_OK;
}

}  // extern "C"
