// Device-side primitives of the VBDR hot path (gfx950).  Internal header of
// libvbdr.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vbdr {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct TrueType {
  static constexpr bool value = true;
};
struct FalseType {
  static constexpr bool value = false;
};
template <int N>
struct Int {
  static constexpr int value = N;
};

constexpr int kBins = 33;     // register values 0..32
constexpr uint32_t kSat = 255; // DR saturation value (InitDR with z = 8)

// MurmurHash3_x86_32 of one 4-byte little-endian key, H(x, 2^32, A)
// (Sec. 4.1 leaves the hash family open; this is the chosen member), split for
// many seeds over one key: mm3_key(x) is the seed-independent block mix,
// mm3_seeded(mm3_key(x), A) == mm3(x, A).  Rotations by v_alignbit: from
// shifts the compiler makes a second multiply of mm3_key's (scans 1 % longer).
__device__ __forceinline__ uint32_t rotl32(uint32_t x, uint32_t r) { return __builtin_amdgcn_alignbit(x, x, 32u - r); }
__device__ __forceinline__ uint32_t mm3_key(uint32_t x) { return rotl32(x * 0xcc9e2d51u, 15) * 0x1b873593u; }
__device__ __forceinline__ uint32_t mm3_seeded(uint32_t kmix, uint32_t seed) {
  uint32_t h = rotl32(seed ^ kmix, 13) * 5u + 0xe6546b64u;
  h ^= 4u;
  h ^= h >> 16;
  h *= 0x85ebca6bu;
  h ^= h >> 13;
  h *= 0xc2b2ae35u;
  h ^= h >> 16;
  return h;
}
__device__ __forceinline__ uint32_t mm3(uint32_t x, uint32_t seed) { return mm3_seeded(mm3_key(x), seed); }

// H(x, m, A) for m < 2^32: the top 32 bits of the 64-bit product h * m.
__device__ __forceinline__ uint32_t reduce_m(uint32_t h, uint32_t m) { return __umulhi(h, m); }

// (vidx, LBP1) of a bip (Alg. 4/7/9): vidx = left b bits of H(bip, 2^32, A1);
// LBP1 = 1 + leading zeros of the remaining 32-b bits, 33-b when they are all
// zero (the sentinel bit 1 << (b-1) caps the count).
__device__ __forceinline__ void bip_map(uint32_t bip, uint32_t A1, uint32_t b, uint32_t& vidx, uint32_t& rho) {
  uint32_t h = mm3(bip, A1);
  vidx = h >> (32 - b);
  rho = __clz((h << b) | (1u << (b - 1))) + 1;
}

// ---- byte-wise (SWAR) operations on four one-byte DRs held in a uint32 ----

// Saturating increment of every byte (SlideDR): bytes below 255 gain 1.  On the
// device each byte sits in the high half of a 16-bit lane for a packed add that
// saturates at 0xFFFF, and v_perm collects the four high bytes: 4 instructions.
__host__ __device__ __forceinline__ uint32_t swar_sat_inc(uint32_t x) {
#ifdef __HIP_DEVICE_COMPILE__
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  const u16x2 one = {0x0100, 0x0100};
  const uint32_t odd = __builtin_bit_cast(uint32_t, __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, x), one));
  const uint32_t even = __builtin_bit_cast(uint32_t, __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, x << 8), one));
  return __builtin_amdgcn_perm(odd, even, 0x07030501u);
#else
  const uint32_t t = ~x;  // a byte of t is zero exactly where x holds 255
  const uint32_t not_sat = (((t & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | t) & 0x80808080u;
  return x + (not_sat >> 7);
#endif
}

// 0xFF in byte j for each set bit j of a 4-bit mask.
__host__ __device__ __forceinline__ uint32_t swar_nibble_to_bytes(uint32_t f4) {
  return ((f4 * 0x00204081u) & 0x01010101u) * 0xFFu;
}

// x with byte j zeroed for each set bit j of a 4-bit mask (SetDR): the mask's
// bits, 4 to a byte, turn a byte selector from x's bytes to zero's.
__device__ __forceinline__ uint32_t swar_zero_bytes(uint32_t x, uint32_t f4) {
  const uint32_t spread = __umul24(f4, 0x00204081u) & 0x01010101u;
  return __builtin_amdgcn_perm(0u, x, 0x03020100u + (spread << 2));
}

// Bias for swar_le_mask: each byte value v sits in its own 16-bit lane, where
// v + (255 - thr) carries into bit 8 exactly when v > thr.
__host__ __device__ __forceinline__ uint32_t swar_gt_bias(uint32_t thr) { return (0xFFu - thr) * 0x00010001u; }

// 0xFF in every byte whose value is <= thr (thr < 255).
__host__ __device__ __forceinline__ uint32_t swar_le_mask(uint32_t v, uint32_t bias) {
  const uint32_t even = ((((v & 0x00FF00FFu) + bias) >> 8) & 0x00010001u);
  const uint32_t odd = ((((v >> 8) & 0x00FF00FFu) + bias) & 0x01000100u);
  return ((even | odd) ^ 0x01010101u) * 0xFFu;
}

// Bit 7 of every byte whose value is below c, for 1 <= c <= 128 (cc = c in
// every byte): (x | 0x80) - c cannot borrow across bytes, and its bit 7 is
// set exactly when (x & 0x7F) >= c; a byte is below c when neither that bit
// nor its own bit 7 is set.  Four operations against the eight or so of
// swar_le_mask, for windows of k <= 128 slices (active DR: DR < k).
__host__ __device__ __forceinline__ uint32_t swar_lt_bit7(uint32_t x, uint32_t cc) {
  const uint32_t t = (x | 0x80808080u) - cc;
  return ~(x | t) & 0x80808080u;
}

// Four register bytes (<= 32) -> four nibbles min(r, 15), byte j -> bits 4j..4j+3.
__host__ __device__ __forceinline__ uint32_t swar_pack_nibbles(uint32_t r) {
  const uint32_t ge15 = ((r + 0x71717171u) & 0x80808080u) >> 7;  // 1 where r >= 15
  const uint32_t c = (r & ~(ge15 * 0xFFu)) | (ge15 * 0x0Fu);
  const uint32_t t = (c | (c >> 4)) & 0x00FF00FFu;
  return (t & 0xFFu) | ((t >> 8) & 0xFF00u);
}

// HyperLogLog alpha_q (Flajolet et al. 2007).
__device__ __forceinline__ double hll_alpha(double q) {
  if (q == 16.0) return 0.673;
  if (q == 32.0) return 0.697;
  if (q == 64.0) return 0.709;
  return 0.7213 / (1.0 + 1.079 / q);
}

// HyperLogLog estimate of q registers whose harmonic sum is U * 2^-32 and of
// which V are zero; linear counting when the raw estimate is <= 2.5 q.
// Each FP64 operation rounds once (no contraction) so that results are
// reproducible across compilers.
__device__ __forceinline__ double hll_estimate(uint64_t U, uint64_t V, double q) {
#pragma clang fp contract(off)
  double S = (double)U * 0x1p-32;
  double E = hll_alpha(q) * q * q / S;
  if (E <= 2.5 * q && V > 0) E = q * log(q / (double)V);
  return E;
}

// ---- per-item bodies shared by the single-sketch and the batched kernels ----

// Scan N pairs (Alg. 7 / Alg. 9 with the hashing of Alg. 4 and getPhyIdx of
// Alg. 3), valid where ok[v].  Fast layout: set bit pidx of bsLBP1 bit-plane
// LBP1-1 with a device-scope atomic OR; small layout: store 0 into DR[LBP1] of
// BDR pidx.  TEST: read first and skip an update that is already made.  The
// state words of all N are located first and, with TEST, read together, so
// that the N random reads overlap instead of each waiting for the one before.
template <bool FAST, bool TEST, int N>
__device__ __forceinline__ void scan_pairs(const u32x2* p, const bool* ok, const uint32_t* s1, uint32_t b, uint32_t A1,
                                           uint32_t m, uint8_t* dr, uint64_t mstride, uint32_t* seen,
                                           uint64_t wstride) {
  uint64_t off[N];
  uint32_t bit[N];
#pragma unroll
  for (int v = 0; v < N; ++v) {
    off[v] = 0;
    bit[v] = 0;
    if (ok[v]) {
      uint32_t vidx, rho;
      bip_map(p[v].y, A1, b, vidx, rho);
      const uint32_t pidx = reduce_m(mm3(p[v].x, s1[vidx]), m);
      off[v] = FAST ? (uint64_t)(rho - 1) * wstride + (pidx >> 5) : (uint64_t)(rho - 1) * mstride + pidx;
      bit[v] = 1u << (pidx & 31);
    }
  }
  uint32_t cur[N];
#pragma unroll
  for (int v = 0; v < N; ++v) cur[v] = TEST && ok[v] ? (FAST ? seen[off[v]] : (uint32_t)dr[off[v]]) : (FAST ? 0u : 1u);
#pragma unroll
  for (int v = 0; v < N; ++v) {
    if (!ok[v]) continue;
    if constexpr (FAST) {
      if (!(cur[v] & bit[v])) atomicOr(seen + off[v], bit[v]);
    } else {
      if (cur[v] != 0) dr[off[v]] = 0;
    }
  }
}

// 4 W consecutive bytes (DRs, registers), four to a word; W = 4 or 8 (2: nibbles of 16).
template <int W>
struct DrWords {
  uint32_t v[W];
};
template <int W>
__device__ __forceinline__ DrWords<W> load_dr(const uint8_t* p) {
  DrWords<W> d;
#pragma unroll
  for (int q = 0; q < W / 4; ++q) {
    const u32x4 t = *reinterpret_cast<const u32x4*>(p + 16 * q);
#pragma unroll
    for (int w = 0; w < 4; ++w) d.v[4 * q + w] = t[w];
  }
  return d;
}
template <int W>
__device__ __forceinline__ void store_dr(uint8_t* p, const DrWords<W>& d) {
  if constexpr (W == 2) {
    *reinterpret_cast<u32x2*>(p) = u32x2{d.v[0], d.v[1]};
  } else {
#pragma unroll
    for (int o = 0; o < W; o += 4)
      *reinterpret_cast<u32x4*>(p + 4 * o) = u32x4{d.v[o], d.v[o + 1], d.v[o + 2], d.v[o + 3]};
  }
}
// Store d, vector by vector, where it differs from what was loaded: a
// saturated DR that was not set this slice stays 255, so most of the high
// planes, whose DRs are rarely set, are not written back.
template <int W>
__device__ __forceinline__ void store_dr_changed(uint8_t* p, const DrWords<W>& d, const DrWords<W>& was) {
#pragma unroll
  for (int q = 0; q < W / 4; ++q) {
    const int o = 4 * q;
    if ((d.v[o] ^ was.v[o]) | (d.v[o + 1] ^ was.v[o + 1]) | (d.v[o + 2] ^ was.v[o + 2]) | (d.v[o + 3] ^ was.v[o + 3]))
      *reinterpret_cast<u32x4*>(p + 16 * q) = u32x4{d.v[o], d.v[o + 1], d.v[o + 2], d.v[o + 3]};
  }
}

// Advance planes hi down to lo of 4 W consecutive BDRs starting at `base` (a
// multiple of 4 W); the planes of a BDR may be split over several threads.  The slice's LBP1 bits of those BDRs come as
// one word per plane, pm[(i - 1) * pm_stride] bit sh + j <-> BDR base + j (the
// tile's records and bsLBP1 words, gathered in LDS).  Small layout (Alg. 8): a
// set bit means DR[i] was set to 0 during the slice (Alg. 9), so it is zeroed;
// the window is read, then the DRs slide.  Fast layout (Alg. 6): every DR
// slides, then the DR of the slice's highest LBP1 is zeroed and the window is
// read (folded: the slice's bits of the planes above hi).  Register (Alg. 2):
// the largest LBP1 whose DR is active, DR <= k-1 at the moment the window is
// read.  R receives it for these planes, 0 if none is active (byte j of word w
// = BDR base + 4w + j).  With PCSA (small layout) Q receives the lowest
// inactive LBP1 of these planes minus 1, 255 if all are active: the least over
// all planes, at most L, is the run of consecutive active DRs from LBP1 1.
// G planes are loaded together, one group ahead of the one being processed, in
// two register buffers (a rotation by copies would wait for the loads just
// issued).  Bit r-1 of sat_in: these DR[r] were all 255 after the last advance
// and nothing but the advance has written DRs since; with no record of this
// slice in that plane they are 255 now and stay 255, so they are neither
// loaded nor stored.
template <bool FAST, bool PCSA, int W, int G>
__device__ __forceinline__ void advance_words(uint8_t* dr, uint64_t mstride, uint64_t base, int hi, int lo,
                                              uint32_t folded, uint32_t gt_bias, uint32_t kk, const uint32_t* pm,
                                              uint32_t pm_stride, uint32_t sh, uint32_t sat_in, uint32_t& sat_out,
                                              DrWords<W>& Rd, DrWords<W>& Qd) {
  uint32_t(&R)[W] = Rd.v;
  uint32_t(&Q)[W] = Qd.v;
  constexpr uint32_t mask = W == 8 ? ~0u : (1u << (4 * (W & 7))) - 1u;
  uint32_t M[W];
#pragma unroll
  for (int w = 0; w < W; ++w) {
    M[w] = R[w] = 0;
    Q[w] = ~0u;
  }
  uint32_t sat = 0;
  // M: bit 7 of the BDRs with an active DR at or above the plane; the planes down to 1 with it count the register
  auto found = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int w = 0; w < W; ++w) R[w] += M[w] >> 7;
  };
  auto bits_of = [&](int r) -> uint32_t { return (pm[(uint32_t)(r - 1) * pm_stride] >> sh) & mask; };
  auto load_group = [&](int top, DrWords<W>(&d)[G]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int r = top - j;
      if (r >= lo && !(((sat_in >> (r - 1)) & 1u) && bits_of(r) == 0u)) {
        d[j] = load_dr<W>(dr + (uint64_t)(r - 1) * mstride + base);
      } else {
#pragma unroll
        for (int w = 0; w < W; ++w) d[j].v[w] = ~0u;
      }
    }
  };
  auto process = [&](int top, const DrWords<W>(&d)[G]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int i = top - j;
      if (i < lo) break;
      const uint32_t bits = bits_of(i);
      uint32_t fold = 0;
      if constexpr (FAST) {
        fold = bits & ~folded;  // only the slice's highest LBP1 is recorded
        folded |= bits;
      }
      // DRs at 255 with no record this slice stay 255, none is active and
      // nothing is stored: the SWAR work below is skipped, by whole waves for
      // most of the high planes.  Decided from the loaded bytes, so it holds
      // whether or not the saturation masks were trusted.
      uint32_t all = ~0u;
#pragma unroll
      for (int w = 0; w < W; ++w) all &= d[j].v[w];
      if (bits == 0u && all == ~0u) {
        sat |= 1u << (i - 1);
        found();
        if (PCSA)
#pragma unroll
          for (int w = 0; w < W; ++w) Q[w] = (uint32_t)(i - 1) * 0x01010101u;  // no active DR: the run restarts below
        continue;
      }
      DrWords<W> x = d[j], nd;
      if constexpr (!FAST) {
        if (bits)
#pragma unroll
          for (int w = 0; w < W; ++w) x.v[w] = swar_zero_bytes(x.v[w], (bits >> (4 * w)) & 0xFu);  // SetDR of the slice
      }
#pragma unroll
      for (int w = 0; w < W; ++w) nd.v[w] = swar_sat_inc(x.v[w]);  // SlideDR
      if constexpr (FAST) {
        if (fold)
#pragma unroll
          for (int w = 0; w < W; ++w) nd.v[w] = swar_zero_bytes(nd.v[w], (fold >> (4 * w)) & 0xFu);  // SetDR
      }
      const DrWords<W>& v = FAST ? nd : x;  // the DRs that the window is read from
      uint32_t a7[W];                      // IsActiveDR: bit 7
      if (kk) {
#pragma unroll
        for (int w = 0; w < W; ++w) a7[w] = swar_lt_bit7(v.v[w], kk);
      } else {
#pragma unroll
        for (int w = 0; w < W; ++w) a7[w] = swar_le_mask(v.v[w], gt_bias) & 0x80808080u;
      }
#pragma unroll
      for (int w = 0; w < W; ++w) {
        M[w] |= a7[w];
        // an inactive DR: the run restarts below; an active one keeps it
        if (PCSA) Q[w] = __builtin_amdgcn_perm((uint32_t)(i - 1) * 0x01010101u, Q[w], 0x07060504u - (a7[w] >> 5));
      }
      found();
      store_dr_changed<W>(dr + (uint64_t)(i - 1) * mstride + base, nd, d[j]);
      all = ~0u;
#pragma unroll
      for (int w = 0; w < W; ++w) all &= nd.v[w];
      if (all == ~0u) sat |= 1u << (i - 1);
    }
  };
  DrWords<W> a[G], b[G];
  load_group(hi, a);
  for (int top = hi; top >= lo; top -= 2 * G) {
    load_group(top - G, b);
    process(top, a);
    if (top - G < lo) break;
    load_group(top - 2 * G, a);
    process(top - G, b);
  }
  sat_out = sat;
  if (lo > 1)  // the planes below lo count too
#pragma unroll
    for (int w = 0; w < W; ++w) R[w] += (M[w] >> 7) * (uint32_t)(lo - 1);
}

// The registers of 4 W BDRs as nibbles min(r, 15).
template <int W>
__device__ __forceinline__ void store_nibbles(uint8_t* reg4, uint64_t base, const DrWords<W>& R) {
  DrWords<W / 2> nib;
#pragma unroll
  for (int q = 0; q < W / 2; ++q)
    nib.v[q] = swar_pack_nibbles(R.v[2 * q]) | (swar_pack_nibbles(R.v[2 * q + 1]) << 16);
  store_dr<W / 2>(reg4 + base / 2, nib);
}

// Sum of the four bytes of x when it is below 256.
__device__ __forceinline__ uint32_t byte_sum(uint32_t x) { return (x * 0x01010101u) >> 24; }

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t olo = __shfl_xor(lo, off), ohi = __shfl_xor(hi, off);
    const uint64_t s = ((uint64_t)hi << 32 | lo) + ((uint64_t)ohi << 32 | olo);
    lo = (uint32_t)s, hi = (uint32_t)(s >> 32);
  }
  return (uint64_t)hi << 32 | lo;
}

// Noise-removed estimate (m E_s - g E_m) / (m - g), each operation rounded once.
__device__ __forceinline__ double noise_removed(double Es, double Em, double m, double g) {
#pragma clang fp contract(off)
  return (m * Es - g * Em) / (m - g);
}

// A sketch's pool statistics (kStatWords uint64): the register histogram of
// the last closed window, its E_m (bits of a double), the sum of all registers
// and how many are 15 and more; then the running sums of an advance in flight and its count of
// finished workgroups, zero between advances.
constexpr int kStatEm = 33, kStatSum = 34, kStatWide = 35, kStatAcc = 64, kStatTicket = kStatAcc + kBins, kStatWords = 128;
__device__ __forceinline__ double stat_em(const unsigned long long* stats) {
  return __longlong_as_double((long long)stats[kStatEm]);
}

// Whether gathers read the registers' bytes and not their nibbles, of which each
// 15 is read again: pools whose bytes an XCD's L2 holds and of which a share of
// 1 / WIDE is 15 and more; in LDS, pools of up to kBytesTabM BDRs.
constexpr uint32_t kBytesMaxM = 1u << 22, kBytesTabM = 1u << 16;
template <uint32_t WIDE>
__device__ __forceinline__ bool gather_bytes(const unsigned long long* stats, uint32_t m) {
  return m <= kBytesMaxM && WIDE * stats[kStatWide] > m;
}

// E_m: the HyperLogLog estimate over all m registers from their histogram.
__device__ __forceinline__ double pool_estimate(const unsigned long long* hist, double m) {
  uint64_t U = 0;
  for (int r = 0; r < kBins; ++r) U += (uint64_t)hist[r] << (32 - r);
  return hll_estimate(U, hist[0], m);
}

// Sum over the LPH lanes (16 or 64) that share a host; every lane gets it.
template <int LPH, class T>
__device__ __forceinline__ T row_sum(T v) {
#pragma unroll
  for (int d = 1; d < LPH; d <<= 1) v += __shfl_xor(v, d);
  return v;
}

// One wave's part of a register-gathering estimate: n <= 64 consecutive hosts,
// LPH lanes each, 64 / LPH at a time.  The hosts' registers (getPhyIdx of
// Alg. 3, gathers of Alg. 5) are read from their nibble copy, of which the
// first tab_n are also in LDS (tab, with TABLE); a nibble of 15 stands for 15
// and more and is read again from the byte array.  The harmonic sum is an
// exact integer: registers below 15 add 2^(32-r) = 2^18 2^(14-r), at most
// g 2^14 <= 2^30 in units of 2^18, to Us; the others add 2^(32-r) to Ux.  Each host's sums move to
// the lane of its place (U and V of host `lane`), so that what follows runs
// once for all of them, a lane per host.  PART: only registers of pool range
// `part` (the hash's bits from part_shift up) are gathered.  bytes: see gather_bytes.
template <int LPH, bool TABLE, bool PART>
__device__ __forceinline__ void gather_hosts(const uint32_t* __restrict__ hosts, uint32_t n, const uint32_t* s1,
                                             uint32_t g, uint32_t m, const uint8_t* __restrict__ reg,
                                             const uint8_t* __restrict__ reg4, const uint8_t* tab, uint32_t tab_n,
                                             uint32_t part, uint32_t part_shift, bool bytes, uint64_t& U,
                                             uint32_t& V) {
  constexpr int kRows = 64 / LPH;  // hosts at a time
  const int lane = threadIdx.x & 63, q = lane / LPH, ql = lane % LPH;
  const uint32_t kmix = mm3_key((uint32_t)lane < n ? hosts[lane] : 0u);
  U = 0;
  V = 0;
  for (uint32_t t = 0; t * kRows < n; ++t) {
    const uint32_t km = (uint32_t)__shfl((int)kmix, (int)(t * kRows) + q);
    uint32_t Us = 0, Vs = 0;
    unsigned long long Ux = 0;
    auto gathers = [&](auto guard, auto flight, auto from_bytes) __attribute__((always_inline)) {
      constexpr bool GUARD = decltype(guard)::value, BYTES = decltype(from_bytes)::value;
      constexpr int kFlight = decltype(flight)::value;  // gathers in flight per lane
      for (uint32_t i0 = (uint32_t)ql; i0 < g; i0 += LPH * kFlight) {
        uint32_t p[kFlight], nib[kFlight];
        bool mine[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
          const uint32_t i = i0 + (uint32_t)(LPH * u);
          const uint32_t h = mm3_seeded(km, s1[!GUARD || i < g ? i : 0u]);
          p[u] = reduce_m(h, m);
          if (PART) mine[u] = h >> part_shift == part;
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
          if (BYTES) nib[u] = TABLE ? (uint32_t)tab[p[u]] : (uint32_t)reg[p[u]];
          else if (TABLE) nib[u] = p[u] < tab_n ? (uint32_t)tab[p[u] >> 1] : (uint32_t)reg4[p[u] >> 1];
          else nib[u] = !PART || mine[u] ? (uint32_t)reg4[p[u] >> 1] : 0u;
        }
        if constexpr (BYTES) {
#pragma unroll
          for (int u = 0; u < kFlight; ++u) {
            const bool in = !GUARD || i0 + (uint32_t)(LPH * u) < g;
            Us += in && nib[u] < 15u ? 0x4000u >> nib[u] : 0u;
            Vs += in && nib[u] == 0u;
            Ux += in && nib[u] >= 15u ? 1ull << (32 - nib[u]) : 0ull;
          }
          continue;
        }
        bool wide = false;
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
          nib[u] = __builtin_amdgcn_ubfe(nib[u], (p[u] & 1u) << 2, 4);
          if ((GUARD && i0 + (uint32_t)(LPH * u) >= g) || (PART && !mine[u])) nib[u] = 16;  // adds nothing below
          Us += 0x4000u >> nib[u];
          Vs += nib[u] == 0u;
          wide |= nib[u] == 15u;
        }
        if (wide)
#pragma unroll
          for (int u = 0; u < kFlight; ++u)
            if (nib[u] == 15u) Ux += 1ull << (32 - reg[p[u]]);
      }
    };
    if (!PART && bytes) gathers(TrueType{}, Int<8>{}, TrueType{});
    else if (g % (LPH * 8) == 0) gathers(FalseType{}, Int<8>{}, FalseType{});
    else if (LPH == 16) gathers(TrueType{}, Int<8>{}, FalseType{});
    else gathers(TrueType{}, Int<4>{}, FalseType{});
    Us = row_sum<LPH>(Us);
    Vs = row_sum<LPH>(Vs);
    // lane l keeps host l: row l % kRows of step l / kRows
    const int from = (lane % kRows) * LPH;
    uint64_t u64 = (uint64_t)(uint32_t)__shfl((int)Us, from) << 18;
    if (__builtin_amdgcn_ballot_w64(Ux != 0ull)) u64 += __shfl(row_sum<LPH>(Ux), from);
    const uint32_t vs = (uint32_t)__shfl((int)Vs, from);
    if ((uint32_t)lane / kRows == t) U = u64, V = vs;
  }
}

// Sums of n <= 64 consecutive hosts' values by one wave, laid out as in
// gather_hosts: lane l < n returns host l's.  The values are the bytes val, or
// with NIB registers, read from their nibbles val4 where below 15.
template <int LPH, bool PART, bool NIB>
__device__ __forceinline__ uint32_t sum_hosts(const uint32_t* __restrict__ hosts, uint32_t n, const uint32_t* s1,
                                              uint32_t g, uint32_t m, const uint8_t* __restrict__ val,
                                              const uint8_t* __restrict__ val4, uint32_t part, uint32_t part_shift) {
  constexpr int kRows = 64 / LPH, kFlight = 8;
  const int lane = threadIdx.x & 63, q = lane / LPH, ql = lane % LPH;
  const uint32_t kmix = mm3_key((uint32_t)lane < n ? hosts[lane] : 0u);
  uint32_t sum = 0;
  for (uint32_t t = 0; t * kRows < n; ++t) {
    const uint32_t km = (uint32_t)__shfl((int)kmix, (int)(t * kRows) + q);
    uint32_t S = 0;
    for (uint32_t i0 = (uint32_t)ql; i0 < g; i0 += LPH * kFlight) {
      uint32_t p[kFlight], v[kFlight];
      bool mine[kFlight];
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const uint32_t i = i0 + (uint32_t)(LPH * u);
        const uint32_t h = mm3_seeded(km, s1[i < g ? i : 0u]);
        p[u] = reduce_m(h, m);
        mine[u] = i < g && (!PART || h >> part_shift == part);
      }
#pragma unroll
      for (int u = 0; u < kFlight; ++u) v[u] = mine[u] ? (uint32_t)(NIB ? val4[p[u] >> 1] : val[p[u]]) : 0u;
      bool wide = false;
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        if (NIB) v[u] = __builtin_amdgcn_ubfe(v[u], (p[u] & 1u) << 2, 4), wide |= v[u] == 15u;
        S += v[u];
      }
      if (NIB && wide)
#pragma unroll
        for (int u = 0; u < kFlight; ++u)
          if (v[u] == 15u) S += (uint32_t)val[p[u]] - 15u;
    }
    S = (uint32_t)__shfl((int)row_sum<LPH>(S), (lane % kRows) * LPH);  // lane l keeps host l
    if ((uint32_t)lane / kRows == t) sum = S;
  }
  return sum;
}

// Register histograms of 64 / LPH hosts by one wave, LPH lanes each (kmix: the
// key of this lane's host), added to this lane's host's row of 33 counts in LDS,
// which is zero before.  Each lane counts nibbles below 15 in registers: four bits a
// value over eight gathers, then bytes (a lane sees at most 128 registers), then
// the lanes' 16-bit sums, halving the values each lane keeps; registers of 15
// and more are read from the byte array and counted with LDS atomics (an LDS
// atomic per register kept whole waves on a few values), which take every register
// where many are (bytes: see gather_bytes).  PART as in
// gather_hosts.  g <= 128 LPH.
template <int LPH, bool PART>
__device__ __forceinline__ void hist_hosts(uint32_t kmix, const uint32_t* s1, uint32_t g, uint32_t m,
                                           const uint8_t* __restrict__ reg, const uint8_t* __restrict__ reg4,
                                           uint32_t part, uint32_t part_shift, bool bytes, uint32_t* row) {
  const uint32_t ql = threadIdx.x % LPH;
  uint64_t even = 0, odd = 0;  // byte j: count of value 2j, 2j + 1
  if (!PART && bytes) {
    constexpr int kFlight = 8;
    for (uint32_t i0 = ql; i0 < g; i0 += LPH * kFlight) {
      uint32_t r[kFlight];
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const uint32_t i = i0 + (uint32_t)(LPH * u);
        r[u] = i < g ? (uint32_t)reg[reduce_m(mm3_seeded(kmix, s1[i]), m)] : 255u;
      }
#pragma unroll
      for (int u = 0; u < kFlight; ++u)
        if (r[u] != 255u) atomicAdd(&row[r[u]], 1u);
    }
    return;
  }
  auto gathers = [&](auto flight) __attribute__((always_inline)) {
    constexpr int kFlight = decltype(flight)::value;  // gathers in flight per lane
    for (uint32_t i0 = ql; i0 < g; i0 += LPH * kFlight) {
      uint32_t p[kFlight], nib[kFlight];
      bool mine[kFlight];
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const uint32_t i = i0 + (uint32_t)(LPH * u);
        const uint32_t h = mm3_seeded(kmix, s1[i < g ? i : 0u]);
        p[u] = reduce_m(h, m);
        mine[u] = i < g && (!PART || h >> part_shift == part);
      }
#pragma unroll
      for (int u = 0; u < kFlight; ++u) nib[u] = mine[u] ? (uint32_t)reg4[p[u] >> 1] : 0u;
      uint64_t acc = 0;
      bool wide = false;
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        nib[u] = __builtin_amdgcn_ubfe(nib[u], (p[u] & 1u) << 2, 4);
        acc += (uint64_t)mine[u] << (4 * nib[u]);
        wide |= mine[u] && nib[u] == 15u;
      }
      even += acc & 0x0F0F0F0F0F0F0F0Full;
      odd += acc >> 4 & 0x0F0F0F0F0F0F0F0Full;
      if (wide)
#pragma unroll
        for (int u = 0; u < kFlight; ++u)
          if (mine[u] && nib[u] == 15u) atomicAdd(&row[reg[p[u]]], 1u);
    }
  };
  if (!PART && g <= LPH * 4) gathers(Int<4>{});  // PART with both: 36 registers a lane for 32, 677 us for 630
  else gathers(Int<8>{});
  constexpr uint64_t kLow = 0x00FF00FF00FF00FFull;
  const uint64_t v[4] = {even & kLow, even >> 8 & kLow, odd & kLow, odd >> 8 & kLow};
  uint32_t w[8];  // two values a word: 0 4 | 8 12 | 2 6 | 10 14 | 1 5 | 9 13 | 3 7 | 11 15
#pragma unroll
  for (int q = 0; q < 4; ++q) w[2 * q] = (uint32_t)v[q], w[2 * q + 1] = (uint32_t)(v[q] >> 32);
#pragma unroll
  for (int d = 1, n = 4; d < 8; d <<= 1, n >>= 1) {  // lanes with bit d keep the upper half
    const bool up = ql & d;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q >= n) break;
      const uint32_t got = (uint32_t)__shfl_xor((int)(up ? w[q] : w[q + n]), d);
      w[q] = (up ? w[q + n] : w[q]) + got;
    }
  }
#pragma unroll
  for (int d = 8; d < LPH; d <<= 1) w[0] += (uint32_t)__shfl_xor((int)w[0], d);
  if (ql < 8) {
    const uint32_t value = (ql & 1u) + (ql & 2u) + 2u * (ql & 4u);
    atomicAdd(&row[value], w[0] & 0xFFFFu);
    if (value != 11u) atomicAdd(&row[value + 4u], w[0] >> 16);
  }
}

// The estimates of n <= 64 consecutive hosts by one wave.
template <int LPH, bool TABLE>
__device__ __forceinline__ void estimate_hosts(const uint32_t* __restrict__ hosts, uint32_t n, const uint32_t* s1,
                                               uint32_t g, uint32_t m, const uint8_t* __restrict__ reg,
                                               const uint8_t* __restrict__ reg4, const uint8_t* tab, uint32_t tab_n,
                                               bool bytes, double Em, float* __restrict__ out) {
  uint64_t U;
  uint32_t V;
  gather_hosts<LPH, TABLE, false>(hosts, n, s1, g, m, reg, reg4, tab, tab_n, 0u, 0u, bytes, U, V);
  const uint32_t lane = threadIdx.x & 63;
  if (lane < n) {
    const double Es = hll_estimate(U, V, (double)g);
    const double e = noise_removed(Es, Em, (double)m, (double)g);
    out[lane] = (float)(e > 0.0 ? e : 0.0);
  }
}

}  // namespace vbdr
