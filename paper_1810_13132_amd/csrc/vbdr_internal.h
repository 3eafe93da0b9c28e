// Host-side internals shared by the translation units of libvbdr.so.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "vbdr.h"
#include "vbdr_device.h"

constexpr uint64_t kPad = 4096;             // BDR padding granule of a plane
constexpr uint32_t kStageMaxG = 8192;       // s1 staged in LDS up to 32 KiB
constexpr uint32_t kCusPerXcd = 32;         // gfx950: 8 XCDs x 32 CUs
constexpr uint64_t kPartMinM = 1ull << 22;  // pools whose registers outgrow one XCD's L2
constexpr uint32_t kPartChunk = 1u << 20;   // hosts per partitioned-estimate pass
// Histograms counted in registers up to this many ranges, with LDS atomics above, where most lanes of a gather idle
// (g = 2048: 2 ranges 2.4e11 gathers a second and 2.0e11, 8 ranges 1.2e11 and 1.6e11; 4 ranges, 100,000 hosts on 1.5
// 2^24 BDRs: 851 us and 843).
constexpr uint32_t kHistRowsParts = 2;
constexpr uint32_t kLearnChunk = 1u << 15;  // hosts per histogram pass whose histograms come in sk->parts ranges
constexpr uint64_t kBinMaxM = 1ull << 27;   // binned scan records pack (pidx << 5) | (LBP1 - 1)
constexpr uint32_t kBinChunk = 1u << 24;    // pairs per binned-scan pass (records stay cache resident)
constexpr uint32_t kBinCap = kBinChunk / 8 + kBinChunk / 32 + 65536;  // records per bin per pass
// BDRs per tile (one advance workgroup of 1024 threads): 2^12 .. 2^15
constexpr uint32_t kMinTileShift = 12, kMaxTileShift = 15;
constexpr uint64_t kDeferMinM = 1ull << 16;       // pools that keep record runs (fast layout, batch members)
constexpr uint64_t kDeferMinSmall = 1ull << 19;   // the same, small layout
constexpr uint32_t kDeferSlots = 2;         // record slots per BDR per slice before the direct fallback, at least
constexpr uint64_t kDeferBudget = 1ull << 27;  // record slots of a sketch where its pool needs fewer per BDR
constexpr uint32_t kDeferSlotsMax = 16;
constexpr uint64_t kDeferLeast = 1ull << 22;   // record slots of a sketch, at least
// Pairs of a scan up to which pools below 2^22 BDRs are updated directly.
constexpr uint64_t kDirectSmall = 1ull << 20, kDirectFast = 1ull << 16;
constexpr uint64_t kOverfullM = 1ull << 20;  // fast pools below scan directly where a slice is far past the runs

// Which estimate gathers how (g <= kStageMaxG, no extra outputs), each line
// with both sides measured at g = 512 (gathers a second, large host lists):
//   up to 2^21 BDRs directly, nibbles in LDS (2^18: 1.28e12, 2^20: 4.0e11, 2^21:
//     3.1e11; all gathers from L2: 3.0e11, 2.7e11, 2.6e11);
//   up to 2^23 directly, the nibbles in every XCD's L2 (2.6e11; ranges on
//     8 XCDs: 1.7e11);
//   above in 2, 4 or 8 ranges by XCD (2^24: 2.6e11, 2^26: 2.0e11; 8 ranges:
//     1.7e11, directly: 1.2e11, 0.65e11), directly below 2^19 to 2^20 gathers;
//   from 2^24 BDRs and enough gathers the LDS-tiled passes (2.9e11; 16384
//     hosts at 2^24: tiled 58 us, ranges 41; 65536: 131 and 139; at 2^26 65
//     and 59, 139 and 199).
constexpr uint64_t kTableMaxM = 1ull << 21;       // pools whose direct estimate may keep registers in LDS
constexpr uint64_t kTableMinUse = 6;              // gathers per register of that table, at least (2^18 BDRs: a step of 2^20
                                                  // pairs, 4096 hosts, g = 256 28.6 us with the table, 27.1 without)
constexpr uint64_t kRangeBytes = 4ull << 20;      // nibbles of a range: an XCD's L2
// Gathers of an estimate below which one range will do: of two; of more for g from 1024 and below, where a host's
// chain of gathers is short (1.05 2^23 BDRs, g = 512: 800 hosts 6 us directly, 8 in ranges, 1500 8 and 9; 1.99 2^23: 1000
// 9 and 9; 0.95 2^25, g = 2048: 100 hosts 9 and 10, 200 11 and 11, 500 18 and 13; 1.1 2^25, g = 512: 1000 11 and 12, 1500
// 14 and 13).
constexpr uint64_t kPartMinGathers = 1ull << 20, kPartMinLongG = 3ull << 17, kPartMinShortG = 5ull << 17;
constexpr uint64_t kTileMinGathers = 3ull << 23, kTileMinGathers8 = 10ull << 20;  // from which tiles pay (8 ranges)

// Shares 1 / k of registers of 15 and more from which gathers read bytes (gather_bytes): from L2, from LDS, and for
// histograms, which then count with LDS atomics alone.  200,000 hosts, g = 1024, 40,000 BDRs, most registers 15 and
// more: LogLog 520 us by nibbles, 270 by bytes, learned 516 and 290, plain (LDS) 270 and 240; g = 256, 131,072 BDRs, one
// in four: learned 212 and 165.
constexpr uint32_t kWideL2 = 16, kWideTab = 4, kWideHist = 32;

struct vbdr_sketch {
  int device;
  int n_cu;
  uint64_t m;
  uint32_t g, b, L, k;
  int layout;
  uint32_t A0, A1;
  uint64_t t;
  uint64_t mstride, wstride;
  uint8_t* dr;                    // byte DRs, plane-major (fast and small layouts)
  uint32_t* bits;                 // packed layout: bit-plane (r-1)*z + b holds bit b of DR r, 32 BDRs a word
  uint32_t z, Lc;                 // packed layout: bits per DR, recorders per BDR (else 8 and L)
  uint32_t* seen;
  uint8_t* reg;
  unsigned long long* hist;       // pool statistics (kStatWords words)
  uint32_t* s1;
  uint8_t* reg4;               // registers as nibbles, min(reg, 15); 15 = read reg
  int parts;                   // XCD partitions of the estimate (1 = direct gather)
  unsigned long long* part_u;  // [parts][kPartChunk] partial harmonic sums
  uint32_t* part_v;            // [parts][kPartChunk] partial zero counts
  uint32_t* hist_ws;           // per-host (partial) histograms of a pass, parts * kLearnChunk * 33 counts
  float* est_ws;               // [kLearnChunk] plain estimates of a histogram pass
  uint32_t* bins;              // [parts][kBinCap] binned scan records (large pools)
  uint32_t* bin_fill;          // [parts] records written per bin
  uint32_t* est_slots;         // [8][est_hc][est_cap] binned-estimate pidx runs
  uint32_t* est_cnt;           // [8][est_hc] run lengths
  unsigned long long* ovf_u;   // [est_hc] overflow partial sums
  uint32_t* ovf_v;             // [est_hc]
  uint32_t est_cap, est_hc;
  bool bin_ok, est_ok;            // the binned scan / estimate workspaces may be allocated (on request)
  bool tl_always;                 // est_binned = 3 was asked for: also for few hosts
  bool tl_ok;                     // the LDS-tiled estimate fits this pool (workspaces on request)
  uint32_t tl_shift, tl_nt, tl_B, tl_cap;  // tile = 2^tl_shift registers; tiles; hosts per block; records per run
  uint32_t tl_capb;               // entries per LDS bucket of a (chunk, tile) in the first pass
  uint32_t* tl_rec;               // [B / 2048][nt][cap] records of a block
  uint32_t* tl_fill;              // [B / 2048][nt] run lengths
  uint32_t* tl_part;              // [nt][B] per-tile sums of a block's hosts, packed (exact or moved to tl_ovf)
  unsigned long long* tl_ovf;     // [B] sums of run overflows
  uint2* tl_wide;                 // [nt][tl_wcap] records of registers >= 15 found by pass 2, then [nt] counts
  uint32_t tl_wcap;
  uint32_t tl_Balloc;             // hosts per block the record, run-length and sum buffers hold (<= tl_B)
  uint32_t* def_rec;              // [def_tiles][def_cap] deferred scan records (pidx << 5 | LBP1-1)
  uint32_t* sat;                  // deferred scans: [wstride] bit r-1 = DR[r] of all 32 BDRs saturated (255, or 2^z - 1)
  unsigned long long* def_fill;   // [def_tiles + 1] records per tile; the last word flags direct updates
  uint32_t def_tiles, def_cap;
  uint64_t open_records;          // pairs that scans of the open slice put through the runs (chooses routes only)
  uint32_t tshift, tiles;         // the advance's tiles: 2^tshift BDRs, tiles of them (def_tiles of them have record runs)
  bool lean;                      // no optional workspaces (sketches owned by a batch)
  uint8_t* preg;                  // small layout, on request: PCSA run of each BDR, last closed window
  unsigned long long* psum;       // sum of preg over the pool, then the running sum of an advance in flight
  bool pcsa_valid;                // preg was written by an advance since it was enabled
  uint64_t bytes;                 // device bytes held: the window state plus every workspace
  uint64_t state_only;            // of which the window state: DRs, bsLBP1, registers, masks, seeds, PCSA runs
  vbdr_tuning tune;
};

// vbdr_sketch_create_layout without the optional large-pool workspaces;
// with defer, pools that scan through records keep their runs.
int vbdr_sketch_create_lean(uint64_t m, uint32_t g, uint32_t k, uint64_t hash_seed, int layout, bool defer,
                            vbdr_sketch** out);

// What the advance of one sketch works on (a kernel argument, or an entry of
// a batch's table).  Without record runs (recs, fill and sat NULL) the bsLBP1
// planes hold the whole slice.
struct AdvSketch {
  uint8_t* dr;
  uint32_t* seen;  // fast layout, else NULL
  uint8_t* reg;
  uint8_t* reg4;
  uint8_t* preg;   // PCSA runs, or NULL
  unsigned long long* psum;
  unsigned long long* stats;
  const uint32_t* recs;
  unsigned long long* fill;
  uint32_t* sat;   // tiles of 2^14 BDRs and more, else NULL
  uint64_t mstride, wstride, m;
  uint32_t L, thr, cap, tiles, tshift, layout;
};

// A batch member as the batch's scan and advance kernels read it from device
// memory.  pairs, n_pairs and scan_item0 change every step; the rest is the
// sketch's.  Members without record runs have no scan items here.
constexpr uint32_t kMaxDeferMembers = 256;
struct DeferItem {
  AdvSketch adv;
  const uint32_t* pairs;
  uint64_t n_pairs;
  const uint32_t* s1;
  uint32_t* recs;
  uint32_t b, A1;
  uint32_t scan_item0;  // first scan item (chunk) of the member this step
  uint32_t adv_item0;   // first advance item (tile) of the member
};
struct DeferHdr {
  uint32_t scan_total;  // scan items of the step
  uint32_t pad[3];
};

// The sketch's fields of its DeferItem (pairs, n_pairs and the item offsets zero).
void vbdr_defer_member(const vbdr_sketch* sk, DeferItem* d);
constexpr uint32_t kDeferChunk = 1u << 15;  // pairs per scan item of a member with record runs
// Phase 0: the scans of members with record runs (grid workgroups over
// hdr->scan_total items; max_tiles of them at most, 0: none; max_g: their
// largest g where their seeds fit in LDS, else 0); phase 1: the
// advances of all members (adv_total tiles, adv_lds bytes of bit words; big:
// some member's tiles are of 2^kMaxTileShift BDRs).
int vbdr_launch_batch_defer(const DeferItem* items_dev, const DeferHdr* hdr_dev, uint32_t S, uint32_t max_tiles,
                            uint32_t max_g, uint32_t adv_lds, uint32_t adv_total, bool big, uint32_t grid, int phase,
                            hipStream_t st);
// LDS bytes of the scans, static ones included.
size_t vbdr_batch_scan_lds(uint32_t max_tiles, uint32_t max_g);
// LDS bytes of a sketch's advance.
uint32_t vbdr_adv_lds(const vbdr_sketch* sk);

constexpr uint64_t kPackedMaxM = 1ull << 26;  // packed pools: records' tiles must fit the deferred scan's LDS

// Records the calling thread's error message and returns code.
int vbdr_fail(int code, const char* fmt, ...);

// hipMalloc for every device allocation of the library, so that
// vbdr_test_fail_alloc can make a chosen one fail.
hipError_t vbdr_malloc_bytes(void** p, size_t bytes);
template <class T>
inline hipError_t vbdr_malloc(T** p, size_t bytes) {
  return vbdr_malloc_bytes(reinterpret_cast<void**>(p), bytes);
}

#define VBDR_HIP(call)                                                                         \
  do {                                                                                         \
    hipError_t e_ = (call);                                                                    \
    if (e_ != hipSuccess) return vbdr_fail(VBDR_EHIP, "%s: %s", #call, hipGetErrorString(e_)); \
  } while (0)

#define VBDR_LAUNCHED(name)                                                                         \
  do {                                                                                              \
    hipError_t e_ = hipGetLastError();                                                              \
    if (e_ != hipSuccess) return vbdr_fail(VBDR_EHIP, "launch of %s: %s", name, hipGetErrorString(e_)); \
  } while (0)

// VBDR_EINVAL unless the sketch's device is current.
int vbdr_check_device(const vbdr_sketch* sk);

// Register histograms of nh <= vbdr_hist_chunk(sk) hosts into sk->hist_ws: one
// partial histogram per pool range, [x][vbdr_hist_chunk(sk)][33], to be summed
// over the vbdr_gather_parts(sk) ranges x.
uint32_t vbdr_gather_parts(const vbdr_sketch* sk);
uint32_t vbdr_hist_chunk(const vbdr_sketch* sk);
int vbdr_hist_pass(vbdr_sketch* sk, const uint32_t* hosts_dev, uint32_t nh, hipStream_t st);
