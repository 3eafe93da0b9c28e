// Many independent sketches (uneven streams, pools, windows, g, layouts)
// advanced per slice by a few kernels over all of them: members with record
// runs (pools of 2^16..2^26 BDRs) scan in sorted chunks and all members
// advance tile by tile, as a single sketch does (both in vbdr.hip); the other
// members' scans and all estimates are persistent work-queue kernels that
// pull (sketch, tile) items from device counters.  Each sketch's per-slice inputs live in
// a device descriptor table refreshed by one host-to-device copy per step, so
// the kernel sequence is captured once into a hipGraph and replayed.  Every
// block leaves its loop when the queue is drained, so a launch always
// completes.
#include <hip/hip_runtime.h>

#include <cstring>
#include <new>
#include <vector>

#include "vbdr_internal.h"

using namespace vbdr;

namespace {

constexpr uint32_t kMaxBatch = 256;
constexpr int kBBlock = 256;

struct BatchDesc {
  uint8_t* dr;
  uint32_t* seen;
  uint8_t* reg;
  uint8_t* reg4;
  unsigned long long* hist;
  const uint32_t* s1;
  uint64_t mstride, wstride;
  uint32_t m, g, b, L, k, layout, A1, test;
  const uint32_t* pairs;  // per step
  uint64_t n_pairs;
  const uint32_t* hosts;
  uint64_t n_hosts;
  float* out;
  uint32_t scan_item0;
  // estimate: what part of the kernel takes the member (EstPart), and its cost there
  uint32_t est_part;
  uint32_t each;               // cost of a host
  uint64_t cost0;              // cost of the members before in that part
  uint32_t parts, part_shift;  // L2 members: pool ranges, the hash bits that choose one
  uint32_t part_off;           // ... first host in the partial sums (ranges > 1)
  uint32_t tab_n;              // LDS members: registers in LDS
};

// Spread: gathers from L2, over all workgroups; L2, LDS: stretches cut by cost.
enum EstPart : uint32_t { kEstNone = 0, kEstSpread = 1, kEstL2 = 2, kEstLdsPart = 3 };

struct BatchHdr {
  uint64_t cost[2];     // cost of all L2 members on one XCD, of all LDS members
  uint32_t scan_total;  // items of the scan
  uint32_t counter;     // scan items taken; reset to 0 by every step's table upload
  uint32_t pad[2];
};

__device__ __forceinline__ uint32_t find_sketch(const uint32_t* starts, uint32_t S, uint32_t item) {
  uint32_t lo = 0, hi = S - 1;  // last s with starts[s] <= item
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (starts[mid] <= item) lo = mid;
    else hi = mid - 1;
  }
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);  // the whole workgroup's
}

// Next work item of a queue, shared by the whole block.
__device__ __forceinline__ uint32_t next_item(uint32_t* counter, uint32_t* sh) {
  __syncthreads();
  if (threadIdx.x == 0) *sh = atomicAdd(counter, 1u);
  __syncthreads();
  return *sh;
}

__global__ __launch_bounds__(kBBlock) void k_batch_scan(const BatchDesc* __restrict__ d, BatchHdr* __restrict__ hdr,
                                                        uint32_t S, uint32_t tile) {
  __shared__ uint32_t starts[kMaxBatch];
  __shared__ uint32_t cur;
  for (uint32_t s = threadIdx.x; s < S; s += kBBlock) starts[s] = d[s].scan_item0;
  const uint32_t total = hdr->scan_total;
  for (;;) {
    const uint32_t item = next_item(&hdr->counter, &cur);
    if (item >= total) break;
    const uint32_t s = find_sketch(starts, S, item);
    const BatchDesc& D = d[s];
    const uint64_t lo = (uint64_t)(item - starts[s]) * tile;
    const uint64_t hi = lo + tile < D.n_pairs ? lo + tile : D.n_pairs;
    const u32x2* pairs = reinterpret_cast<const u32x2*>(D.pairs);
    constexpr int kPer = 8;  // pairs per thread at a time: their loads and state reads overlap
    for (uint64_t i0 = lo + threadIdx.x; i0 < hi; i0 += (uint64_t)kPer * kBBlock) {
      u32x2 p[kPer];
      bool ok[kPer];
#pragma unroll
      for (int v = 0; v < kPer; ++v) {
        const uint64_t i = i0 + (uint64_t)v * kBBlock;
        ok[v] = i < hi;
        p[v] = ok[v] ? __builtin_nontemporal_load(pairs + i) : u32x2{0u, 0u};
      }
      if (D.layout == VBDR_LAYOUT_FAST) {
        if (D.test) scan_pairs<true, true, kPer>(p, ok, D.s1, D.b, D.A1, D.m, D.dr, D.mstride, D.seen, D.wstride);
        else scan_pairs<true, false, kPer>(p, ok, D.s1, D.b, D.A1, D.m, D.dr, D.mstride, D.seen, D.wstride);
      } else {
        if (D.test) scan_pairs<false, true, kPer>(p, ok, D.s1, D.b, D.A1, D.m, D.dr, D.mstride, D.seen, D.wstride);
        else scan_pairs<false, false, kPer>(p, ok, D.s1, D.b, D.A1, D.m, D.dr, D.mstride, D.seen, D.wstride);
      }
    }
  }
}

// Estimates of all members by one workgroup per CU.  Work is handed out by
// position alone (a counter for items of a few hosts served one wave every 20 ns:
// 858 us).  First the members whose gathers go to L2: an XCD takes a range of
// the pool where its nibbles outgrow a part of the L2 (8 / parts XCDs share a
// range, each takes its share of the hosts; k_batch_estimate_final adds the
// ranges' sums), many hosts are spread over all workgroups, one member after
// the other, so that they share the L2, few are cut by cost.  Then the members
// with (part of) their registers in LDS: a workgroup takes one stretch of all
// their hosts, so that it loads one or two members' tables.
// 1.29e8 gathers of 32 members: 837 us with every gather from L2, one host a
// wave; 392 us now.
constexpr int kEBlock = 1024, kEWaves = kEBlock / 64;
constexpr uint32_t kEstLds = 152u << 10;     // seeds and table
constexpr uint64_t kEstTableM = 1ull << 20;  // pools up to this keep registers in LDS
constexpr uint64_t kEstRange = 2ull << 20;   // nibbles of a range: half an L2, which a few members share
constexpr uint32_t kPartEntries = 1u << 19;  // (range, host) sums of a step; members past that gather directly
__global__ __launch_bounds__(kEBlock) void k_batch_estimate(const BatchDesc* __restrict__ d,
                                                            const BatchHdr* __restrict__ hdr, uint32_t S,
                                                            unsigned long long* __restrict__ part_u,
                                                            uint32_t* __restrict__ part_v) {
  extern __shared__ uint32_t lds[];
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t xcd = blockIdx.x & 7u;  // workgroups are dispatched round-robin over the 8 XCDs
  const uint32_t mine = blockIdx.x >> 3, per_xcd = gridDim.x >> 3;
  auto work = [&](const BatchDesc& D, uint64_t lo, uint64_t hi, auto in_lds) __attribute__((always_inline)) {
    constexpr bool TABLE = decltype(in_lds)::value;
    const uint32_t g = D.g;
    const bool staged = g <= kStageMaxG;
    uint32_t* tab = lds + g;  // 16-byte aligned: g >= 4
    __syncthreads();          // nobody reads the member's before any more
    if (staged)
      for (uint32_t i = threadIdx.x; i < g; i += kEBlock) lds[i] = D.s1[i];
    if (TABLE) {
      const u32x4* src = reinterpret_cast<const u32x4*>(D.reg4);
      for (uint32_t q = threadIdx.x; q < D.tab_n / 32; q += kEBlock) reinterpret_cast<u32x4*>(tab)[q] = src[q];
    }
    __syncthreads();
    const uint64_t n = hi - lo;
    uint64_t per = ((n + kEWaves - 1) / kEWaves + 3) / 4 * 4;
    per = per > 64 ? 64 : per;
    for (uint64_t h = wave * per; h < n; h += kEWaves * per) {
      const uint32_t c = n - h < per ? (uint32_t)(n - h) : (uint32_t)per;
      const uint32_t* hosts = D.hosts + lo + h;
      float* out = D.out + lo + h;
      if (TABLE) {
        estimate_hosts<16, true>(hosts, c, lds, g, D.m, D.reg, D.reg4, reinterpret_cast<const uint8_t*>(tab), D.tab_n,
                                 false, stat_em(D.hist), out);
      } else if (D.parts > 1) {
        const uint32_t part = xcd % D.parts;
        uint64_t U;
        uint32_t V;
        gather_hosts<16, false, true>(hosts, c, lds, g, D.m, D.reg, D.reg4, nullptr, 0u, part, D.part_shift, false, U, V);
        if (lane < c) {
          const uint64_t at = D.part_off + part * D.n_hosts + lo + h + lane;
          part_u[at] = U;
          part_v[at] = V;
        }
      } else if (staged) {
        estimate_hosts<16, false>(hosts, c, lds, g, D.m, D.reg, D.reg4, nullptr, 0u, false, stat_em(D.hist), out);
      } else {
        estimate_hosts<16, false>(hosts, c, D.s1, g, D.m, D.reg, D.reg4, nullptr, 0u, false, stat_em(D.hist), out);
      }
    }
  };
  for (uint32_t s = 0; s < S; ++s) {
    const BatchDesc& D = d[s];
    if (D.est_part != kEstSpread) continue;
    const uint64_t shares = 8u / D.parts * per_xcd, share = xcd / D.parts * per_xcd + mine;
    const uint64_t lo = D.n_hosts * share / shares, hi = D.n_hosts * (share + 1) / shares;
    if (lo < hi) work(D, lo, hi, FalseType{});
  }
  // the hosts of a member whose cost starts in [from, to), of hosts first .. first + n
  auto stretch = [&](const BatchDesc& D, uint64_t from, uint64_t to, uint64_t first, uint64_t n, auto in_lds)
                     __attribute__((always_inline)) {
    const uint64_t end = D.cost0 + D.each * n;
    if (end <= from || D.cost0 >= to) return;
    const uint64_t lo = from <= D.cost0 ? 0 : (from - D.cost0 + D.each - 1) / D.each;
    const uint64_t hi = to >= end ? n : (to - D.cost0 + D.each - 1) / D.each;
    if (lo < hi) work(D, first + lo, first + hi, in_lds);
  };
  for (uint32_t s = 0; s < S; ++s) {
    const BatchDesc& D = d[s];
    if (D.est_part != kEstL2) continue;
    const uint64_t shares = 8u / D.parts, share = xcd / D.parts;  // this XCD's hosts
    const uint64_t first = D.n_hosts * share / shares, past = D.n_hosts * (share + 1) / shares;
    stretch(D, hdr->cost[0] * mine / per_xcd, hdr->cost[0] * (mine + 1) / per_xcd, first, past - first, FalseType{});
  }
  for (uint32_t s = 0; s < S; ++s) {
    const BatchDesc& D = d[s];
    if (D.est_part != kEstLdsPart) continue;
    stretch(D, hdr->cost[1] * blockIdx.x / gridDim.x, hdr->cost[1] * (blockIdx.x + 1) / gridDim.x, 0, D.n_hosts,
            TrueType{});
  }
}

// The estimates of members gathered in ranges, from their ranges' sums.
__global__ __launch_bounds__(256) void k_batch_estimate_final(const BatchDesc* __restrict__ d, uint32_t S,
                                                              const unsigned long long* __restrict__ part_u,
                                                              const uint32_t* __restrict__ part_v) {
  for (uint32_t s = blockIdx.y; s < S; s += gridDim.y) {
    const BatchDesc& D = d[s];
    if (D.parts < 2) continue;  // also members without hosts
    for (uint64_t h = blockIdx.x * 256 + threadIdx.x; h < D.n_hosts; h += gridDim.x * 256) {
      uint64_t U = 0, V = 0;
      for (uint32_t x = 0; x < D.parts; ++x) {
        U += part_u[D.part_off + x * D.n_hosts + h];
        V += part_v[D.part_off + x * D.n_hosts + h];
      }
      const double Es = hll_estimate(U, V, (double)D.g);
      const double e = noise_removed(Es, stat_em(D.hist), (double)D.m, (double)D.g);
      D.out[h] = (float)(e > 0.0 ? e : 0.0);
    }
  }
}

}  // namespace

struct vbdr_batch {
  int device;
  int n_cu;
  uint32_t S;
  std::vector<vbdr_sketch*> sk;
  BatchDesc* desc_dev;
  BatchHdr* hdr_dev;
  uint8_t* staging[2];  // pinned: descriptors then header
  hipEvent_t staged[2];
  int next;
  hipStream_t st;       // batch-owned stream (graphs cannot capture the null stream)
  hipEvent_t ev_in, ev_out;
  hipGraph_t graph;
  hipGraphExec_t exec;
  vbdr_batch_tuning tune;
  uint32_t runs_max_tiles;     // most tiles of a member with record runs; 0: none has any
  uint32_t runs_max_g;         // largest g of these members if their seeds fit the scan's LDS, else 0
  uint32_t adv_lds, adv_tiles; // the advance's LDS bytes (largest member) and tiles (all members)
  bool direct, big;            // some member scans without record runs; has tiles of 2^kMaxTileShift BDRs
  // sums of members whose gathers are partitioned (NULL: there is none), [kPartEntries]
  unsigned long long* part_u;
  uint32_t* part_v;
  // learned estimators by member (NULL: plain), owned by the caller
  std::vector<const vbdr_mlp*> mlp;
};

namespace {

// Device table: [S] BatchDesc, BatchHdr, [S] DeferItem, DeferHdr.
size_t table_bytes(uint32_t S) {
  return sizeof(BatchDesc) * S + sizeof(BatchHdr) + sizeof(DeferItem) * S + sizeof(DeferHdr);
}
DeferItem* defer_items(uint8_t* table, uint32_t S) {
  return reinterpret_cast<DeferItem*>(table + sizeof(BatchDesc) * S + sizeof(BatchHdr));
}
DeferHdr* defer_hdr(uint8_t* table, uint32_t S) {
  return reinterpret_cast<DeferHdr*>(table + sizeof(BatchDesc) * S + sizeof(BatchHdr) + sizeof(DeferItem) * S);
}

// Ranges of a member's gathers.
uint32_t member_parts(const vbdr_sketch* k) {
  uint32_t p = 1;
  while (p < 8u && (k->mstride / 2) / p > kEstRange) p *= 2;
  return k->g > kStageMaxG || k->n_cu < (int)(8 * kCusPerXcd) ? 1u : p;
}

// Where a member is estimated.  A host costs its gathers, weighted by their
// rate: registers in LDS (up to kEstTableM BDRs) 4 where all are (1.28e12 a
// second), 6 at 2^19 (8.2e11), 13 at 2^20 (4.0e11); from L2 in p ranges 1 / p
// and the hashes.  Members with est_tile / 4 hosts and more for every workgroup are
// spread over all of them (32 members: 392 us with 16 hosts, 442 with 64, 412
// with 2).  part_used: (range, host) sums taken so far.
void estimate_plan(const vbdr_batch* bt, const vbdr_sketch* k, uint64_t n_plain, uint32_t* part_used, uint64_t cost[2],
                   BatchDesc* D) {
  D->est_part = kEstNone, D->each = 0, D->cost0 = 0;
  D->parts = 1, D->part_shift = D->part_off = D->tab_n = 0;
  if (n_plain == 0) return;
  if (k->m <= kEstTableM && k->g >= 4 && k->g <= kStageMaxG) {
    const uint64_t most = (kEstLds - k->g * 4u) * 2ull / 32 * 32;
    D->tab_n = (uint32_t)(most < k->mstride ? most : k->mstride);
    D->est_part = kEstLdsPart;
    D->each = k->g * (most >= k->m ? 4u : k->m <= (1ull << 19) ? 6u : 13u);
    D->cost0 = cost[1];
    cost[1] += n_plain * D->each;
    return;
  }
  const uint32_t parts = bt->part_u ? member_parts(k) : 1u;
  if (parts > 1 && (uint64_t)*part_used + n_plain * parts <= kPartEntries) {
    D->parts = parts, D->part_shift = 32u - (parts == 8 ? 3u : parts == 4 ? 2u : 1u), D->part_off = *part_used;
    *part_used += (uint32_t)n_plain * parts;
  }
  const uint64_t shares = 8u / D->parts, hosts = (n_plain + shares - 1) / shares;  // of one XCD
  if (hosts >= (uint64_t)bt->tune.est_tile * (uint32_t)(bt->n_cu / 8) / 4) {
    D->est_part = kEstSpread;
    return;
  }
  D->est_part = kEstL2;
  D->each = k->g * (16u / D->parts + 4u);
  D->cost0 = cost[0];
  cost[0] += hosts * D->each;
}

int launch_step_kernels(vbdr_batch* bt) {
  if (bt->direct) {
    const uint32_t grid = (uint32_t)bt->n_cu * bt->tune.blocks_per_cu;
    hipLaunchKernelGGL(k_batch_scan, dim3(grid), dim3(kBBlock), 0, bt->st, bt->desc_dev, bt->hdr_dev, bt->S,
                       bt->tune.scan_tile);
    VBDR_LAUNCHED("k_batch_scan");
  }
  uint8_t* table = reinterpret_cast<uint8_t*>(bt->desc_dev);
  DeferItem* ditems = defer_items(table, bt->S);
  DeferHdr* dhdr = defer_hdr(table, bt->S);
  for (int phase = 0; phase < 2; ++phase)
    if (int rc = vbdr_launch_batch_defer(ditems, dhdr, bt->S, bt->runs_max_tiles, bt->runs_max_g, bt->adv_lds, bt->adv_tiles, bt->big,
                                         (uint32_t)bt->n_cu, phase, bt->st))
      return rc;
  hipLaunchKernelGGL(k_batch_estimate, dim3((uint32_t)bt->n_cu < 8 ? 8 : (uint32_t)bt->n_cu / 8 * 8), dim3(kEBlock), kEstLds, bt->st, bt->desc_dev,
                     bt->hdr_dev, bt->S, bt->part_u, bt->part_v);
  VBDR_LAUNCHED("k_batch_estimate");
  if (bt->part_u) {
    hipLaunchKernelGGL(k_batch_estimate_final, dim3(64, bt->S), dim3(256), 0, bt->st, bt->desc_dev, bt->S, bt->part_u,
                       bt->part_v);
    VBDR_LAUNCHED("k_batch_estimate_final");
  }
  return VBDR_OK;
}

void drop_graph(vbdr_batch* bt) {
  if (bt->exec) (void)hipGraphExecDestroy(bt->exec);
  if (bt->graph) (void)hipGraphDestroy(bt->graph);
  bt->exec = nullptr;
  bt->graph = nullptr;
}

}  // namespace

extern "C" {

int vbdr_batch_create(uint32_t n_sketches, const vbdr_batch_params* params, vbdr_batch** out) {
  if (!out || !params) return vbdr_fail(VBDR_EINVAL, "NULL argument");
  *out = nullptr;
  if (n_sketches < 1 || n_sketches > kMaxBatch) return vbdr_fail(VBDR_EINVAL, "1..%u sketches per batch", kMaxBatch);
  vbdr_batch* bt = new (std::nothrow) vbdr_batch();
  if (!bt) return vbdr_fail(VBDR_ENOMEM, "host allocation failed");
  bt->S = n_sketches;
  bt->tune.scan_tile = 8192;
  bt->tune.est_tile = 64;
  bt->tune.blocks_per_cu = 8;
  bt->tune.use_graph = 1;
  int rc = VBDR_OK;
  uint64_t total_tiles = 0;
  do {
    if (hipGetDevice(&bt->device) != hipSuccess ||
        hipDeviceGetAttribute(&bt->n_cu, hipDeviceAttributeMultiprocessorCount, bt->device) != hipSuccess) {
      rc = vbdr_fail(VBDR_EHIP, "device query failed");
      break;
    }
    for (uint32_t i = 0; i < n_sketches; ++i) {
      vbdr_sketch* s = nullptr;
      const vbdr_batch_params& p = params[i];
      if ((rc = vbdr_sketch_create_lean(p.m, p.g, p.k, p.hash_seed, p.layout, true, &s)) != VBDR_OK) break;
      bt->sk.push_back(s);
      bt->mlp.push_back(nullptr);
      if (!s->def_rec) bt->direct = true;
      else {
        if (bt->runs_max_tiles < s->def_tiles) bt->runs_max_tiles = s->def_tiles;
        if (bt->runs_max_g < s->g) bt->runs_max_g = s->g;
      }
      const uint32_t lds = vbdr_adv_lds(s);
      bt->adv_lds = bt->adv_lds > lds ? bt->adv_lds : lds;
      total_tiles += s->tiles;
      bt->big |= s->tshift == kMaxTileShift;
    }
    if (rc != VBDR_OK) break;
    int lds_max = 0;
    if (hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, bt->device) != hipSuccess ||
        vbdr_batch_scan_lds(bt->runs_max_tiles, bt->runs_max_g) > (size_t)lds_max)
      bt->runs_max_g = 0;
    if (total_tiles >= (1ull << 31)) {
      rc = vbdr_fail(VBDR_EINVAL, "the batch's pools have too many tiles");
      break;
    }
    bt->adv_tiles = (uint32_t)total_tiles;
    const size_t tb = table_bytes(n_sketches);
    if (vbdr_malloc(&bt->desc_dev, tb) != hipSuccess || hipHostMalloc(&bt->staging[0], tb) != hipSuccess ||
        hipHostMalloc(&bt->staging[1], tb) != hipSuccess) {
      rc = vbdr_fail(VBDR_ENOMEM, "batch table allocation failed");
      break;
    }
    bool parts = false;
    for (const vbdr_sketch* s : bt->sk) parts |= member_parts(s) > 1;
    if (parts && (vbdr_malloc(&bt->part_u, kPartEntries * 8ull) != hipSuccess ||
                  vbdr_malloc(&bt->part_v, kPartEntries * 4ull) != hipSuccess)) {
      (void)hipGetLastError();
      rc = vbdr_fail(VBDR_ENOMEM, "allocation of the batch's partial sums failed");
      break;
    }
    bt->hdr_dev = reinterpret_cast<BatchHdr*>(reinterpret_cast<uint8_t*>(bt->desc_dev) + sizeof(BatchDesc) * n_sketches);
    if (hipStreamCreateWithFlags(&bt->st, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&bt->ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&bt->ev_out, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&bt->staged[0], hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&bt->staged[1], hipEventDisableTiming) != hipSuccess) {
      rc = vbdr_fail(VBDR_EHIP, "stream or event creation failed");
      break;
    }
  } while (0);
  if (rc != VBDR_OK) {
    vbdr_batch_destroy(bt);
    return rc;
  }
  *out = bt;
  return VBDR_OK;
}

void vbdr_batch_destroy(vbdr_batch* bt) {
  if (!bt) return;
  (void)hipDeviceSynchronize();
  drop_graph(bt);
  for (vbdr_sketch* s : bt->sk) vbdr_sketch_destroy(s);
  if (bt->desc_dev) (void)hipFree(bt->desc_dev);
  if (bt->part_u) (void)hipFree(bt->part_u);
  if (bt->part_v) (void)hipFree(bt->part_v);
  for (int i = 0; i < 2; ++i) {
    if (bt->staging[i]) (void)hipHostFree(bt->staging[i]);
    if (bt->staged[i]) (void)hipEventDestroy(bt->staged[i]);
  }
  if (bt->ev_in) (void)hipEventDestroy(bt->ev_in);
  if (bt->ev_out) (void)hipEventDestroy(bt->ev_out);
  if (bt->st) (void)hipStreamDestroy(bt->st);
  delete bt;
}

int vbdr_batch_set_mlp(vbdr_batch* bt, uint32_t i, const vbdr_mlp* mlp) {
  if (!bt || i >= bt->S) return vbdr_fail(VBDR_EINVAL, "no sketch %u in this batch", i);
  VBDR_HIP(hipStreamSynchronize(bt->st));  // steps already enqueued keep the estimator they were given
  bt->mlp[i] = mlp;
  return VBDR_OK;
}

vbdr_sketch* vbdr_batch_sketch(vbdr_batch* bt, uint32_t i) {
  if (!bt || i >= bt->S) {
    vbdr_fail(VBDR_EINVAL, "no sketch %u in this batch", i);
    return nullptr;
  }
  return bt->sk[i];
}

int vbdr_batch_set_tuning(vbdr_batch* bt, const vbdr_batch_tuning* t) {
  if (!bt || !t) return vbdr_fail(VBDR_EINVAL, "NULL argument");
  if (t->scan_tile < 256 || t->scan_tile > (1u << 22) || t->est_tile < 4 || t->est_tile > (1u << 16) ||
      t->blocks_per_cu < 1 || t->blocks_per_cu > 32 || t->use_graph < 0 || t->use_graph > 1)
    return vbdr_fail(VBDR_EINVAL, "tuning out of range");
  if (std::memcmp(t, &bt->tune, sizeof(*t)) != 0) {
    VBDR_HIP(hipStreamSynchronize(bt->st));
    drop_graph(bt);  // launch shapes are baked into the captured graph
    bt->tune = *t;
  }
  return VBDR_OK;
}

int vbdr_batch_get_tuning(const vbdr_batch* bt, vbdr_batch_tuning* t) {
  if (!bt || !t) return vbdr_fail(VBDR_EINVAL, "NULL argument");
  *t = bt->tune;
  return VBDR_OK;
}

int vbdr_batch_step(vbdr_batch* bt, const uint32_t* const* pairs_dev, const uint64_t* n_pairs,
                    const uint32_t* const* hosts_dev, const uint64_t* n_hosts, float* const* out_dev, void* stream) {
  if (!bt || !pairs_dev || !n_pairs || !hosts_dev || !n_hosts || !out_dev) return vbdr_fail(VBDR_EINVAL, "NULL argument");
  int cur = -1;
  VBDR_HIP(hipGetDevice(&cur));
  if (cur != bt->device) return vbdr_fail(VBDR_EINVAL, "batch lives on device %d", bt->device);
  const uint32_t S = bt->S;
  uint64_t scan_total = 0, est_total = 0;
  for (uint32_t s = 0; s < S; ++s) {
    if (n_pairs[s] && (!pairs_dev[s] || (reinterpret_cast<uintptr_t>(pairs_dev[s]) & 7u)))
      return vbdr_fail(VBDR_EINVAL, "sketch %u: pairs must be non-NULL and 8-byte aligned", s);
    if (n_hosts[s] && (!hosts_dev[s] || !out_dev[s])) return vbdr_fail(VBDR_EINVAL, "sketch %u: NULL hosts or out", s);
    scan_total += (n_pairs[s] + bt->tune.scan_tile - 1) / bt->tune.scan_tile;
    est_total += (n_hosts[s] + bt->tune.est_tile - 1) / bt->tune.est_tile;
  }
  if (scan_total >= (1ull << 31) || est_total >= (1ull << 31))
    return vbdr_fail(VBDR_EINVAL, "too many work items in one step");
  // fill a pinned staging table (wait until its previous upload has run)
  const int buf = bt->next;
  bt->next ^= 1;
  VBDR_HIP(hipEventSynchronize(bt->staged[buf]));
  BatchDesc* desc = reinterpret_cast<BatchDesc*>(bt->staging[buf]);
  BatchHdr* hdr = reinterpret_cast<BatchHdr*>(bt->staging[buf] + sizeof(BatchDesc) * S);
  DeferItem* ditems = defer_items(bt->staging[buf], S);
  DeferHdr* dhdr = defer_hdr(bt->staging[buf], S);
  const uint32_t chunk = kDeferChunk;
  uint32_t si = 0, dsi = 0, dai = 0, part_used = 0;
  uint64_t cost[2] = {0, 0};
  for (uint32_t s = 0; s < S; ++s) {
    const vbdr_sketch* k = bt->sk[s];
    const bool runs = k->def_rec != nullptr;  // scanned in chunks, no items in the direct scan
    DeferItem& I = ditems[s];
    vbdr_defer_member(k, &I);
    I.pairs = pairs_dev[s], I.n_pairs = n_pairs[s];
    I.scan_item0 = dsi, I.adv_item0 = dai;
    if (runs) dsi += (uint32_t)((n_pairs[s] + chunk - 1) / chunk);
    dai += k->tiles;
    BatchDesc& D = desc[s];
    D.dr = k->dr, D.seen = k->seen, D.reg = k->reg, D.reg4 = k->reg4, D.hist = k->hist, D.s1 = k->s1;
    D.mstride = k->mstride, D.wstride = k->wstride;
    D.m = (uint32_t)k->m, D.g = k->g, D.b = k->b, D.L = k->L, D.k = k->k, D.layout = (uint32_t)k->layout;
    D.A1 = k->A1, D.test = k->tune.scan_test_first == 1;
    D.pairs = pairs_dev[s], D.n_pairs = n_pairs[s];
    D.hosts = hosts_dev[s], D.n_hosts = n_hosts[s], D.out = out_dev[s];
    D.scan_item0 = si;
    // members with a learned estimator are estimated after the step's kernels
    const uint64_t n_plain = bt->mlp[s] ? 0 : n_hosts[s];
    if (!runs) si += (uint32_t)((n_pairs[s] + bt->tune.scan_tile - 1) / bt->tune.scan_tile);
    estimate_plan(bt, k, n_plain, &part_used, cost, &D);
  }
  std::memset(hdr, 0, sizeof(*hdr));
  hdr->scan_total = si, hdr->cost[0] = cost[0], hdr->cost[1] = cost[1];
  std::memset(dhdr, 0, sizeof(*dhdr));
  dhdr->scan_total = dsi;
  // order after the caller's stream, run on the batch stream, order the caller after it
  hipStream_t user = reinterpret_cast<hipStream_t>(stream);
  VBDR_HIP(hipEventRecord(bt->ev_in, user));
  VBDR_HIP(hipStreamWaitEvent(bt->st, bt->ev_in, 0));
  VBDR_HIP(hipMemcpyAsync(bt->desc_dev, bt->staging[buf], table_bytes(S), hipMemcpyHostToDevice, bt->st));
  VBDR_HIP(hipEventRecord(bt->staged[buf], bt->st));
  if (bt->tune.use_graph) {
    if (!bt->exec) {
      VBDR_HIP(hipStreamBeginCapture(bt->st, hipStreamCaptureModeThreadLocal));
      const int rc = launch_step_kernels(bt);
      hipGraph_t g = nullptr;
      const hipError_t e = hipStreamEndCapture(bt->st, &g);
      if (rc != VBDR_OK) return rc;
      if (e != hipSuccess) return vbdr_fail(VBDR_EHIP, "graph capture failed: %s", hipGetErrorString(e));
      bt->graph = g;
      VBDR_HIP(hipGraphInstantiate(&bt->exec, bt->graph, nullptr, nullptr, 0));
    }
    VBDR_HIP(hipGraphLaunch(bt->exec, bt->st));
  } else if (int rc = launch_step_kernels(bt)) {
    return rc;
  }
  for (uint32_t s = 0; s < S; ++s)
    if (bt->mlp[s] && n_hosts[s])
      if (int rc = vbdr_estimate_learned(bt->sk[s], bt->mlp[s], hosts_dev[s], n_hosts[s], out_dev[s], nullptr, bt->st))
        return rc;
  VBDR_HIP(hipEventRecord(bt->ev_out, bt->st));
  VBDR_HIP(hipStreamWaitEvent(user, bt->ev_out, 0));
  for (vbdr_sketch* k : bt->sk) k->t++, k->open_records = 0;
  return VBDR_OK;
}

}  // extern "C"
