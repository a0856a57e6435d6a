// Uneven batches: populations of many graphs (different n, k, budgets) in one
// hipGraph, captured once and replayed.
//
// Work items are (graph, individual) pairs ordered longest-first (graphs by
// n * k * iterations, descending).  Graphs that the wave table holds within
// the launch's LDS budget run the WAVE8 search, one workgroup per item, with
// one, two or four waves each; the launches of the three are branches of the
// graph beside the block search of the others, and one more node reruns what
// the wave table gave up on.  A batch lasts as long as its longest chain: 12
// graphs of 100 to 1,000 vertices with 64 individuals each (the longest: 854
// vertices, k = 174) took 170 ms on the block search alone.
//
// The others share one persistent launch: as many workgroups as the device
// keeps resident at its LDS size; each workgroup pops items
// from an atomic counter until the queue is empty, so every workgroup exits.
// A graph whose table fits the launch's LDS budget runs the LDS16 table, one
// whose byte gamma alone fits runs the SPLIT8 table (expiries in device
// memory, a rerun with the device-memory table in the same slot if a colour
// class would pass 255 vertices), the others the device-memory table; device
// storage is one slot per workgroup.  The search itself is the same function
// as dlm_tabu_batch's, so trajectories are identical to single-graph runs
// with the same seeds and indices.
#include <algorithm>
#include <chrono>
#include <map>
#include <mutex>
#include <numeric>
#include <vector>

#include "tabu_wave.h"
#include "tabu_wave_launch.h"
#include "tabu_wave_multi.h"

namespace dlm {

struct MultiDesc {
  TabuArgs a;
  int32_t tier;        // 0 = LDS16, 1 = GLOBAL16, 3 = SPLIT8 (GLOBAL16 rerun past 255 per class)
  int32_t first_item;  // items [first_item, first_item + pop) belong to this graph
  int32_t pop;
  int32_t pad;
};

__global__ void fill_u32_kernel(uint32_t* p, int32_t n, uint32_t v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void tabu_multi_kernel(const MultiDesc* __restrict__ descs, int32_t ndesc,
                                                           int32_t total, uint32_t* __restrict__ queue,
                                                           uint32_t* __restrict__ gslots, int64_t slot_words) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t s_item;
  unsigned char* gtab =
      gslots ? reinterpret_cast<unsigned char*>(gslots + (size_t)blockIdx.x * (size_t)slot_words) : nullptr;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = (int32_t)atomicAdd(queue, 1u);
    __syncthreads();
    const int32_t item = s_item;
    if (item >= total) break;  // uniform: every workgroup reaches this exit
    int g = 0;
    while (g + 1 < ndesc && descs[g + 1].first_item <= item) ++g;
    const MultiDesc& d = descs[g];
    const int li = item - d.first_item;
    if (d.tier == 0) {
      tabu_individual<BLOCK, TabLds16>(d.a, li, nullptr, smem);
    } else if (d.tier == 3) {
      // byte gamma; the start colouring waits behind the slot's table for a
      // 16-bit rerun if a colour class would pass 255 vertices
      const int n = d.a.n;
      int16_t* gcol = d.a.colors + (size_t)li * n;
      int16_t* save = reinterpret_cast<int16_t*>(gtab + tab_entries(n, d.a.k) * TabGlobal16::kGlobalBytes);
      for (int v = threadIdx.x; v < n; v += BLOCK) save[v] = gcol[v];
      __syncthreads();
      tabu_individual<BLOCK, TabSplit8>(d.a, li, gtab, smem);
      __syncthreads();
      if (d.a.iters[li] == -2) {
        for (int v = threadIdx.x; v < n; v += BLOCK) gcol[v] = save[v];
        __syncthreads();
        tabu_individual<BLOCK, TabGlobal16>(d.a, li, gtab, smem);
      }
    } else {
      tabu_individual<BLOCK, TabGlobal16>(d.a, li, gtab, smem);
    }
  }
}

// What the wave tables gave up on, from its saved start with the packed 16-bit
// table in device memory, one slot per workgroup.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void tabu_multi_rerun_kernel(const WaveDesc* __restrict__ descs, int32_t ndesc,
                                                                 int32_t total, unsigned char* __restrict__ slots,
                                                                 int64_t slot_bytes) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* gtab = slots + (size_t)blockIdx.x * (size_t)slot_bytes;
  int g = 0;
  for (int32_t item = blockIdx.x; item < total; item += gridDim.x) {
    while (g + 1 < ndesc && descs[g + 1].first_item <= item) ++g;
    const WaveDesc& d = descs[g];
    const int li = item - d.first_item;
    if (d.a.iters[li] != kW8GaveUp) continue;
    const size_t row = (size_t)li * (size_t)d.a.n;
    for (int v = threadIdx.x; v < d.a.n; v += BLOCK) d.a.colors[row + v] = d.start[row + v];
    __syncthreads();
    tabu_individual<BLOCK, TabGlobal16>(d.a, li, gtab, smem);
    __syncthreads();
  }
}

}  // namespace dlm

using namespace dlm;

struct dlm_multi_plan {
  int32_t block = 256, lds_budget = 0, grid = 0, total = 0, block_items = 0, ndesc = 0, n_global = 0;
  size_t lds = 0, info_lds = 0;
  int64_t slot_words = 0;
  MultiDesc* d_descs = nullptr;
  uint32_t* d_queue = nullptr;
  uint32_t* d_slots = nullptr;
  // the wave table's share: its descriptors launch by launch, then those of the
  // reruns with 8-bit entries
  struct Launch {
    int32_t waves, desc, ndesc, item, items;
    size_t lds;
  };
  std::vector<Launch> launches;
  int32_t wave_descs = 0, wave_items = 0, again_descs = 0, again_items = 0;
  size_t again_lds = 0;
  int32_t rr_grid = 0;
  size_t rr_lds = 0;
  int64_t rr_slot_bytes = 0;
  WaveDesc* d_wdescs = nullptr;
  int16_t* d_start = nullptr;
  unsigned char* d_rr_slots = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace {

int validate_items(const dlm_multi_item* items, int32_t count) {
  if (count < 1 || !items) return set_error(DLM_E_INVAL, "dlm_multi: count=%d", count);
  int64_t total = 0;
  for (int i = 0; i < count; ++i) {
    const dlm_multi_item& it = items[i];
    if (!it.g) return set_error(DLM_E_INVAL, "dlm_multi: item %d has no graph", i);
    if (it.k < 1 || it.k > 32767 || it.max_iters < 0 || it.max_iters > (1 << 30) || it.pop < 0 ||
        it.ten_den <= 0 || it.ten_num < 0 || it.ten_num > 32767 || it.ten_rand < 1 || it.ten_rand > 1024 ||
        it.ind_base < 0 || (int64_t)it.ind_base + it.pop > 0x7fffffffll || it.reserved != 0)
      return set_error(DLM_E_INVAL, "dlm_multi: item %d has invalid parameters", i);
    if (it.pop > 0 && (!it.colors_dev || !it.f_best_dev || !it.iters_dev))
      return set_error(DLM_E_INVAL, "dlm_multi: item %d has a null output buffer", i);
    total += it.pop;
  }
  if (total > 0x7fffffffll) return set_error(DLM_E_INVAL, "dlm_multi: too many individuals");
  return DLM_OK;
}

template <int BLOCK>
int occupancy(size_t lds, int* per_cu) {
  DLM_HIP(hipFuncSetAttribute((const void*)tabu_multi_kernel<BLOCK>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  DLM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, tabu_multi_kernel<BLOCK>, BLOCK, lds));
  return DLM_OK;
}

int launch_persistent(const dlm_multi_plan* p, hipStream_t s) {
  switch (p->block) {
#define DLM_CASE(B)                                                                                       \
  case B:                                                                                                 \
    hipLaunchKernelGGL(tabu_multi_kernel<B>, dim3(p->grid), dim3(B), p->lds, s, p->d_descs, p->ndesc,     \
                       p->block_items, p->d_queue, p->d_slots, p->slot_words);                                  \
    break;
    DLM_CASE(64)
    DLM_CASE(128)
    DLM_CASE(256)
    DLM_CASE(512)
#undef DLM_CASE
    default:
      return set_error(DLM_E_INVAL, "dlm_multi: block=%d not in {64,128,256,512}", p->block);
  }
  DLM_HIP(hipGetLastError());
  return DLM_OK;
}

void free_plan(dlm_multi_plan* p) {
  if (!p) return;
  if (p->exec) (void)hipGraphExecDestroy(p->exec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  (void)hipFree(p->d_descs);
  (void)hipFree(p->d_queue);
  (void)hipFree(p->d_slots);
  (void)hipFree(p->d_wdescs);
  (void)hipFree(p->d_start);
  (void)hipFree(p->d_rr_slots);
  delete p;
}

constexpr int kRerunBlock = 256;
constexpr uint64_t kRerunSlotBytes = 256ull << 20;  // of all rerun slots together

// One graph of the batch on the wave table.
struct WaveItem {
  int oi;  // index into items
  W8Pick pick;
  int instance;
  int64_t least;  // LDS with the side list a random start needs
};

dlm_tabu_params item_params(const dlm_multi_item& it) {
  dlm_tabu_params q{};
  q.k = it.k;
  q.max_iters = it.max_iters;
  q.ten_num = it.ten_num;
  q.ten_den = it.ten_den;
  q.ten_rand = it.ten_rand;
  q.ind_base = it.ind_base;
  q.seed = it.seed;
  return q;
}

// Whether a graph of the batch runs the wave table, and how.  Classes of more
// than half the limit in the mean are left to the block search: a rerun here
// begins when everything else has ended.  pop: the individuals that the
// number of waves is picked for; crowd: those that share the card.
bool wave_item(const dlm_multi_item& it, int64_t pop, int64_t crowd, int64_t budget, WaveItem& w) {
  const dlm_tabu_params q = item_params(it);
  if (!it.g->ell || !w8_auto(it.g, &q) || it.g->n > (int)(kW8ClassMax / 2) * it.k || block_faster(it.g, &q, crowd))
    return false;
  w.pick = w8_pick(it.g, &q, pop);
  w.instance = w8_multi_instance(it.k, w.pick.bits);
  w.least = (int64_t)w8_layout(it.g->n, it.k, w.pick.bits, w.pick.waves, (int)w.pick.side).bytes;
  const int64_t rr = (int64_t)tabu_layout(it.g->n, it.k, kRerunBlock / kWave, 0).bytes;
  return w.instance >= 0 && w.least <= budget && rr <= device_lds_limit();
}

// A launch of the wave search: graphs with the same number of waves, longest
// first.  Every workgroup of it gets the LDS of the largest.
struct WaveLaunch {
  std::vector<WaveItem> graphs;
  int64_t lds = 0, pop = 0;

  void add(const WaveItem& w, int64_t individuals) {
    graphs.push_back(w);
    lds = std::max(lds, w.least);
    pop += individuals;
  }
  // CUs that its individuals fill by their LDS
  double cus() const {
    return pop == 0 ? 0.0 : (double)pop / std::max<int64_t>(1, device_lds_per_cu() / kLdsGranule / ((lds + kLdsGranule - 1) / kLdsGranule));
  }
};

// CUs that the individuals fill by their LDS, each launch by itself.
double cus_of(const std::vector<WaveLaunch>& launches) {
  double c = 0.0;
  for (const WaveLaunch& l : launches) c += l.cus();
  return c;
}

// At most `most` launches: one per number of waves; while the card does not hold
// them, the one whose parting by LDS leaves the most CUs free is parted.  Without
// it one graph of 854 vertices (88 KB) gave 576 individuals of four waves a CU
// each, though most of them need 12 to 63 KB, and 320 of them had to queue.
std::vector<WaveLaunch> wave_launches(const dlm_multi_item* items, const std::vector<WaveItem>& graphs, size_t most) {
  std::vector<WaveLaunch> r;
  for (int waves : {4, 2, 1}) {
    WaveLaunch l;
    for (const WaveItem& w : graphs)
      if (w.pick.waves == waves) l.add(w, items[w.oi].pop);
    if (!l.graphs.empty()) r.push_back(l);
  }
  while (r.size() < most && cus_of(r) > device_cu_count()) {
    double best = 1.0;  // CUs
    size_t at = 0;
    WaveLaunch large, small;
    for (size_t i = 0; i < r.size(); ++i)
      for (const WaveItem& cut : r[i].graphs) {
        WaveLaunch a, b;
        for (const WaveItem& w : r[i].graphs) (w.least >= cut.least ? a : b).add(w, items[w.oi].pop);
        const double free = r[i].cus() - a.cus() - b.cus();
        if (free > best) {
          best = free;
          at = i;
          large = a;
          small = b;
        }
      }
    if (large.graphs.empty()) break;
    r[at] = large;
    r.insert(r.begin() + (std::ptrdiff_t)at + 1, small);
  }
  return r;
}

// Branches of the plan's graph: up to three launches of the wave table, one per
// number of waves, and the block search.
constexpr size_t kStreams = 4;
// Launches are parted up to so many branches.  A process has four hardware
// queues; with a fourth wave launch two of them came to lie on one queue, one
// after the other (a batch of 9 graphs of 75 to 534 vertices: 47 ms instead of 27).
constexpr size_t kParted = 3;

// The launches of the wave table's graphs.  A batch that the card holds whole
// is as long as its longest individual: each graph gets the waves it would get
// alone.  Otherwise the individuals share the CUs and the whole batch counts.
std::vector<WaveLaunch> wave_plan(const dlm_multi_item* items, const std::vector<int>& order, int64_t budget) {
  int64_t total = 0;
  for (int oi : order) total += items[oi].pop;
  auto launches = [&](bool alone) {
    std::vector<WaveItem> graphs;
    bool block = false;  // the block search takes a branch
    for (int oi : order) {
      WaveItem w{};
      w.oi = oi;
      if (items[oi].pop == 0) continue;
      // a graph that the budget holds only with fewer waves than it would get
      // alone is the batch's longest chain on the wave table: left to the block
      // search (one of 832 vertices in the 64-graph batch: 1,400 instead of 1,030 ms)
      const int64_t crowd = alone ? items[oi].pop : total;
      bool fits = wave_item(items[oi], items[oi].pop, crowd, budget, w);
      if (fits && !alone) fits = wave_item(items[oi], total, crowd, budget, w);
      if (fits)
        graphs.push_back(w);
      else
        block = true;
    }
    return wave_launches(items, graphs, kParted - (block ? 1 : 0));
  };
  std::vector<WaveLaunch> r = launches(true);
  int64_t waves = 0;
  for (const WaveLaunch& l : r) waves += l.pop * l.graphs[0].pick.waves;
  if (cus_of(r) > device_cu_count() || waves > 16 * (int64_t)device_cu_count()) r = launches(false);
  return r;
}

// The plan's nodes onto cs[kStreams - 1] (capturing), the launches of the wave
// table on branches of their own; the last is the block search's.
int capture_plan(const dlm_multi_plan* p, const hipStream_t* cs, const hipEvent_t* ev) {
  static_assert(kParted < kStreams, "every wave launch has a stream of its own");
  hipStream_t s = cs[kStreams - 1];
  hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, p->d_queue, 1, 0u);
  DLM_HIP(hipGetLastError());
  DLM_HIP(hipEventRecord(ev[kStreams - 1], s));
  for (size_t i = 0; i < p->launches.size(); ++i) {
    const dlm_multi_plan::Launch& l = p->launches[i];
    DLM_HIP(hipStreamWaitEvent(cs[i], ev[kStreams - 1], 0));
    const auto launch = l.waves == 4 ? launch_multi_w8_4 : l.waves == 2 ? launch_multi_w8_2 : launch_multi_w8_1;
    const int rc = launch(p->d_wdescs + l.desc, l.ndesc, l.item, l.items, l.lds, cs[i]);
    if (rc != DLM_OK) return rc;
    DLM_HIP(hipEventRecord(ev[i], cs[i]));
  }
  if (p->block_items > 0) {
    const int rc = launch_persistent(p, s);
    if (rc != DLM_OK) return rc;
  }
  for (size_t i = 0; i < p->launches.size(); ++i) DLM_HIP(hipStreamWaitEvent(s, ev[i], 0));
  if (p->again_items > 0) {
    const int rc = launch_multi_w8_again(p->d_wdescs + p->wave_descs, p->again_descs, p->again_items, p->again_lds, s);
    if (rc != DLM_OK) return rc;
  }
  if (p->rr_grid > 0) {
    auto kern = tabu_multi_rerun_kernel<kRerunBlock>;
    DLM_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p->rr_lds));
    hipLaunchKernelGGL(kern, dim3(p->rr_grid), dim3(kRerunBlock), p->rr_lds, s, p->d_wdescs, p->wave_descs,
                       p->wave_items, p->d_rr_slots, p->rr_slot_bytes);
    DLM_HIP(hipGetLastError());
  }
  return DLM_OK;
}

}  // namespace

extern "C" {

int dlm_multi_plan_create(const dlm_multi_item* items, int32_t count, const dlm_multi_config* cfg,
                          void* stream, dlm_multi_plan** out) {
  if (!out) return set_error(DLM_E_INVAL, "dlm_multi_plan_create: out is NULL");
  *out = nullptr;
  int rc = validate_items(items, count);
  if (rc != DLM_OK) return rc;
  const int block = cfg && cfg->block ? cfg->block : 256;
  if (block != 64 && block != 128 && block != 256 && block != 512)
    return set_error(DLM_E_INVAL, "dlm_multi_plan_create: block=%d not in {64,128,256,512}", block);
  const int nw = block / kWave;
  const int64_t lds_max = device_lds_limit();
  const int64_t budget = cfg && cfg->lds_budget ? std::min<int64_t>(cfg->lds_budget, lds_max) : lds_max;
  // longest first
  std::vector<int> order(count);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
    const double ca = (double)items[a].g->n * items[a].k * items[a].max_iters;
    const double cb = (double)items[b].g->n * items[b].k * items[b].max_iters;
    return ca > cb;
  });
  dlm_multi_plan* p = new dlm_multi_plan();
  p->block = block;
  p->lds_budget = (int32_t)budget;
  std::vector<MultiDesc> descs;
  const std::vector<WaveLaunch> wave = wave_plan(items, order, budget);
  std::vector<char> on_wave(count, 0);
  for (const WaveLaunch& l : wave)
    for (const WaveItem& w : l.graphs) on_wave[w.oi] = 1;
  int32_t first = 0;
  size_t lds = tabu_layout(1, 1, nw, 0).bytes;
  for (int oi : order) {
    const dlm_multi_item& it = items[oi];
    if (it.pop == 0) continue;
    const int n = it.g->n;
    MultiDesc d{};
    d.a = TabuArgs{it.g->row_ptr, it.g->col_idx, it.g->erow, it.colors_dev, it.f_best_dev, it.iters_dev,
                   it.stats_dev, it.hash_dev, nullptr, nullptr, make_key(it.seed), n, it.k, it.max_iters,
                   it.ten_num, it.ten_den, it.ten_rand, it.ind_base, 0};
    const uint64_t lds16 = tabu_layout(n, it.k, nw, TabLds16::kLdsBytes).bytes;
    const uint64_t lds8 = tabu_layout(n, it.k, nw, TabSplit8::kLdsBytes).bytes;
    if (on_wave[oi]) {
      if ((int64_t)lds16 > budget) ++p->n_global;
      continue;
    }
    if ((int64_t)lds16 <= budget) {
      d.tier = 0;
      lds = std::max<size_t>(lds, lds16);
    } else if ((int64_t)lds8 <= budget) {
      d.tier = 3;
      ++p->n_global;
      lds = std::max<size_t>(lds, lds8);
      // packed 16-bit table for a rerun (the byte run's expiries use the first half) + the start colouring
      p->slot_words = std::max<int64_t>(p->slot_words, (int64_t)tab_entries(n, it.k) + (n + 1) / 2);
    } else {
      d.tier = 1;
      ++p->n_global;
      lds = std::max<size_t>(lds, tabu_layout(n, it.k, nw, 0).bytes);
      p->slot_words = std::max<int64_t>(p->slot_words, (int64_t)tab_entries(n, it.k));
    }
    d.first_item = first;
    d.pop = it.pop;
    first += it.pop;
    descs.push_back(d);
  }
  p->slot_words = (p->slot_words + 3) & ~int64_t(3);  // 16-byte aligned slots
  p->block_items = first;
  // the wave table's descriptors; a launch's LDS leaves its smaller individuals
  // more side-list entries
  std::vector<WaveDesc> wdescs;
  std::vector<size_t> start_at;
  std::vector<const WaveItem*> wave_of;
  size_t start_cells = 0;
  int32_t witems = 0;
  for (const WaveLaunch& l : wave) {
    const int nwv = l.graphs[0].pick.waves;
    p->launches.push_back({nwv, (int32_t)wdescs.size(), (int32_t)l.graphs.size(), witems, (int32_t)l.pop, (size_t)l.lds});
    for (const WaveItem& w : l.graphs) {
      wave_of.push_back(&w);
      const dlm_multi_item& it = items[w.oi];
      const int n = it.g->n;
      WaveDesc d{};
      d.a = TabuArgs{it.g->row_ptr, it.g->col_idx, it.g->erow, it.colors_dev, it.f_best_dev, it.iters_dev,
                     it.stats_dev, it.hash_dev, nullptr, nullptr, make_key(it.seed), n, it.k, it.max_iters,
                     it.ten_num, it.ten_den, it.ten_rand, it.ind_base, 0, it.g->ell, it.g->adj, it.g->ell_stride};
      const int64_t room = l.lds - (int64_t)w8_layout(n, it.k, w.pick.bits, nwv, 0).bytes;
      W8Pick b;
      const dlm_tabu_params q = item_params(it);
      const bool again = w.pick.bits == 4 && w8_pick_bytes(it.g, &q, it.pop, b);
      const int64_t most = again ? w.pick.side + kW4Spare : kW8SideMax;
      d.acap = (int32_t)std::max<int64_t>(w.pick.side, std::min<int64_t>(most, (room / 6) & ~63ll));
      d.instance = w.instance;
      d.first_item = witems;
      d.pop = it.pop;
      witems += it.pop;
      start_at.push_back(start_cells);
      start_cells += (size_t)it.pop * n;
      wdescs.push_back(d);
      p->rr_slot_bytes = std::max<int64_t>(p->rr_slot_bytes, (int64_t)((tab_entries(n, it.k) * TabGlobal16::kGlobalBytes + 15) & ~15ull));
      p->rr_lds = std::max(p->rr_lds, (size_t)tabu_layout(n, it.k, kRerunBlock / kWave, 0).bytes);
    }
    p->info_lds = std::max(p->info_lds, (size_t)l.lds);
  }
  p->wave_descs = (int32_t)wdescs.size();
  // reruns with 8-bit entries: few and late, so four waves each
  for (int32_t i = 0; i < p->wave_descs; ++i) {
    const WaveItem& w = *wave_of[i];
    const dlm_multi_item& it = items[w.oi];
    const dlm_tabu_params q = item_params(it);
    W8Pick b;
    if (w.pick.bits != 4 || !w8_pick_bytes(it.g, &q, it.pop, b)) continue;
    WaveDesc d = wdescs[i];
    const int64_t room = std::min(budget, lds_max) - (int64_t)w8_layout(it.g->n, it.k, 8, 4, 0).bytes;
    d.instance = w8_multi_instance(it.k, 8);
    if (d.instance < 0 || room < 6 * kWave) continue;
    d.acap = (int32_t)std::min<int64_t>(std::max<int64_t>(w.pick.side, kWave), (room / 6) & ~63ll);
    d.first_item = p->again_items;
    p->again_items += it.pop;
    start_at.push_back(start_at[i]);
    p->again_lds = std::max(p->again_lds, (size_t)w8_layout(it.g->n, it.k, 8, 4, d.acap).bytes);
    wdescs.push_back(d);
  }
  p->again_descs = (int32_t)wdescs.size() - p->wave_descs;
  p->info_lds = std::max(p->info_lds, p->again_lds);
  p->wave_items = witems;
  if (witems > 0)
    p->rr_grid = (int32_t)std::max<int64_t>(
        1, std::min<int64_t>({(int64_t)witems, 2 * (int64_t)device_cu_count(), (int64_t)(kRerunSlotBytes / (uint64_t)p->rr_slot_bytes)}));
  p->total = first + witems;
  p->ndesc = (int32_t)descs.size();
  p->lds = lds;
  if (first > 0) p->info_lds = std::max(p->info_lds, lds);
  if ((int64_t)lds > lds_max) {
    free_plan(p);
    return set_error(DLM_E_UNSUPPORTED, "dlm_multi_plan_create: %zu bytes of LDS needed", lds);
  }
  int per_cu = 0;
  switch (block) {
    case 64: rc = occupancy<64>(lds, &per_cu); break;
    case 128: rc = occupancy<128>(lds, &per_cu); break;
    case 256: rc = occupancy<256>(lds, &per_cu); break;
    default: rc = occupancy<512>(lds, &per_cu); break;
  }
  if (rc != DLM_OK) {
    free_plan(p);
    return rc;
  }
  p->grid = std::max(1, std::min(per_cu * device_cu_count(), std::max(p->block_items, 1)));
  hipStream_t s = (hipStream_t)stream;
  auto fail = [&](hipError_t e, const char* what) {
    free_plan(p);
    return hip_fail(e, what);
  };
  hipError_t e;
  if ((e = hipMalloc(&p->d_descs, sizeof(MultiDesc) * std::max<size_t>(descs.size(), 1))) != hipSuccess)
    return fail(e, "hipMalloc");
  if ((e = hipMalloc(&p->d_queue, 256)) != hipSuccess) return fail(e, "hipMalloc");
  if (p->slot_words > 0 &&
      (e = hipMalloc(&p->d_slots, sizeof(uint32_t) * (size_t)p->slot_words * p->grid)) != hipSuccess)
    return fail(e, "hipMalloc");
  if (!descs.empty() &&
      (e = hipMemcpy(p->d_descs, descs.data(), sizeof(MultiDesc) * descs.size(), hipMemcpyHostToDevice)) !=
          hipSuccess)
    return fail(e, "hipMemcpy");
  if (!wdescs.empty()) {
    if ((e = hipMalloc(&p->d_wdescs, sizeof(WaveDesc) * wdescs.size())) != hipSuccess) return fail(e, "hipMalloc");
    if ((e = hipMalloc(&p->d_start, sizeof(int16_t) * start_cells)) != hipSuccess) return fail(e, "hipMalloc");
    if ((e = hipMalloc(&p->d_rr_slots, (size_t)p->rr_slot_bytes * p->rr_grid)) != hipSuccess)
      return fail(e, "hipMalloc");
    for (size_t i = 0; i < wdescs.size(); ++i) wdescs[i].start = p->d_start + start_at[i];
    if ((e = hipMemcpy(p->d_wdescs, wdescs.data(), sizeof(WaveDesc) * wdescs.size(), hipMemcpyHostToDevice)) !=
        hipSuccess)
      return fail(e, "hipMemcpy");
  }
  // capture: queue reset (a fill kernel, no memset node), the wave launches and
  // the persistent kernel side by side, the reruns
  hipStream_t cs[kStreams] = {};
  hipEvent_t ev[kStreams] = {};
  auto release = [&]() {
    for (size_t i = 0; i < kStreams; ++i) {
      if (ev[i]) (void)hipEventDestroy(ev[i]);
      if (cs[i]) (void)hipStreamDestroy(cs[i]);
    }
  };
  for (size_t i = 0; i < kStreams; ++i)
    if ((e = hipStreamCreateWithFlags(&cs[i], hipStreamNonBlocking)) != hipSuccess ||
        (e = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming)) != hipSuccess) {
      release();
      return fail(e, "hipStreamCreate");
    }
  if ((e = hipStreamBeginCapture(cs[kStreams - 1], hipStreamCaptureModeThreadLocal)) != hipSuccess) {
    release();
    return fail(e, "hipStreamBeginCapture");
  }
  rc = capture_plan(p, cs, ev);
  e = hipStreamEndCapture(cs[kStreams - 1], &p->graph);
  release();
  if (rc != DLM_OK) {
    free_plan(p);
    return rc;
  }
  if (e != hipSuccess) return fail(e, "hipStreamEndCapture");
  if ((e = hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0)) != hipSuccess)
    return fail(e, "hipGraphInstantiate");
  (void)s;
  *out = p;
  return DLM_OK;
}

int dlm_multi_plan_launch(dlm_multi_plan* p, void* stream) {
  if (!p) return set_error(DLM_E_INVAL, "dlm_multi_plan_launch: plan is NULL");
  DLM_HIP(hipGraphLaunch(p->exec, (hipStream_t)stream));
  return DLM_OK;
}

int dlm_multi_plan_info(const dlm_multi_plan* p, int32_t* grid, int32_t* lds_bytes, int32_t* n_global,
                        int32_t* total_items) {
  if (!p) return set_error(DLM_E_INVAL, "dlm_multi_plan_info: plan is NULL");
  if (grid) *grid = (p->block_items > 0 ? p->grid : 0) + p->wave_items;
  if (lds_bytes) *lds_bytes = (int32_t)p->info_lds;
  if (n_global) *n_global = p->n_global;
  if (total_items) *total_items = p->total;
  return DLM_OK;
}

int dlm_multi_plan_destroy(dlm_multi_plan* p) {
  free_plan(p);
  return DLM_OK;
}

// Calibration: each candidate (block, LDS budget) runs the batch on scratch
// copies of the colourings with `calib_iters` iterations per individual;
// the fastest in iterations per second wins.  Results are cached per
// (device, item shapes).
int dlm_multi_autotune(const dlm_multi_item* items, int32_t count, int32_t calib_iters,
                       dlm_multi_config* best, float* rates, void* stream) {
  int rc = validate_items(items, count);
  if (rc != DLM_OK) return rc;
  if (!best || calib_iters < 1) return set_error(DLM_E_INVAL, "dlm_multi_autotune: bad arguments");
  static std::mutex mu;
  static std::map<std::vector<int64_t>, dlm_multi_config> cache;
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::vector<int64_t> key{dev, calib_iters};
  for (int i = 0; i < count; ++i) {
    key.push_back(items[i].g->n);
    key.push_back(items[i].g->nnz);
    key.push_back(items[i].k);
    key.push_back(items[i].pop);
  }
  const int blocks[] = {64, 128, 256, 512};
  const int64_t lds_max = device_lds_limit();
  const int64_t budgets[] = {lds_max / 4, lds_max / 2, lds_max};
  {
    std::lock_guard<std::mutex> lk(mu);
    auto hit = cache.find(key);
    if (hit != cache.end() && !rates) {
      *best = hit->second;
      return DLM_OK;
    }
  }
  hipStream_t s = (hipStream_t)stream;
  // scratch copies and outputs
  std::vector<dlm_multi_item> cal(items, items + count);
  std::vector<void*> bufs;
  auto cleanup = [&]() {
    for (void* b : bufs) (void)hipFree(b);
  };
  int64_t total_iters_bound = 0;
  for (int i = 0; i < count; ++i) {
    dlm_multi_item& c = cal[i];
    if (c.pop == 0) continue;
    const size_t cb = sizeof(int16_t) * (size_t)c.pop * c.g->n;
    void *col, *fb, *it;
    hipError_t e;
    if ((e = hipMalloc(&col, cb)) != hipSuccess || (e = hipMalloc(&fb, 4 * (size_t)c.pop)) != hipSuccess ||
        (e = hipMalloc(&it, 4 * (size_t)c.pop)) != hipSuccess) {
      cleanup();
      return hip_fail(e, "hipMalloc (autotune)");
    }
    bufs.push_back(col);
    bufs.push_back(fb);
    bufs.push_back(it);
    c.colors_dev = (int16_t*)col;
    c.f_best_dev = (int32_t*)fb;
    c.iters_dev = (int32_t*)it;
    c.stats_dev = nullptr;
    c.hash_dev = nullptr;
    c.max_iters = std::min(c.max_iters, calib_iters);
    total_iters_bound += (int64_t)c.pop * c.max_iters;
  }
  hipEvent_t e0, e1;
  (void)hipEventCreate(&e0);
  (void)hipEventCreate(&e1);
  float best_rate = -1.f;
  dlm_multi_config best_cfg{256, 0};
  int ci = 0;
  for (int b : blocks)
    for (int64_t bud : budgets) {
      dlm_multi_config cfg{b, (int32_t)bud};
      for (int i = 0; i < count; ++i)
        if (cal[i].pop)
          (void)hipMemcpyAsync(cal[i].colors_dev, items[i].colors_dev,
                               sizeof(int16_t) * (size_t)cal[i].pop * cal[i].g->n, hipMemcpyDeviceToDevice, s);
      dlm_multi_plan* p = nullptr;
      float rate = 0.f;
      if (dlm_multi_plan_create(cal.data(), count, &cfg, stream, &p) == DLM_OK) {
        (void)hipEventRecord(e0, s);
        rc = dlm_multi_plan_launch(p, stream);
        (void)hipEventRecord(e1, s);
        (void)hipEventSynchronize(e1);
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        // iterations actually run (early stops at f = 0 count as run iterations)
        int64_t iters = 0;
        for (int i = 0; i < count; ++i) {
          if (!cal[i].pop) continue;
          std::vector<int32_t> h(cal[i].pop);
          (void)hipMemcpy(h.data(), cal[i].iters_dev, 4 * (size_t)cal[i].pop, hipMemcpyDeviceToHost);
          for (int32_t x : h) iters += x;
        }
        rate = ms > 0.f && rc == DLM_OK ? (float)(iters / (ms * 1e-3)) : 0.f;
        dlm_multi_plan_destroy(p);
      }
      if (rates) rates[ci] = rate;
      ++ci;
      if (rate > best_rate) {
        best_rate = rate;
        best_cfg = cfg;
      }
    }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  cleanup();
  (void)total_iters_bound;
  if (best_rate <= 0.f) return set_error(DLM_E_HIP, "dlm_multi_autotune: no configuration ran");
  *best = best_cfg;
  std::lock_guard<std::mutex> lk(mu);
  cache[key] = best_cfg;
  return DLM_OK;
}

}  // extern "C"
