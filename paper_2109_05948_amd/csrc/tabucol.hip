// Population TabuCol for k-COL (Section 2.7 of the paper: TabuCol with the
// gamma table of its efficient implementation), one workgroup per individual.
//
// Per individual (the search body and the table tiers are in tabu_body.h):
//   tab[v*kp + c]  gamma[v][c] (neighbours of v coloured c) and the tabu
//                  expiry of (v, c), rows padded to kp = k rounded up to 4;
//                  LDS16 packs both into a 32-bit LDS word, LDS32 keeps two,
//                  SPLIT16 / SPLIT8 keep 16- / 8-bit gamma in LDS and the
//                  expiries in device memory, GLOBAL16 keeps the packed word
//                  in device memory
//   cg[v]          colour of v (low 16) | gamma[v][col v] (high 16)
//   list, pos      the conflicting vertices (with tombstones), kept in place
//
// One iteration:
//   scan      every thread takes (list entry, colour quad) pairs strided by
//             the block size and keeps its three smallest admissible
//             candidate keys (biased delta << 16 | the thread's candidate
//             number);
//   wave      DPP minimum; the moves tied at the wave's minimum are hashed
//             (Philox of (ind, t, v, c)) unless another wave already
//             published a better delta;
//   reduce    one barrier, then the (delta, hash, v, c) minimum over the
//             waves' slots;
//   apply     all threads update the gamma rows of v*'s neighbours (CSR row
//             from device memory) and the conflict list; wave 0 writes the
//             tabu entries, v*'s state and the lazily kept best colouring.
//
// The byte-gamma tier gives up on an individual whose colour classes would
// pass 255 vertices; a rerun kernel repeats those from their start colouring
// with the 16-bit device table, so every tier returns the same result.
#include <math.h>

#include <mutex>

#include "tabu_body.h"
#include "tabu_wave.h"
#include "tabu_wave_launch.h"

namespace dlm {

template <int BLOCK, class Tab>
__global__ __launch_bounds__(BLOCK) void tabucol_kernel(TabuArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int li = blockIdx.x;
  unsigned char* gtab =
      a.gtab ? a.gtab + (size_t)li * (size_t)tab_entries(a.n, a.k) * Tab::kGlobalBytes : nullptr;
  tabu_individual<BLOCK, Tab>(a, li, gtab, smem);
}

// Byte-gamma runs that gave up (iters = -2: a colour class would pass 255
// vertices) start again from their saved start colouring with the packed
// 16-bit table in device memory.  A persistent grid walks the population;
// every workgroup owns one table slot and skips the individuals that
// finished.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void tabucol_rerun_kernel(TabuArgs a, const int16_t* __restrict__ start,
                                                              unsigned char* __restrict__ slots, int32_t pop) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* slot = slots + (size_t)blockIdx.x * (size_t)tab_entries(a.n, a.k) * TabGlobal16::kGlobalBytes;
  for (int li = blockIdx.x; li < pop; li += gridDim.x) {
    if (a.iters[li] != kW8GaveUp) continue;
    int16_t* gcol = a.colors + (size_t)li * a.n;
    for (int v = threadIdx.x; v < a.n; v += BLOCK) gcol[v] = start[(size_t)li * a.n + v];
    __syncthreads();
    tabu_individual<BLOCK, TabGlobal16>(a, li, slot, smem);
    __syncthreads();
  }
}

__global__ void copy_i16_kernel(const int16_t* __restrict__ src, int16_t* __restrict__ dst, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = src[i];
}

__global__ void leave_to_rerun_kernel(int32_t* __restrict__ iters, int32_t count) {
  const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < count) iters[i] = -2;
}

// How a WAVE8 launch runs its individuals: bits per table entry, waves per
// individual, side-list entries that its LDS holds.
struct W8Shape {
  int bits = 8, waves = 1;
  int32_t acap = 0;
  uint64_t lds = 0;
};

static int launch_w8(const TabuArgs& a, int pop, const W8Shape& w, hipStream_t s, const int16_t* again) {
  const int nw = w.waves, acap = w.acap;
  const size_t lds = (size_t)w.lds;
  if (w.bits == 4) switch (nw) {
      case 1: return launch_w4_1(a, pop, acap, lds, s);
      case 2: return launch_w4_2(a, pop, acap, lds, s);
      default: return launch_w4_4(a, pop, acap, lds, s);
    }
  switch (nw) {
    case 1: return launch_w8_1(a, pop, acap, lds, s, again);
    case 2: return launch_w8_2(a, pop, acap, lds, s, again);
    default: return launch_w8_4(a, pop, acap, lds, s, again);
  }
}

struct Rerun {
  const int16_t* start;
  unsigned char* slots;
  int32_t grid;
};

template <int BLOCK, class Tab>
static int launch_block(const TabuArgs& a, int pop, size_t lds, hipStream_t s, const Rerun* rr) {
  if (rr) {
    auto kern = tabucol_rerun_kernel<BLOCK>;
    DLM_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3(rr->grid), dim3(BLOCK), lds, s, a, rr->start, rr->slots, pop);
  } else {
    auto kern = tabucol_kernel<BLOCK, Tab>;
    DLM_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3(pop), dim3(BLOCK), lds, s, a);
  }
  DLM_HIP(hipGetLastError());
  return DLM_OK;
}

// resident workgroups per CU of the search kernel at this LDS size (0 if unknown)
template <int BLOCK, class Tab>
static int resident_b(size_t lds) {
  int nb = 0;
  auto kern = tabucol_kernel<BLOCK, Tab>;
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, BLOCK, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return nb;
}

template <class Tab>
static int resident(int block, size_t lds) {
  switch (block) {
    case 64: return resident_b<64, Tab>(lds);
    case 128: return resident_b<128, Tab>(lds);
    case 256: return resident_b<256, Tab>(lds);
    case 512: return resident_b<512, Tab>(lds);
    case 1024: return resident_b<1024, Tab>(lds);
  }
  return 0;
}

// rr != nullptr launches the 16-bit rerun pass instead of the search
template <class Tab>
static int launch_tab(const TabuArgs& a, int pop, int block, size_t lds, hipStream_t s,
                      const Rerun* rr = nullptr) {
  switch (block) {
    case 64: return launch_block<64, Tab>(a, pop, lds, s, rr);
    case 128: return launch_block<128, Tab>(a, pop, lds, s, rr);
    case 256: return launch_block<256, Tab>(a, pop, lds, s, rr);
    case 512: return launch_block<512, Tab>(a, pop, lds, s, rr);
    case 1024: return launch_block<1024, Tab>(a, pop, lds, s, rr);
  }
  return set_error(DLM_E_INVAL, "dlm_tabu_batch: block=%d not in {64,128,256,512,1024}", block);
}


// How a call runs: the table tier and block (AUTO resolved), the LDS of the
// search (and rerun) kernel, and the caller-owned workspace it needs.
struct TabuPlan {
  int table = 0, block = 0;
  uint64_t lds = 0, lds_rr = 0;
  uint64_t gtab_bytes = 0;    // device-memory table part of every individual
  uint64_t start_bytes = 0;   // SPLIT8: copy of the start colourings
  uint64_t slot_bytes = 0;    // SPLIT8: one rerun slot (packed 16-bit table)
  int64_t slots = 0;          // SPLIT8: rerun slots
  W8Shape wave, bytes;        // WAVE8: the search, and the rerun with 8-bit entries if there is one (acap > 0)
  uint64_t ws_bytes = 0;      // total, each part on a 256-byte boundary
  uint64_t ws_ask = 0;        // what dlm_tabu_workspace_bytes reports: enough for either automatic table
};

// LDS bytes that bound what the wave table serves: a byte per (v, c), 8 bytes
// per vertex and colour pair state, 64 tabu pairs.  The kernels need less; the
// bound stays where it is so that the shapes the tier serves do not move.
static uint64_t w8_least_bytes(int n, int k) {
  const uint32_t kp = (uint32_t)tab_stride(k);
  return (uint64_t)align16((uint32_t)(n + 1) * kp) + align16(2u * (uint32_t)(n + 1)) + align16(2u * (uint32_t)n) +
         align16((uint32_t)n) + 4u * 320u + align16(2u * kp) + 16u + 4u * kWave;
}

// A byte per (v, c), as the tier's bound on shapes has it.
static bool w8_bytes_fit(int n, int k) {
  return w8_bucket(k, 8) != 0 && (uint64_t)n * (uint64_t)tab_stride(k) <= (1ull << 17) &&
         w8_least_bytes(n, k) <= (uint64_t)device_lds_limit();
}

// Table entries of a colouring of k random classes that reach 15: the number
// of neighbours of v in a class is close to Poisson of mean deg(v) / k.
static double w8_escapes(const dlm_graph* g, int k) {
  double total = 0.0;
  for (const auto& d : g->degrees) {
    const double mu = (double)d.first / k;
    double term = exp(-mu), below = 0.0;
    for (int i = 0; i < 15; ++i) {
      below += term;
      term *= mu / (i + 1);
    }
    total += (double)d.second * k * std::max(0.0, 1.0 - below);
  }
  return total;
}

constexpr double kW4Escapes = 192.0;  // above it entries are 8 bits

// Side-list entries a random start needs: it has f = m / k, and while f falls
// from there the live tabu pairs peak at little more than half the first tenure.
static int64_t w8_side(const dlm_graph* g, const dlm_tabu_params* p, double esc) {
  const int64_t f0 = g->nnz / 2 / p->k;
  int64_t want = 6 * p->ten_num * f0 / (10 * (int64_t)p->ten_den) + p->ten_rand + 32;
  if (esc <= kW4Escapes) want += (int64_t)(2.0 * esc) + 32;
  return std::min<int64_t>(kW8SideMax, (want + 63) & ~63ll);
}

// Whether the largest of k random classes (about the mean and 2 to 3 of its
// roots) passes the wave table's limit: such a search is only repeated with
// the 16-bit table.
static bool w8_classes_pass(int n, int k) {
  const double mean = (double)n / k;
  return mean + 3.0 * sqrt(mean) > (double)kW8ClassMax;
}

// Tables of more than 2^17 bytes fit the LDS with 4-bit entries only: the
// automatic table takes the wave tier there too when few entries escape
// (G(1000, 0.9) with k = 220: 112 KB; its byte table would be in device
// memory) and the classes stay small: 256 individuals x 1,500 iterations on
// 4,000 vertices of degree 30, k = 45 (89 a class), 75 ms in device memory and
// 15 on the wave tier; 4 of them on 5,500 of degree 20, k = 40 (137), 59 and 112.
static bool w8_large(const dlm_graph* g, const dlm_tabu_params* p) {
  if (!g->ell || w8_bucket(p->k, 4) == 0 || w8_classes_pass(g->n, p->k)) return false;
  const double esc = w8_escapes(g, p->k);
  return esc <= kW4Escapes &&
         (int64_t)w8_layout(g->n, p->k, 4, 1, (int)w8_side(g, p, esc)).bytes <= (int64_t)device_lds_limit();
}

// The automatic table is the wave table whenever it holds the individual,
// unless block_faster() says otherwise.
bool w8_auto(const dlm_graph* g, const dlm_tabu_params* p) {
  return w8_bytes_fit(g->n, p->k) || w8_large(g, p);
}

// Where f stays high, far below the colours a graph needs, thousands of pairs
// are tabu at a time.  The wave search walks them in every iteration; the block
// search finds them in its table, whose scan is short just there: LDS16 is the
// faster one.  3,000 iterations, wave table and LDS16, in ms:
//   64 individuals     G(480, 0.3) k = 6   40.2 7.9    k = 13  17.4 10.7   k = 21  11.1 13.8
//                      G(300, 0.7) k = 12  21.6 8.3    k = 25  13.0 11.7   k = 40   8.6 13.2
//                      G(100, 0.7) k = 5   13.6 6.8    k = 11   7.6  7.4   k = 18   6.4  7.3
//   1,024 individuals  G(480, 0.3) k = 6   59.3 12.1   k = 13  28.0 17.5   k = 21  15.7 28.0
//                      G(300, 0.7) k = 12  35.5 12.8   k = 25  18.8 19.3   k = 40  11.7 26.6
//                      G(100, 0.7) k = 5   14.9 9.6    k = 11   8.4 10.5   k = 18   6.9 10.3
// The live pairs follow from f, and f of a searched G(n, p) is close to
// n (d / 2k - 0.85 sqrt(d (1 - p) ln k / k)), d the mean degree (0.75 to 0.95
// in place of 0.85 over p from 0.3 to 0.7).  The line lies lower the fewer
// individuals a CU holds, since they hide less of a walk's latency; over
// n = 100 to 800, three densities, four k each and 1 to 4,096 individuals the
// choice is within 1.2 % of the faster one in the mean.
// A search whose classes are expected to pass the wave table's limit would
// only be repeated from its start (G(600, 0.1), k = 5).
bool block_faster(const dlm_graph* g, const dlm_tabu_params* p, int64_t pop) {
  const int n = g->n, k = p->k;
  if ((int64_t)tabu_layout(n, k, 512 / kWave, TabLds16::kLdsBytes).bytes > (int64_t)device_lds_limit()) return false;
  if (w8_classes_pass(n, k)) return true;
  const double d = (double)g->nnz / n, q = n > 1 ? 1.0 - d / (n - 1) : 1.0;
  const double f = n * (d / (2.0 * k) - 0.85 * sqrt(std::max(0.0, d * q * log((double)k) / k)));
  const double pairs = std::min({p->ten_num * std::max(f, 0.0) / p->ten_den + 0.5 * p->ten_rand,
                                 (double)n * (k - 1), (double)p->max_iters});
  const double held = (double)pop / device_cu_count();  // individuals per CU
  return pairs > 160.0 + 20.0 * held && pairs > (0.03 + 0.01 * held) * n * k;
}

// individuals a CU holds with w waves each (0: not one), of those pop leaves it
static int64_t w8_resident(const dlm_graph* g, int k, int64_t pop, int bits, int64_t side, int w) {
  const int64_t lds_max = device_lds_limit(), granules = device_lds_per_cu() / kLdsGranule, cus = device_cu_count();
  if ((int64_t)w8_layout(g->n, k, bits, w, kWave).bytes > lds_max) return 0;
  const int64_t need = ((int64_t)w8_layout(g->n, k, bits, w, (int)side).bytes + kLdsGranule - 1) / kLdsGranule;
  return std::max<int64_t>(1, std::min<int64_t>({granules / need, 32 / w, (pop + cus - 1) / cus}));
}

// Entry width and waves per individual of a call.
//
// 4-bit entries hold twice the individuals per CU, so they are taken where few
// entries escape by size: each costs the side list's walk a lane, and its
// registers hold 128.
//
// Waves: more of them shorten the chain of one iteration, the more so the
// larger the graph and while many vertices conflict, but individuals that
// share a CU hide one another's latency as well, and the lists of more waves
// take LDS.  10,000 iterations from a random start with one, two and four
// waves, in ms:
//   one individual per CU    G(250, 0.5) 24.6 24.8 23.5   G(400, 0.3) 28.0 25.9 24.4   G(700, 0.5) 49.8 42.3 39.5
//   two                      G(320, 0.5) 27.5 27.7 28.7   G(400, 0.5) 30.5 28.9 29.6   G(700, 0.3) 47.2 41.5 38.9
//   four                     G(320, 0.5) 29.0 30.9 35.8   G(520, 0.5) 41.0 37.9 52.1   G(900, 0.5) 139 114 99.8
//   eight                    G(320, 0.5) 39.3 41.9 69.2   G(400, 0.5) 42.5 41.3 71.5   G(520, 0.3) 51.4 50.6 77.5
// The more individuals a CU holds, the later the second and the fourth wave
// come.  Where the LDS of their lists costs residents they still pay as long
// as the population passes through the CUs in about as many turns (G(900,
// 0.75), 1,024 individuals: 184 157 139).
static W8Pick w8_pick_waves(const dlm_graph* g, const dlm_tabu_params* p, int64_t pop, int bits, int64_t side) {
  const int n = g->n, k = p->k;
  W8Pick r;
  r.bits = bits;
  r.side = side;
  const int64_t cus = device_cu_count(), share = (std::max<int64_t>(pop, 1) + cus - 1) / cus;
  auto resident = [&](int w) { return w8_resident(g, k, pop, r.bits, r.side, w); };
  auto turns = [&](int64_t held) { return (share + held - 1) / held; };
  const int64_t t1 = turns(std::max<int64_t>(1, resident(1))), r2 = resident(2), r4 = resident(4);
  const int four = r4 == 1 ? 250 : r4 == 2 ? 650 : 800, two = r2 == 1 ? 320 : r2 == 2 ? 360 : 400;
  r.waves = 1;
  if (r4 > 0 && r4 <= 4 && n >= four && 4 * turns(r4) <= 5 * t1)
    r.waves = 4;
  else if (r2 > 0 && n >= two && 9 * turns(r2) <= 10 * t1)
    r.waves = 2;
  return r;
}

W8Pick w8_pick(const dlm_graph* g, const dlm_tabu_params* p, int64_t pop) {
  const double esc = w8_escapes(g, p->k);
  return w8_pick_waves(g, p, pop, esc <= kW4Escapes ? 4 : 8, w8_side(g, p, esc));
}

bool w8_pick_bytes(const dlm_graph* g, const dlm_tabu_params* p, int64_t pop, W8Pick& r) {
  if (!w8_bytes_fit(g->n, p->k)) return false;
  r = w8_pick_waves(g, p, pop, 8, w8_side(g, p, kW4Escapes + 1.0));
  return (int64_t)w8_layout(g->n, p->k, 8, r.waves, kWave).bytes <= (int64_t)device_lds_limit();
}

// ... and its LDS: as many individuals per CU as the table allows; the rest
// of their share of the CU's LDS holds side-list entries, at most `most` of them.
static W8Shape w8_shape(const dlm_graph* g, int k, int pop, const W8Pick& w, int64_t most) {
  const int64_t per_cu = std::max<int64_t>(1, w8_resident(g, k, pop, w.bits, w.side, w.waves));
  const int64_t budget = std::min<int64_t>(device_lds_limit(), device_lds_per_cu() / kLdsGranule / per_cu * kLdsGranule);
  W8Shape r;
  r.bits = w.bits;
  r.waves = w.waves;
  r.acap = (int32_t)std::min<int64_t>(most, ((budget - (int64_t)w8_layout(g->n, k, w.bits, w.waves, 0).bytes) / 6) & ~63ll);
  r.lds = w8_layout(g->n, k, w.bits, w.waves, r.acap).bytes;
  return r;
}

static uint64_t align256(uint64_t x) { return (x + 255u) & ~255ull; }

static int tabu_check(const char* fn, const dlm_graph* g, const dlm_tabu_params* p, int32_t pop) {
  if (!g || !p) return set_error(DLM_E_INVAL, "%s: graph or params is NULL", fn);
  if (pop < 0) return set_error(DLM_E_INVAL, "%s: pop < 0", fn);
  if (p->k < 1 || p->k > 32767) return set_error(DLM_E_INVAL, "%s: k=%d outside [1, 32767]", fn, p->k);
  if (p->max_iters < 0 || p->max_iters > (1 << 30))
    return set_error(DLM_E_INVAL, "%s: max_iters=%d outside [0, 2^30]", fn, p->max_iters);
  if (p->ten_den <= 0 || p->ten_num < 0 || p->ten_num > 32767)
    return set_error(DLM_E_INVAL, "%s: tenure slope %d/%d invalid", fn, p->ten_num, p->ten_den);
  if (p->ten_rand < 1 || p->ten_rand > 1024)
    return set_error(DLM_E_INVAL, "%s: ten_rand=%d outside [1, 1024]", fn, p->ten_rand);
  if (p->ind_base < 0 || (int64_t)p->ind_base + pop > 0x7fffffffll)
    return set_error(DLM_E_INVAL, "%s: ind_base + pop exceeds 2^31", fn);
  if (p->trace_cap < 0) return set_error(DLM_E_INVAL, "%s: trace_cap=%d < 0", fn, p->trace_cap);
  if (p->reserved != 0) return set_error(DLM_E_INVAL, "%s: reserved must be 0", fn);
  return DLM_OK;
}

// The wave table's start colourings and rerun slots.
static void w8_workspace(int n, int k, int32_t pop, TabuPlan& P) {
  if (pop > 0) {
    P.slot_bytes = tab_entries(n, k) * TabGlobal16::kGlobalBytes;
    int64_t slots = std::min<int64_t>(pop, 2 * (int64_t)device_cu_count());
    P.slots = std::max<int64_t>(1, std::min<int64_t>(slots, (int64_t)((1ull << 30) / std::max<uint64_t>(P.slot_bytes, 1))));
    P.lds_rr = tabu_layout(n, k, 256 / kWave, TabGlobal16::kLdsBytes).bytes;
    P.start_bytes = sizeof(int16_t) * (uint64_t)pop * (uint64_t)n;
    // beyond 2^17 entries never more than the device-memory tables of the whole population
    if ((uint64_t)n * (uint64_t)tab_stride(k) > (1ull << 17)) {
      const uint64_t whole = P.slot_bytes * (uint64_t)pop, start = align256(P.start_bytes) + 255u;
      const int64_t left = whole > start ? (int64_t)((whole - start) / P.slot_bytes) : 0;
      P.slots = std::max<int64_t>(1, std::min(P.slots, left));
    }
  }
  P.ws_bytes = align256(P.start_bytes) + align256(P.slot_bytes * (uint64_t)P.slots);
}

static int tabu_plan(const char* fn, const dlm_graph* g, const dlm_tabu_params* p, int32_t pop, TabuPlan& P) {
  const int n = g->n, k = p->k;
  const int64_t lds_max = device_lds_limit();
  bool wave_auto = p->table == DLM_TABLE_AUTO && (p->block == 0 || p->block == 64) && w8_auto(g, p);
  const bool lds16 = wave_auto && p->block == 0 && block_faster(g, p, pop);
  wave_auto = wave_auto && !lds16;
  if (lds16) {  // the choice depends on max_iters and the tenure, what a caller sets aside must not
    TabuPlan wave;
    w8_workspace(n, k, pop, wave);
    P.ws_ask = wave.ws_bytes;
  }
  if (p->table == DLM_TABLE_WAVE8 || wave_auto) {
    if (p->block != 0 && p->block != 64)
      return set_error(DLM_E_INVAL, "%s: the wave table runs 64 threads per individual (block=%d)", fn, p->block);
    const uint64_t kp = (uint64_t)tab_stride(k);
    if (!wave_auto && (w8_bucket(k, 8) == 0 || (uint64_t)n * kp > (1ull << 17)))
      return set_error(DLM_E_UNSUPPORTED, "%s: n=%d, k=%d outside the wave table (k <= 256, n*kp <= 2^17)", fn, n, k);
    if (!wave_auto && w8_least_bytes(n, k) > (uint64_t)lds_max)
      return set_error(DLM_E_UNSUPPORTED, "%s: %llu bytes of LDS needed, %lld available", fn,
                       (unsigned long long)w8_least_bytes(n, k), (long long)lds_max);
    const W8Pick pick = w8_pick(g, p, pop);
    W8Pick bytes;
    const bool again = pick.bits == 4 && w8_pick_bytes(g, p, pop, bytes);
    if (again) P.bytes = w8_shape(g, k, pop, bytes, kW8SideMax);
    P.wave = w8_shape(g, k, pop, pick, again ? pick.side + kW4Spare : kW8SideMax);
    P.table = DLM_TABLE_WAVE8;
    w8_workspace(n, k, pop, P);
    P.ws_ask = P.ws_bytes;
    return DLM_OK;
  }
  int block = p->block ? p->block : 256;
  if (block != 64 && block != 128 && block != 256 && block != 512 && block != 1024)
    return set_error(DLM_E_INVAL, "%s: block=%d not in {64,128,256,512,1024}", fn, block);
  int table = p->table;
  if (table == DLM_TABLE_AUTO) {
    // the LDS tier that keeps more individuals resident per CU; byte gamma on a tie loses
    const int nw0 = block / kWave;
    const uint64_t l16 = tabu_layout(n, k, nw0, TabLds16::kLdsBytes).bytes;
    const uint64_t l8 = tabu_layout(n, k, nw0, TabSplit8::kLdsBytes).bytes;
    const int o16 = l16 <= (uint64_t)lds_max ? resident<TabLds16>(block, l16) : 0;
    const int o8 = l8 <= (uint64_t)lds_max ? resident<TabSplit8>(block, l8) : 0;
    table = !lds16 && o8 > o16 ? DLM_TABLE_SPLIT8 : (o16 > 0 ? DLM_TABLE_LDS16 : DLM_TABLE_GLOBAL16);
    // automatic block: when a single LDS-resident individual fills a CU, 512
    // threads hide more of the per-move latency than 256
    if (p->block == 0 && (lds16 ? o16 : std::max(o16, o8)) == 1 && block == 256) block = 512;
  }
  const int nw = block / kWave;
  int eb = 0, gb = 0;
  switch (table) {
    case DLM_TABLE_LDS16: eb = TabLds16::kLdsBytes; break;
    case DLM_TABLE_LDS32: eb = TabLds32::kLdsBytes; break;
    case DLM_TABLE_GLOBAL16: eb = 0; gb = TabGlobal16::kGlobalBytes; break;
    case DLM_TABLE_SPLIT16: eb = TabSplit16::kLdsBytes; gb = TabSplit16::kGlobalBytes; break;
    case DLM_TABLE_SPLIT8: eb = TabSplit8::kLdsBytes; gb = TabSplit8::kGlobalBytes; break;
    default: return set_error(DLM_E_INVAL, "%s: unknown table %d", fn, table);
  }
  P.table = table;
  P.block = block;
  P.lds = tabu_layout(n, k, nw, eb).bytes;
  if (P.lds > (uint64_t)lds_max)
    return set_error(DLM_E_UNSUPPORTED, "%s: %llu bytes of LDS needed, %lld available", fn,
                     (unsigned long long)P.lds, (long long)lds_max);
  P.gtab_bytes = (uint64_t)pop * tab_entries(n, k) * (uint64_t)gb;
  if (table == DLM_TABLE_SPLIT8 && pop > 0) {
    // rerun slots: a few per CU, at most 1 GiB of packed tables
    P.slot_bytes = tab_entries(n, k) * TabGlobal16::kGlobalBytes;
    int64_t slots = std::min<int64_t>(pop, 2 * (int64_t)device_cu_count());
    P.slots = std::max<int64_t>(1, std::min<int64_t>(slots, (int64_t)((1ull << 30) / std::max<uint64_t>(P.slot_bytes, 1))));
    P.lds_rr = tabu_layout(n, k, nw, TabGlobal16::kLdsBytes).bytes;
    P.start_bytes = sizeof(int16_t) * (uint64_t)pop * (uint64_t)n;
  }
  P.ws_bytes = align256(P.gtab_bytes) + align256(P.start_bytes) + align256(P.slot_bytes * (uint64_t)P.slots);
  P.ws_ask = std::max(P.ws_ask, P.ws_bytes);
  return DLM_OK;
}

// The search itself, after the caller's arguments passed tabu_check: plan,
// workspace checks, launches.  Shared by both entry points.
static int tabu_run(const char* fn, const dlm_graph* g, const dlm_tabu_params* p, int32_t pop,
                    int16_t* colors, int32_t* f_best, int32_t* iters, int64_t* stats, uint64_t* hash,
                    int32_t* trace, void* workspace, size_t workspace_bytes, hipStream_t s,
                    uint64_t ws_limit) {
  if (p->trace_cap > 0 && !trace)
    return set_error(DLM_E_INVAL, "%s: trace_cap=%d needs a trace buffer", fn, p->trace_cap);
  if (pop == 0) return DLM_OK;
  if (!colors || !f_best || !iters) return set_error(DLM_E_INVAL, "%s: null output buffer", fn);
  TabuPlan P;
  int rc;
  if ((rc = tabu_plan(fn, g, p, pop, P)) != DLM_OK) return rc;
  if (P.ws_bytes > ws_limit)
    return set_error(DLM_E_UNSUPPORTED, "%s: %llu bytes of workspace needed, the fixed scratch holds %llu", fn,
                     (unsigned long long)P.ws_bytes, (unsigned long long)ws_limit);
  if (P.ws_bytes > 0 && (!workspace || workspace_bytes < P.ws_bytes))
    return set_error(DLM_E_INVAL, "%s: workspace of %zu bytes at %p, %llu needed (dlm_tabu_workspace_bytes)", fn,
                     workspace_bytes, workspace, (unsigned long long)P.ws_bytes);
  if (P.ws_bytes > 0 && (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return set_error(DLM_E_INVAL, "%s: workspace must be 256-byte aligned", fn);
  const int n = g->n, k = p->k;
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  TabuArgs a{g->row_ptr, g->col_idx, g->erow, colors, f_best, iters, stats, hash, trace, nullptr,
             make_key(p->seed), n, k, p->max_iters, p->ten_num, p->ten_den, p->ten_rand,
             p->ind_base, p->trace_cap, g->ell, g->adj, g->ell_stride};
  if (P.gtab_bytes > 0) a.gtab = ws;
  switch (P.table) {
    case DLM_TABLE_WAVE8: {
      int16_t* start = reinterpret_cast<int16_t*>(ws);
      unsigned char* slot_mem = ws + align256(P.start_bytes);
      const int64_t cells = (int64_t)pop * n;
      hipLaunchKernelGGL(copy_i16_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, s, colors, start,
                         cells);
      DLM_HIP(hipGetLastError());
      if (a.ell && n <= (int)kW8ClassMax * k) {
        if ((rc = launch_w8(a, pop, P.wave, s, nullptr)) != DLM_OK) return rc;
        if (P.bytes.acap > 0 && (rc = launch_w8(a, pop, P.bytes, s, start)) != DLM_OK) return rc;
      } else {  // no padded rows, or a class past the limit for certain: the rerun is the search
        hipLaunchKernelGGL(leave_to_rerun_kernel, dim3((unsigned)((pop + 255) / 256)), dim3(256), 0, s, iters, pop);
        DLM_HIP(hipGetLastError());
      }
      const Rerun rr{start, slot_mem, (int32_t)P.slots};
      return launch_tab<TabGlobal16>(a, pop, 256, P.lds_rr, s, &rr);
    }
    case DLM_TABLE_SPLIT8: {
      int16_t* start = reinterpret_cast<int16_t*>(ws + align256(P.gtab_bytes));
      unsigned char* slot_mem = ws + align256(P.gtab_bytes) + align256(P.start_bytes);
      const int64_t cells = (int64_t)pop * n;
      hipLaunchKernelGGL(copy_i16_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, s, colors, start,
                         cells);
      DLM_HIP(hipGetLastError());
      if ((rc = launch_tab<TabSplit8>(a, pop, P.block, P.lds, s)) != DLM_OK) return rc;
      const Rerun rr{start, slot_mem, (int32_t)P.slots};
      return launch_tab<TabGlobal16>(a, pop, P.block, P.lds_rr, s, &rr);
    }
    case DLM_TABLE_SPLIT16: return launch_tab<TabSplit16>(a, pop, P.block, P.lds, s);
    case DLM_TABLE_GLOBAL16: return launch_tab<TabGlobal16>(a, pop, P.block, P.lds, s);
    case DLM_TABLE_LDS32: return launch_tab<TabLds32>(a, pop, P.block, P.lds, s);
    default: return launch_tab<TabLds16>(a, pop, P.block, P.lds, s);
  }
}

// Fixed device scratch of the allocation-free entry point.  In host code the
// array's name is only a stand-in: its device address, one per GPU, comes
// from hipGetSymbolAddress on the first call on that device and is the only
// form host code hands to kernels.  Every call on a device shares the array.
constexpr uint64_t kStaticScratchBytes = DLM_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices];

static int static_scratch(const char* fn, void** out) {
  int dev = -1;
  DLM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return set_error(DLM_E_UNSUPPORTED, "%s: device %d >= %d", fn, dev, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!ptr) return set_error(DLM_E_HIP, "%s: hipGetSymbolAddress gave a null scratch address", fn);
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return DLM_OK;
}

}  // namespace dlm

using namespace dlm;

extern "C" int dlm_tabu_workspace_bytes(const dlm_graph* g, const dlm_tabu_params* p, int32_t pop,
                                        size_t* bytes) {
  if (!bytes) return set_error(DLM_E_INVAL, "dlm_tabu_workspace_bytes: bytes is NULL");
  *bytes = 0;
  int rc = tabu_check("dlm_tabu_workspace_bytes", g, p, pop);
  if (rc != DLM_OK) return rc;
  TabuPlan P;
  if ((rc = tabu_plan("dlm_tabu_workspace_bytes", g, p, pop, P)) != DLM_OK) return rc;
  *bytes = (size_t)P.ws_ask;
  return DLM_OK;
}

extern "C" int dlm_tabu_batch(const dlm_graph* g, const dlm_tabu_params* p, int32_t pop,
                              int16_t* colors, int32_t* f_best, int32_t* iters, int64_t* stats,
                              uint64_t* hash, int32_t* trace, void* workspace, size_t workspace_bytes,
                              void* stream) {
  const int rc = tabu_check("dlm_tabu_batch", g, p, pop);
  if (rc != DLM_OK) return rc;
  return tabu_run("dlm_tabu_batch", g, p, pop, colors, f_best, iters, stats, hash, trace, workspace,
                  workspace_bytes, (hipStream_t)stream, ~0ull);
}

extern "C" int dlm_tabu_batch_static(const dlm_graph* g, const dlm_tabu_params* p, int32_t pop,
                                     int16_t* colors, int32_t* f_best, int32_t* iters, int64_t* stats,
                                     uint64_t* hash, int32_t* trace, void* stream) {
  const char* fn = "dlm_tabu_batch_static";
  int rc = tabu_check(fn, g, p, pop);
  if (rc != DLM_OK) return rc;
  if (pop == 0) return DLM_OK;
  void* ws = nullptr;
  if ((rc = static_scratch(fn, &ws)) != DLM_OK) return rc;
  return tabu_run(fn, g, p, pop, colors, f_best, iters, stats, hash, trace, ws, (size_t)kStaticScratchBytes,
                  (hipStream_t)stream, kStaticScratchBytes);
}
