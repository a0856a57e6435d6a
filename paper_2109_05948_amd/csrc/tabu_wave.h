// TabuCol with one to four wavefronts per individual and a 4- or 8-bit table
// entry per (vertex, colour) (the WAVE8 table tier).
//
// Per individual, all in LDS:
//   tab[v][c]   BITS bits: gamma[v][c], or all ones ("escaped") when c is v's
//               current colour, c is a padding colour (c >= k), the pair
//               (v, c) is tabu, or gamma does not fit.  An entry that is not
//               escaped is a move that no tenure forbids, and the smallest
//               entry of a row is the row's best such move.
//   side list   the escaped pairs other than the current and the padding
//               colours, each with its gamma, its expiry and whether it is
//               still tabu.  About 0.6 f + 5 tabu pairs are live at a time, and
//               4-bit tables are taken where few entries reach 15, so the list
//               is walked whole in every iteration: gamma follows the move by
//               v*'s adjacency bits, expired pairs lose their tabu state, and a
//               pair that is neither tabu nor too large returns to the table.
//               128 entries live in registers of the last wave, one or two per
//               lane; the rest in act[] = v << 17 | c << 9 | low 9 bits of the
//               expiry mod 2^17 and actg[] = its high 8 bits << 8 | gamma | 0x80
//               on a pair that is not tabu
//   cg[v]       colour (bits 0..7) | gamma[v][col v] (bits 8..14) |
//               "listed" (bit 15)
//   list[w]     per wave, the listed vertices it scans: every conflicting
//               vertex is in one wave's list once, beside vertices that
//               stopped conflicting ("stale", compacted away when they cost a
//               scan round)
//   stage[w]    rows at the wave's best delta
//   slot[w]     the wave's best move
//   The colour class sizes live in registers of every wave (gamma <= class
//   size <= 127 fits seven bits).  A run that would pass it, or that finds no
//   room in a list, gives up with iters = -2.  What 4-bit entries gave up on is
//   run again with 8-bit entries where the LDS holds those: graphs whose
//   vertices share neighbourhoods fill the table in ways that the rule for 4
//   bits does not foresee (64 individuals x 3,000 iterations on 40 groups of 20
//   vertices, k = 40: 15.0 ms without that run, 4.2 with it, 3.5 in bytes at once).  What is left is
//   run with the 16-bit device table.  (One code for every reason: two of them
//   moved the code about and cost one wave 2 %.)
//
// One iteration, two barriers (none for a single wave):
//   scan   lane i takes list entry i of its wave (64 per round) and reads its
//          row: the smallest entry in packed 16-bit minima whose top bits are
//          the entries; the last wave adds the side list's admissible pairs;
//   ties   the rows at the wave's minimum (DPP) are staged and read again, one
//          dword per lane; each lane hashes its tied moves (Philox);
//   fold   the waves publish (delta, hash, v, c); after the barrier each folds
//          the slots to the smallest;
//   apply  the neighbours of v* (16-bit padded rows in device memory) are split
//          over the waves; a neighbour's row and cg word belong to one lane;
//          the last wave also writes v*'s state and walks the side list.
//
// What bounds it: one wave's chain of dependent steps.  G(500, 0.5), k = 49,
// eight individuals of one wave per CU: 518 vector, 288 scalar and 57 memory
// instructions in 7,500 cycles a move, half of them the wave's own issue, the
// rest latency (36 %) and the other wave of the SIMD.  G(1000, 0.5), k = 85, two
// of four waves: 12,000 cycles, the waves waiting 57 % of them for one another
// or for memory.  Measured here, in cycles: a vector operation 4, an LDS read 57, a neighbour row from the L2
// about 200, a vector result brought to the scalar unit 31, a branch on it
// 52, a lane-masked block 44.  So Philox (about 190) is cheaper than avoiding
// it, and the code selects addresses and values instead of branching.
#pragma once

#include <type_traits>

#include "tabu_body.h"
#include "wave_util.h"

namespace dlm {

constexpr uint32_t kW8ClassMax = 127u;
constexpr uint32_t kW8None = 255u;        // biased delta (delta + 128) of "no admissible move"
constexpr uint32_t kW8ExpMask = 0x1ffffu;  // expiries are kept modulo 2^17: no tenure reaches it (32,757 + 1,023)
constexpr uint32_t kW8NoKey = 0xffffffffu;
constexpr uint32_t kW8Free = 0x80u;  // gamma of a side-list pair: not tabu
constexpr int kW8GaveUp = -2;        // iters of a search that is left to a rerun
constexpr int kW8Stage = 128;        // tied rows a wave stages: up to 64 waiting and 64 more
constexpr int kW8Mail = 64;          // entries that can escape by growth in one move

struct W8Layout {
  uint32_t tab, cg, list, stage, slot, mail, act, actg, bytes;
};

__host__ __device__ constexpr int w8_row_dwords(int k, int bits) { return (k * bits + 31) >> 5; }

// Vertices one wave's list holds: all of them for one wave.  Several waves
// start with equal shares, and rows of many neighbours keep them so; what joins
// by rows of up to 16 neighbours joins wave 0.  Half of the vertices and 64 is
// room enough in earnest (G(450, 0.03), four waves: lists of 121, 50, 64 and 63
// in the mean); a list that is full all the same leaves the individual to a rerun.
__host__ __device__ constexpr int w8_list_cap(int n, int nw) { return nw == 1 || n / 2 + 64 > n ? n : n / 2 + 64; }

// LDS of one individual searched by nw waves, with room for acap side-list
// entries (a multiple of 64).  A row read covers up to RW dwords; reads past
// the last row land in the arrays that follow the table.  list and stage,
// adjacent, are the scratch of the construction.  Two rows follow the
// vertices', all escaped: n, read by scan lanes without a vertex, and n + 1,
// where the ends of neighbour rows point.
__host__ __device__ inline W8Layout w8_layout(int n, int k, int bits, int nw, int acap) {
  W8Layout L;
  uint32_t o = 0;
  L.tab = o;
  o += align16(4u * (uint32_t)(n + 2) * (uint32_t)w8_row_dwords(k, bits));
  L.cg = o;
  o += align16(2u * (uint32_t)(n + 2));
  L.list = o;  // one entry more than a list holds: where lanes without a vertex to append write
  o += (uint32_t)nw * align16(2u * (uint32_t)(w8_list_cap(n, nw) + 1));
  L.stage = o;  // one entry more than kW8Stage: where lanes without a tied row write
  o += (uint32_t)nw * 4u * (kW8Stage + 4);
  L.slot = o;  // 16 bytes per wave, then "give up" and the mail count
  o += 16u * ((uint32_t)nw + 1u);
  L.mail = o;
  o += bits == 8 ? 0u : 4u * kW8Mail;
  L.act = o;  // one entry more than acap: where lanes without an entry write
  o += 4u * (uint32_t)acap + 4u;
  L.actg = o;
  o += 2u * (uint32_t)acap + 12u;
  L.bytes = o;
  return L;
}

// dwords a kernel reads per row: exact up to 12, then buckets (0: k > 256)
__host__ __device__ constexpr int w8_bucket(int k, int bits) {
  const int w = w8_row_dwords(k, bits);
  return k > 256 ? 0 : w <= 12 ? w : w <= 16 ? 16 : w <= 24 ? 24 : w <= 32 ? 32 : 64;
}

typedef unsigned short w8_u16x2 __attribute__((ext_vector_type(2)));

// per 16-bit half minimum (one v_pk_min_u16)
__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b) {
  const w8_u16x2 x = __builtin_bit_cast(w8_u16x2, a), y = __builtin_bit_cast(w8_u16x2, b);
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(x, y));
}

// Barrier of the waves that share an individual.
template <int NW>
__device__ __forceinline__ void team_sync() {
  if constexpr (NW == 1)
    wave_sync();
  else
    __syncthreads();
}

// The conflicting vertices of every NW-th group of 64, in vertex order, as
// this wave's list; sets "listed" on exactly those.  Returns the list length.
template <int NW>
__device__ __forceinline__ int w8_build_list(uint16_t* cg, uint16_t* list, int n, int wid, int lane) {
  int base = 0;
  for (int v0 = wid * kWave; v0 < n; v0 += NW * kWave) {
    const int v = v0 + lane;
    const uint32_t x = v < n ? (uint32_t)cg[v] : 0u;
    const bool cf = ((x >> 8) & 0x7fu) != 0u;
    const uint64_t m = __ballot(cf);
    if (cf) {
      cg[v] = (uint16_t)(x | 0x8000u);
      list[base + (int)lane_rank(m)] = (uint16_t)v;
    }
    base += __popcll(m);
  }
  return base;
}

// Drops the stale entries (vertices no longer conflicting) from a wave's list
// in place and clears their "listed" bit.  Returns the new length.
__device__ __forceinline__ int w8_compact_list(uint16_t* cg, uint16_t* list, int len, int lane) {
  int base = 0;
  for (int i0 = 0; i0 < len; i0 += kWave) {
    const int i = i0 + lane;
    const uint32_t v = i < len ? (uint32_t)list[i] : 0u;
    const uint32_t x = i < len ? (uint32_t)cg[v] : 0u;
    const bool keep = ((x >> 8) & 0x7fu) != 0u;
    if (i < len && !keep) cg[v] = (uint16_t)(x & 0x7fffu);
    lanes_joined();
    const uint64_t m = __ballot(keep);
    if (keep) list[base + (int)lane_rank(m)] = (uint16_t)v;  // base <= i0: entries are read before they are overwritten
    lanes_joined();
    base += __popcll(m);
  }
  return base;
}

// f(groups, first) over the 64-entry groups of a list: G at a time, whose
// loads are then issued together, while more than one is left.
template <int G, class F>
__device__ __forceinline__ void for_groups(int len, F f) {
  int i = 0;
  for (; len - i > kWave; i += G * kWave) f(std::integral_constant<int, G>{}, i);
  if (i < len) f(std::integral_constant<int, 1>{}, i);
}

// One individual (row li of a.colors) searched by the NW waves of the calling
// workgroup.  RW: dwords read per row, of which the first RLO lie in every row
// the kernel serves; acap: side-list entries the LDS holds; late(): the
// argument block again, read where its fields are needed late and rarely.
template <int BITS, int NW, int RW, int RLO, class Late>
__device__ __forceinline__ void tabu_w8_individual(const TabuArgs& a, int li, int acap, unsigned char* smem, Late late) {
  constexpr int BLOCK = NW * kWave;
  constexpr uint32_t PER = 32u / BITS, ESC = (1u << BITS) - 1u;  // entries per dword, the escaped entry
  constexpr uint32_t ONES = BITS == 4 ? 0x11111111u : 0x01010101u;
  constexpr uint32_t LOW = ONES * (ESC >> 1), TOP = ~LOW;  // the lower bits and the top bit of every entry
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wid = NW == 1 ? 0 : (int)rfl((uint32_t)tid / kWave);
  const bool tail_wave = wid == NW - 1;  // keeps v*'s state and the side list
  // every field the search needs, as a value of its own: the argument block
  // as a whole (about 30 scalar registers) would otherwise stay live in, and
  // spill from, scalar registers
  const uint32_t ind = own_u32((uint32_t)(a.ind_base + li));
  const int n = (int)own_u32((uint32_t)a.n), k = (int)own_u32((uint32_t)a.k);
  const uint32_t rw = (uint32_t)w8_row_dwords(k, BITS), kp = rw * PER;
  const gptr<const uint16_t> ell = own_sgpr(a.ell);
  const gptr<const uint32_t> adj = own_sgpr(a.adj);
  const uint32_t stride = own_u32((uint32_t)a.ell_stride), aw = 2u * (((uint32_t)n >> 6) + 1u);
  const int trace_cap = (int)own_u32((uint32_t)(a.trace ? a.trace_cap : 0)), T = (int)own_u32((uint32_t)a.T);
  const Key key{own_u32(a.key.k0), own_u32(a.key.k1)};
  const uint32_t ten_num = own_u32((uint32_t)a.ten_num), ten_den = own_u32((uint32_t)a.ten_den);
  const uint32_t ten_rand = own_u32((uint32_t)a.ten_rand);
  const uint32_t den_inv = 0xffffffffu / ten_den;
  const W8Layout L = w8_layout(n, k, BITS, NW, acap);
  uint32_t* tabw = reinterpret_cast<uint32_t*>(smem + L.tab);
  uint16_t* cg = reinterpret_cast<uint16_t*>(smem + L.cg);
  uint16_t* list = reinterpret_cast<uint16_t*>(smem + L.list + (uint32_t)wid * align16(2u * (uint32_t)(w8_list_cap(n, NW) + 1)));
  const int lcap = w8_list_cap(n, NW);
  uint32_t* stage = reinterpret_cast<uint32_t*>(smem + L.stage + (uint32_t)wid * 4u * (kW8Stage + 4));
  uint4* slot = reinterpret_cast<uint4*>(smem + L.slot);
  // "give up" is written between the fold's barrier and the iteration's last
  // one, and read by every wave before the next fold
  uint32_t* full = reinterpret_cast<uint32_t*>(smem + L.slot + 16u * NW);
  uint32_t* mailn = full + 1;
  uint32_t* mail = reinterpret_cast<uint32_t*>(smem + L.mail);
  uint32_t* act = reinterpret_cast<uint32_t*>(smem + L.act);
  uint16_t* actg = reinterpret_cast<uint16_t*>(smem + L.actg);
  const gptr<int16_t> gcol = own_sgpr(a.colors + (size_t)li * n);
  const __attribute__((address_space(4))) int32_t* row_c =
      (const __attribute__((address_space(4))) int32_t*)(const int32_t*)own_sgpr(a.row_ptr);
  // tie pass: one dword per lane, rpp rows per pass; this lane's row within a pass and its dword
  const int rpp = kWave / (int)rw;
  const int lrow = lane / (int)rw, lj = lane - lrow * (int)rw;
  auto shift = [&](uint32_t c) { return BITS * (c & (PER - 1u)); };  // of entry c within its dword c / PER
  // Written by every lane: a lane-masked store here would meet the search
  // loop's end in one block, and the compiler would then keep the loop's
  // uniform values (f, t, the lists' lengths) in vector registers.
  auto give_up = [&]() { late()->iters[li] = kW8GaveUp; };

  // 1. start colouring (rejected whole if a colour is outside [0, k)), class sizes
  int bad = 0;
  for (int v = tid; v < n; v += BLOCK) {
    const int c = gcol[v];
    bad |= (c < 0) | (c >= k);
    cg[v] = (uint16_t)(c & 0xff);
  }
  uint32_t* scr = reinterpret_cast<uint32_t*>(smem + L.list);
  for (int i = tid; i < k; i += BLOCK) reinterpret_cast<uint16_t*>(scr)[i] = 0;
  for (int i = tid; i < 2 * (int)rw; i += BLOCK) tabw[(uint32_t)n * rw + (uint32_t)i] = 0xffffffffu;
  if (tid == 0) {
    cg[n] = 0;
    cg[n + 1] = 0x80ffu;  // "listed": never appended
    *full = 0u;
    *mailn = 0u;
  }
  team_sync<NW>();
  if (__ballot(bad) && lane == 0) *full = 1u;
  team_sync<NW>();
  if (rfl(*full)) {
    if (tid == 0) {
      a.f_best[li] = -1;
      a.iters[li] = -1;
    }
    return;
  }
  for (int v = tid; v < n; v += BLOCK) {
    const uint32_t c = cg[v];
    atomicAdd(&scr[c >> 1], 1u << (16u * (c & 1u)));
  }
  team_sync<NW>();
  constexpr int NR = ((int)PER * RW + kWave - 1) / kWave;
  uint32_t cz[NR];  // size of class lane + 64 r
  {
    uint32_t big = 0u;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int c = lane + kWave * r;
      cz[r] = c < k ? (uint32_t)reinterpret_cast<uint16_t*>(scr)[c] : 0u;
      big = max(big, cz[r]);
    }
    if (__ballot(big > kW8ClassMax)) {  // every wave looks at every class: uniform
      give_up();
      return;
    }
  }
  team_sync<NW>();
  // 2. the table, a chunk of vertices at a time: gamma in bytes from the CSR
  // entries into the scratch, then packed; entries that do not fit join the side list
  uint32_t fs = 0;
  {
    const uint32_t sw = (kp + 3u) >> 2;  // scratch dwords per vertex
    const int rows = (int)((L.slot - L.list) / (4u * sw));
    for (int v0 = 0; v0 < n; v0 += rows) {
      const int v1 = min(n, v0 + rows);
      for (int i = tid; i < (v1 - v0) * (int)sw; i += BLOCK) scr[i] = 0u;
      team_sync<NW>();
      const int e1 = row_c[v1];
      for (int e = row_c[v0] + tid; e < e1; e += BLOCK) {
        const uint32_t c = (uint32_t)cg[a.col_idx[e]] & 0xffu;
        atomicAdd(&scr[(uint32_t)(a.erow[e] - v0) * sw + (c >> 2)], 1u << (8u * (c & 3u)));
      }
      team_sync<NW>();
      for (int i = tid; i < (v1 - v0) * (int)rw; i += BLOCK) {
        const int r = i / (int)rw, q = i - r * (int)rw;
        const uint32_t v = (uint32_t)(v0 + r), cv = (uint32_t)cg[v] & 0xffu;
        uint32_t w = 0u;
#pragma unroll
        for (uint32_t b = 0; b < PER; ++b) {
          const uint32_t c = PER * (uint32_t)q + b;
          uint32_t g = (scr[(uint32_t)r * sw + (c >> 2)] >> (8u * (c & 3u))) & 0xffu;
          if (c == cv) {
            cg[v] = (uint16_t)(cv | (g << 8));
            fs += g;
            g = ESC;
          } else if (c >= (uint32_t)k) {
            g = ESC;
          } else if (g >= ESC) {
            const uint32_t p = atomicAdd(mailn, 1u);
            if (p < (uint32_t)acap) {
              act[p] = (v << 17) | (c << 9);
              actg[p] = (uint16_t)(g | kW8Free);
            }
            g = ESC;
          }
          w |= g << (BITS * b);
        }
        tabw[v * rw + (uint32_t)q] = w;
      }
      team_sync<NW>();
    }
  }
  int A = (int)rfl(*mailn);  // side-list entries in act (the tail wave's count)
  if (A > acap) {
    give_up();
    return;
  }
  // 3. f = half the sum of the own gammas
  fs = wave_sum_u32(fs);
  if constexpr (NW > 1) {
    if (lane == 0) slot[wid].x = fs;
  }
  team_sync<NW>();
  if constexpr (NW > 1) {
    fs = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) fs += rfl(slot[w].x);
  }
  int f = (int)(fs >> 1);
  if (tid == 0) *mailn = 0u;
  int len = w8_build_list<NW>(cg, list, n, wid, lane);
  // a longer list is compacted: stale entries cost a scan round; so is any
  // list of several rounds every 64 iterations, since conflicts get fewer
  int len_max = max(64, (len + 63) & ~63);
  team_sync<NW>();

  int t = 0, f_best = f;
  bool best_cur = true;
  // statistics (st_conf per lane) and fingerprint; moves = t - no-ops
  uint64_t st_conf = 0, st_deg = 0, fp = kFnvOffset;
  uint32_t st_noops = 0, st_ties = 0, st_cap = 0;
  const bool l0 = lane == 0;
  uint32_t Lreg = 0;
  bool spill = false;  // the tail wave could not take an entry
  bool mailed = false;  // entries wait in mail (one wave: known without a look)
  const RoundKeys rk = round_keys(key);
  // the tail wave's register part of the side list: vertex, colour, expiry mod
  // 2^17, gamma | kW8Free; a free lane holds vertex n and a colour that matches nothing
  constexpr int NB = 2;
  constexpr uint32_t kNoColour = 0xfffeu;
  uint32_t sv[NB], sc[NB], sx[NB], sg[NB];
  uint64_t room[NB];  // free lanes
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    sv[b] = (uint32_t)n;
    sc[b] = kNoColour;
    sx[b] = 0u;
    sg[b] = 0u;
    room[b] = ~0ull;
  }
  // Groups of the LDS part that the scan looks at together: a long list (f stays
  // high with far too few colours) is walked in every iteration, one round trip
  // to the LDS after the other, and the tie pass walks it only if a pair of it is
  // at the best delta.  An uneven batch of 12 graphs of 100 to 1,000 vertices:
  // 101.7 ms one group at a time, 95.5 two at a time, 80.4 with the tie pass
  // skipped as well.  (Four at a time, and the walk after the move by groups, gave
  // no more and cost short lists 2 to 3 %.)  With one or two waves per individual
  // the registers it takes cost short lists 2 to 5 %, and long ones are rarer there.
  constexpr int GROUPS = NW == 4 ? 2 : 1;
  auto refill = [&]() {  // from the end of act
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int rank = (int)lane_rank(room[b]);
      const bool get = ((room[b] >> lane) & 1ull) != 0ull && rank < A;
      const int i = get ? A - 1 - rank : acap;
      const uint32_t e = act[i], g = actg[i];
      sv[b] = get ? e >> 17 : sv[b];
      sc[b] = get ? (e >> 9) & 0xffu : sc[b];
      sx[b] = get ? (e & 0x1ffu) | ((g >> 8) << 9) : sx[b];
      sg[b] = get ? g & 0xffu : sg[b];
      const uint64_t got = __ballot(get);
      A -= __popcll(got);
      room[b] &= ~got;
    }
  };

  while (t < T && f > 0) {
    if ((t & 63) == 0) {
      if (rfl(*full)) {  // an entry was lost: left to a rerun
        give_up();
        return;
      }
      if (tail_wave) {
        Lreg = lemire(philox_w0_rk(ind, (uint32_t)(t + lane), 0u, kDomTenure, rk), ten_rand);
        if (A > 0) refill();
      }
    }
    uint32_t mails = 0u;
    if (BITS == 4 && NW > 1 && tail_wave) mails = *mailn;
    if (len > ((t & 63) != 0 ? len_max : 64)) {
      wave_sync();
      len = w8_compact_list(cg, list, len, lane);
      len_max = max(64, (len + 63) & ~63);
      wave_sync();
    }

    // ---- scan: list entry (r << 6) + lane in round r.  Biased deltas
    // (delta + 128) of the first eight rounds stay in dp0 (rounds 0..3) and dp1
    const int rounds = (len + 63) >> 6;
    uint32_t best = kW8None, dp0 = 0u, dp1 = 0u, vlast = (uint32_t)n, xlast = 0u, dlast = kW8None;
    uint32_t conf = 0u;
    for (int r = 0; r < rounds; ++r) {
      const int i = (r << 6) + lane;
      const uint32_t v0 = list[min(i, len - 1)];
      const uint32_t v = i < len ? v0 : (uint32_t)n;
      const uint32_t x = cg[v], g = (x >> 8) & 0x7fu;
      const uint32_t* row = tabw + __umul24(v, rw);
      uint32_t w[RW];
#pragma unroll
      for (int q = 0; q < RW; ++q) w[q] = row[q];
      conf += g != 0u ? 1u : 0u;
      // the entries at the top of each 16-bit half of w, w << BITS, ...: the
      // packed minima's top bits are the smallest entries
      uint32_t mn[16 / BITS];
#pragma unroll
      for (int j = 0; j < 16 / BITS; ++j) mn[j] = 0xffffffffu;
#pragma unroll
      for (int q = 0; q < RW; ++q) {
        if (q >= RLO && q >= (int)rw) w[q] = 0xffffffffu;
#pragma unroll
        for (int j = 0; j < 16 / BITS; ++j) mn[j] = pk_min_u16(mn[j], w[q] << (BITS * j));
      }
#pragma unroll
      for (int j = 1; j < 16 / BITS; ++j) mn[0] = pk_min_u16(mn[0], mn[j]);
      const uint32_t m = min(mn[0] & 0xffffu, mn[0] >> 16) >> (16 - BITS);
      const uint32_t d = (g != 0u && m != ESC) ? m + 128u - g : kW8None;
      if (r < rounds - 1) {
        const uint32_t sh = 8u * (uint32_t)(r & 3);
        dp0 |= r < 4 ? d << sh : 0u;
        dp1 |= r >= 4 && r < 8 ? d << sh : 0u;
      }
      best = min(best, d);
      vlast = v;
      xlast = x;
      dlast = d;
    }
    st_conf += conf;
    // the side list's admissible pairs: not tabu, or aspiring (f + delta < f_best)
    const int aspd = f_best - f - 1;
    auto pair_delta = [&](uint32_t x, uint32_t ga) -> uint32_t {  // 255 or more: not admissible
      const int g = (int)((x >> 8) & 0x7fu), dd = (int)(ga & 0x7fu) - g;
      return g != 0 && (ga >= kW8Free || dd <= aspd) ? (uint32_t)(dd + 128) : kW8None;
    };
    auto act_delta = [&](int i0, uint32_t& v, uint32_t& c, uint32_t& x) -> uint32_t {
      const int i = i0 + lane < A ? i0 + lane : acap;
      const uint32_t e = act[i], ga = actg[i] & 0xffu;
      v = i < acap ? e >> 17 : (uint32_t)n;
      c = (e >> 9) & 0xffu;
      x = cg[v];
      return pair_delta(x, ga);
    };
    auto act_deltas = [&](auto groups, int i0, uint32_t* d) {
      constexpr int U = decltype(groups)::value;
      uint32_t v[U], ga[U], x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + kWave * u + lane < A ? i0 + kWave * u + lane : acap;
        ga[u] = actg[i] & 0xffu;
        v[u] = i < acap ? act[i] >> 17 : (uint32_t)n;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = cg[v[u]];
#pragma unroll
      for (int u = 0; u < U; ++u) d[u] = pair_delta(x[u], ga[u]);
    };
    uint32_t side[NB], sxg[NB], listed = kW8None;  // listed: the LDS part's smallest delta
#pragma unroll
    for (int b = 0; b < NB; ++b) side[b] = kW8None, sxg[b] = 0u;
    if (tail_wave) {
      if (BITS == 4 && (NW > 1 ? rfl(mails) != 0u : mailed)) {  // entries that the last move made escape
        const int got = (int)rfl(*mailn), cnt = min(got, min(kW8Mail, acap - A));
        spill |= cnt < got;
        if (lane < cnt) {
          act[A + lane] = mail[lane] << 9;
          actg[A + lane] = (uint16_t)(ESC | kW8Free);
        }
        lanes_joined();
        A += cnt;
        if (l0) *mailn = 0u;
        lanes_joined();
        mailed = false;
        wave_sync();
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b == 0 || room[b] != ~0ull) {
          sxg[b] = cg[sv[b]];
          side[b] = pair_delta(sxg[b], sg[b]);
          best = min(best, side[b]);
        }
      if constexpr (GROUPS == 1) {
        for (int i0 = 0; i0 < A; i0 += kWave) {
          uint32_t v, c, x;
          best = min(best, act_delta(i0, v, c, x));
        }
      } else {
        for_groups<GROUPS>(A, [&](auto groups, int i0) {
          constexpr int U = decltype(groups)::value;
          uint32_t d[U];
          act_deltas(groups, i0, d);
#pragma unroll
          for (int u = 0; u < U; ++u) listed = min(listed, d[u]);
        });
        best = min(best, listed);
      }
    }
    const uint32_t cur = wave_min_u32(best);

    // ---- the wave's best move: every admissible move at cur, hashed where it is found
    uint32_t vc = 0u, h = 0u, xs = 0u;
    int seen = 0;
    if (cur != kW8None) {
      uint64_t hk = ~0ull;  // hash << 32 | v << 8 | c of this lane's smallest
      uint32_t hx = 0u;     // the cg word of its vertex
      auto hash_move = [&](bool has, uint32_t v, uint32_t c, uint32_t x) {
        const uint64_t y = ((uint64_t)philox_w0_rk(ind, (uint32_t)t, v, c, rk) << 32) | (v << 8) | c;
        const bool lt = has && y < hk;
        hx = lt ? x : hx;
        hk = lt ? y : hk;
      };
      auto scan_rows = [&](int cnt) {
        for (int p0 = 0; p0 < cnt; p0 += rpp) {
          const int ri = p0 + lrow;
          const bool ok = lrow < rpp && ri < cnt;
          const uint32_t e = stage[ok ? ri : 0];
          const uint32_t v = e >> 8;
          const uint32_t y = tabw[__umul24(v, rw) + (uint32_t)lj] ^ (e & 0xffu) * ONES;
          const uint32_t x = cg[v];
          // top bit of an entry set iff it equals the target (below ESC, so escaped entries never match)
          uint32_t z = ok ? ~(((y & LOW) + LOW) | y) & TOP : 0u;
          for (uint64_t b = __ballot(z != 0u); b; b = __ballot(z != 0u)) {
            const uint32_t c = PER * (uint32_t)lj + (((uint32_t)__ffs((int)z) - 1u) / BITS);
            hash_move(z != 0u, v, c, x);
            seen += __popcll(b);
            z &= z - 1u;
          }
        }
      };
      int cnt = 0;
      for (int r = 0; r < rounds; ++r) {
        uint32_t v = vlast, x = xlast, d = dlast;
        if (r != rounds - 1) {
          v = list[(r << 6) + lane];  // full rounds
          x = cg[v];
          const uint32_t dp = (r < 4 ? dp0 : dp1) >> (8 * (r & 3));
          // beyond the rounds kept: any row may be at cur, the comparison below tells
          d = r < 8 ? dp & 0xffu : (((x >> 8) & 0x7fu) != 0u ? cur : kW8None);
        }
        const uint32_t tgt = cur + ((x >> 8) & 0x7fu) - 128u;
        const bool tied = d == cur && tgt < ESC;
        const uint64_t M = __ballot(tied);
        stage[tied ? cnt + (int)lane_rank(M) : kW8Stage] = (v << 8) | tgt;
        cnt += __popcll(M);
        if (cnt > kW8Stage - kWave || r == rounds - 1) {
          wave_sync();
          scan_rows(cnt);
          cnt = 0;
          wave_sync();
        }
      }
      if (tail_wave) {
        // both banks asked at once first: 1 to 2 % of a lone individual's time
        if (__ballot(min(side[0], side[NB - 1]) == cur)) {
#pragma unroll
          for (int b = 0; b < NB; ++b)
            if (const uint64_t m = __ballot(side[b] == cur)) {
              hash_move(side[b] == cur, sv[b], sc[b], sxg[b]);
              seen += __popcll(m);
            }
        }
        for (int i0 = 0; i0 < A; i0 += kWave) {
          if (NW == 4 && i0 == 0 && !__ballot(listed == cur)) break;
          uint32_t v, c, x;
          const uint32_t d = act_delta(i0, v, c, x);
          if (const uint64_t m = __ballot(d == cur)) {
            hash_move(d == cur, v, c, x);
            seen += __popcll(m);
          }
        }
      }
      h = wave_min_u32((uint32_t)(hk >> 32));
      uint64_t at = __ballot((uint32_t)(hk >> 32) == h);
      if (at & (at - 1ull)) {  // equal hashes: the smallest (v, c)
        const uint32_t lo = wave_min_u32((uint32_t)(hk >> 32) == h ? (uint32_t)hk : 0xffffffffu);
        at = __ballot(hk == (((uint64_t)h << 32) | lo));
      }
      const int wl = __builtin_ctzll(at);
      vc = readlane((uint32_t)hk, wl);
      xs = readlane(hx, wl);
    }
    uint32_t dstar = cur;
    bool shared = seen > 1;  // two or more admissible moves at the best delta
    if constexpr (NW > 1) {
      // delta 8 bits, hash 32, v << 8 | c 23 bits, the "more than one" bit
      const uint32_t khi = cur != kW8None ? (cur << 24) | (h >> 8) : 0xffffffffu;
      const uint32_t klo = cur != kW8None ? (h << 24) | (vc << 1) | (seen > 1 ? 1u : 0u) : 0xffffffffu;
      if (l0) slot[wid] = make_uint4(klo, khi, xs, 0u);
      lanes_joined();
      __syncthreads();
      const uint4 e = slot[lane & (NW - 1)];
      const uint64_t kx = ((uint64_t)e.y << 32) | e.x;
      uint64_t km = umin64(kx, ((uint64_t)dpp_mov<dpp::kXor1>(e.y) << 32) | dpp_mov<dpp::kXor1>(e.x));
      if constexpr (NW > 2)
        km = umin64(km, ((uint64_t)dpp_mov<dpp::kXor2>((uint32_t)(km >> 32)) << 32) | dpp_mov<dpp::kXor2>((uint32_t)km));
      xs = readlane(e.z, __builtin_ctzll(__ballot(kx == km)));
      dstar = rfl((uint32_t)(km >> 56));
      const uint32_t lo = rfl((uint32_t)km);
      vc = (lo >> 1) & 0x7fffffu;
      const uint64_t level = __ballot((e.y >> 24) == dstar) & ((1ull << NW) - 1ull);  // waves at the best delta
      shared = (lo & 1u) != 0u || (level & (level - 1ull)) != 0ull;
    }

    uint32_t vs = (uint32_t)n, cs = 0xffffu, old = 0xffffu;  // no move: they match nothing
    int fnew = f, deg = 0;
    bool snap = false;
    if (dstar != kW8None) {
      vs = vc >> 8;
      cs = vc & 0xffu;
      old = xs & 0xffu;
      fnew = f + (int)dstar - 128;
    }
    // ---- apply.  Neighbour u of v*: gamma[u][old] - 1, gamma[u][c*] + 1; if
    // u has colour old or c*, its own gamma and list membership follow.
    // Groups of 16 consecutive neighbours go to the waves in turn, the first to
    // wave 0: the waves share rows of 64 and more evenly, a row of up to 16 is
    // wave 0's alone.  (Turning the first wave with v* evened the lists of sparse
    // graphs out, but changed no time: G(450, 0.03), k = 4, 9.84 and 9.84 ms.)  A
    // row ends in entries n + 1, where nothing changes.
    const uint32_t nrow = 2u * vs * stride, arow = 4u * vs * aw;  // bytes
    auto adj_word = [&](uint32_t v) { return *(gptr<const uint32_t>)((gptr<const char>)adj + (arow + 4u * (v >> 5))); };
    const uint32_t e0 = (uint32_t)(((lane & ~15) * NW) + (wid << 4) + (lane & 15));
    const uint32_t wo = (old & 0xffu) / PER, wn = (cs & 0xffu) / PER, so = shift(old), sn = shift(cs);
    uint32_t sa[NB];  // adjacency of the side list's vertices to v*
    auto neighbours = [&](auto rounds_c, uint32_t eb, bool with_side) {
      constexpr int R = decltype(rounds_c)::value;
      uint32_t nb[R], ra[R], rb[R], xn[R], grew = 0u;
      uint64_t mi[R];
      bool ins[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t at = nrow + 2u * min(eb + e0 + r * BLOCK, stride - 1u);
        nb[r] = (uint32_t)*(gptr<const uint16_t>)((gptr<const char>)ell + at);
      }
      if (with_side && tail_wave) {
#pragma unroll
        for (int b = 0; b < NB; ++b) sa[b] = adj_word(sv[b]);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t* ru = tabw + __umul24(nb[r], rw);
        ra[r] = ru[wo];
        rb[r] = ru[wn];
        xn[r] = cg[nb[r]];
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        uint32_t* ru = tabw + __umul24(nb[r], rw);
        const uint32_t ea = (ra[r] >> so) & ESC, ec = (rb[r] >> sn) & ESC;
        atomicAdd(ru + wo, ea != ESC ? 0u - (1u << so) : 0u);
        atomicAdd(ru + wn, ec != ESC ? 1u << sn : 0u);
        const uint32_t x = xn[r], cu = x & 0xffu;
        // 256 colours leave none that the rows' ends could hold
        const bool hi = cu == cs && (PER * RW < 256u || nb[r] < (uint32_t)n);
        // a neighbour that starts to conflict and is not listed yet is appended
        ins[r] = hi && (x & 0xff00u) == 0u;
        cg[nb[r]] = (uint16_t)(x + (hi ? 0x100u : 0u) - (cu == old && (PER * RW < 256u || nb[r] < (uint32_t)n) ? 0x100u : 0u) + (ins[r] ? 0x8000u : 0u));
        grew |= ec == ESC - 1u ? 1u << r : 0u;
        mi[r] = __ballot(ins[r]);
      }
      if constexpr (NW > 1) {
        int more = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) more += __popcll(mi[r]);
        if (len + more > lcap) {  // this wave's list is full: nothing is appended, and the run is left to the rerun
#pragma unroll
          for (int r = 0; r < R; ++r) mi[r] = 0ull, ins[r] = false;
          *full = 1u;
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        list[ins[r] ? len + (int)lane_rank(mi[r]) : lcap] = (uint16_t)nb[r];
        len += __popcll(mi[r]);
      }
      if (BITS == 4 && __ballot(grew != 0u)) {  // gamma[u][c*] no longer fits
        mailed = true;
#pragma unroll
        for (int r = 0; r < R; ++r)
          if ((grew >> r) & 1u) {
            const uint32_t p = atomicAdd(mailn, 1u);
            if (p < (uint32_t)kW8Mail)
              mail[p] = (nb[r] << 8) | cs;
            else
              *full = 1u;
          }
        lanes_joined();
      }
    };
    if (dstar != kW8None) {
      deg = row_c[vs + 1] - row_c[vs];
      constexpr int R = NW == 1 ? 4 : 2;  // rounds whose loads are issued before any is used
      if (stride <= (uint32_t)BLOCK) {
        neighbours(std::integral_constant<int, 1>{}, 0u, true);
      } else if (NW == 1 && stride <= 2u * BLOCK) {
        neighbours(std::integral_constant<int, 2>{}, 0u, true);
      } else {
        neighbours(std::integral_constant<int, R>{}, 0u, true);
        for (uint32_t eb = R * BLOCK; eb < (uint32_t)deg; eb += BLOCK)
          neighbours(std::integral_constant<int, 1>{}, eb, false);
      }
      snap = best_cur && fnew >= f_best;  // leaving the best state: keep a copy
      if (snap)
        for (int v = tid; v < n; v += BLOCK)
          gcol[v] = (int16_t)((uint32_t)v == vs ? old : (uint32_t)cg[v] & 0xffu);
      lanes_joined();
      // class sizes; a class that would pass its limit leaves the individual to the 16-bit rerun
      uint32_t csz = 0u;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const uint32_t c = (uint32_t)(lane + kWave * r);
        if (NR == 1 || (int)(cs >> 6) == r) csz = readlane(cz[r], cs & 63);
        cz[r] += (c == cs ? 1u : 0u) - (c == old ? 1u : 0u);
      }
      if (csz >= kW8ClassMax) {  // the same in every wave
        give_up();
        return;
      }
    } else {
#pragma unroll
      for (int b = 0; b < NB; ++b) sa[b] = 0u;
    }
    ++t;
    if (tail_wave) {
      // ---- side list for iteration t: gammas, expiries, the pair v* moved
      // onto, entries that return to the table.  One that this move touches
      // waits: a neighbour's lane may be looking at its table entry.
      const uint32_t texp = (uint32_t)t & kW8ExpMask;
      auto walk = [&](uint32_t v, uint32_t c, uint32_t ex, uint32_t& ga, bool nbr, bool& gone) {
        const bool up = nbr && c == cs, down = nbr && c == old;
        const uint32_t g = (ga & 0x7fu) + (up ? 1u : 0u) - (down ? 1u : 0u);
        const bool open = ga >= kW8Free || ex == texp;
        gone = v == vs && c == cs;
        const bool back = !gone && open && g < ESC && !up && !down && v != (uint32_t)n;
        if (back) atomicAdd(&tabw[__umul24(v, rw) + c / PER], 0u - ((ESC - g) << shift(c)));
        lanes_joined();
        ga = g | (open ? kW8Free : 0u);
        gone |= back;
      };
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b == 0 || room[b] != ~0ull) {
          bool gone;
          walk(sv[b], sc[b], sx[b], sg[b], ((sa[b] >> (sv[b] & 31u)) & 1u) != 0u, gone);
          sv[b] = gone ? (uint32_t)n : sv[b];
          sc[b] = gone ? kNoColour : sc[b];
          room[b] |= __ballot(gone);
        }
      if (A > 0) {
        int base = 0;
        // in place: entries are read before those positions are written (base <= i0)
        for (int i0 = 0; i0 < A; i0 += kWave) {
          const bool alive = i0 + lane < A;
          const int i = alive ? i0 + lane : acap;
          const uint32_t e = act[i], eg = actg[i], v = alive ? e >> 17 : (uint32_t)n;
          const uint32_t c = alive ? (e >> 9) & 0xffu : kNoColour;
          uint32_t ga = eg & 0xffu;
          const uint32_t ad = dstar != kW8None ? adj_word(v) >> (v & 31u) : 0u;
          bool gone;
          walk(v, c, (e & 0x1ffu) | ((eg >> 8) << 9), ga, (ad & 1u) != 0u, gone);
          const bool keep = alive && !gone;
          const uint64_t mk = __ballot(keep);
          const int p = keep ? base + (int)lane_rank(mk) : acap;
          act[p] = e;
          actg[p] = (uint16_t)((eg & 0xff00u) | ga);
          base += __popcll(mk);
        }
        A = base;
      }
      if (dstar != kW8None) {
        // v*: its new colour escaped, its state, the pair it left
        const uint32_t gown = (xs >> 8) & 0x7fu, gnew = gown + dstar - 128u;
        // tenure term floor(num * f / den), capped (as in the block kernel)
        const uint64_t prod = (uint64_t)ten_num * (uint32_t)fnew;
        uint32_t ttf;
        if (prod <= 0xffffffffull) {
          const uint32_t x = (uint32_t)prod;
          ttf = __umulhi(x, den_inv);
          uint32_t rem = x - ttf * ten_den;
          if (rem >= ten_den) {
            rem -= ten_den;
            ++ttf;
          }
          if (rem >= ten_den) ++ttf;
        } else {
          ttf = (uint32_t)std::min<uint64_t>(prod / ten_den, kTenureCap + 1);
        }
        const bool capped = ttf > (uint32_t)kTenureCap;
        if (capped) ttf = kTenureCap;
        st_cap += capped ? 1u : 0u;
        const uint32_t expiry = (uint32_t)t - 1u + readlane(Lreg, (t - 1) & 63) + ttf;
        // a tenure of 0 or 1 never forbids anything
        const uint32_t gl = gown | (expiry > (uint32_t)t ? 0u : kW8Free);
        bool put = false;
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (!put && room[b] != 0ull) {
            const int at = __builtin_ctzll(room[b]);
            const bool me = lane == at;
            sv[b] = me ? vs : sv[b];
            sc[b] = me ? old : sc[b];
            sx[b] = me ? expiry & kW8ExpMask : sx[b];
            sg[b] = me ? gl : sg[b];
            room[b] &= room[b] - 1ull;
            put = true;
          }
        if (!put) {
          if (l0 && A < acap) {
            act[A] = (vs << 17) | (old << 9) | (expiry & 0x1ffu);
            actg[A] = (uint16_t)((((expiry & kW8ExpMask) >> 9) << 8) | gl);
          }
          lanes_joined();
          spill |= A >= acap;
          A = min(A + 1, acap);
        }
        if (l0) {
          atomicOr(&tabw[vs * rw + wn], ESC << sn);
          cg[vs] = (uint16_t)(cs | (gnew << 8) | 0x8000u);
        }
        lanes_joined();
      }
      if (spill) {
        if (NW == 1) {
          give_up();
          return;
        }
        if (l0) *full = 1u;
        lanes_joined();
      }
    }
    if (wid == 0) {
      const uint32_t vrec = dstar != kW8None ? vs : 0xffffu;
      if (t <= trace_cap) {  // every lane writes the same record
        int32_t* tr = late()->trace + ((size_t)li * trace_cap + (t - 1)) * 2;
        tr[0] = (int32_t)(vrec | (cs << 16));
        tr[1] = fnew;
      }
      st_deg += (uint64_t)deg;
      st_noops += dstar == kW8None ? 1u : 0u;
      st_ties += dstar != kW8None && shared ? 1u : 0u;
      fp = fnv_step(fp, vrec, cs, fnew);
    }
    f = fnew;
    if (f < f_best) {
      f_best = f;
      best_cur = true;
    } else if (snap) {
      best_cur = false;
    }
    team_sync<NW>();
  }

  if (rfl(*full)) {  // an entry was lost in the last iteration: the result may be off
    give_up();
    return;
  }
  if (best_cur)
    for (int v = tid; v < n; v += BLOCK) gcol[v] = (int16_t)(cg[v] & 0xffu);
  // the lanes' conflict counts (up to 2^41 each) in two halves
  {
    const uint64_t lo = (uint64_t)wave_sum_u32((uint32_t)st_conf & 0xffffffu) + ((uint64_t)wave_sum_u32((uint32_t)(st_conf >> 24)) << 24);
    st_conf = lo;
  }
  if constexpr (NW > 1) {
    if (l0) slot[wid] = make_uint4((uint32_t)st_conf, (uint32_t)(st_conf >> 32), st_cap, 0u);
    __syncthreads();
    if (tid == 0) {
      st_conf = 0ull;
      st_cap = 0u;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const uint4 e = slot[w];
        st_conf += ((uint64_t)e.y << 32) | e.x;
        st_cap += e.z;
      }
    }
  }
  if (tid == 0) {
    const TabuArgs* o = late();
    o->f_best[li] = f_best;
    o->iters[li] = t;
    if (o->stats) {
      int64_t* s = o->stats + (size_t)li * DLM_NSTATS;
      s[0] = (int64_t)(t - (int)st_noops);
      s[1] = (int64_t)st_noops;
      s[2] = (int64_t)st_conf;
      s[3] = (int64_t)st_deg;
      s[4] = (int64_t)st_ties;
      s[5] = (int64_t)st_cap;
      s[6] = 0;
      s[7] = 0;
    }
    if (o->hash) o->hash[li] = fp;
  }
}

}  // namespace dlm
