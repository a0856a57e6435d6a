// The weighted search of wvcp.hip with one wavefront per individual, for up to
// 512 vertices and 128 colours with 32-bit keys: the same trajectories, but a
// move re-examines only what it changed.
//
// A vertex's best move splits into e(v, c) = (max(m1[c], w) - m1[c]) << S + phi
// gamma[v][c], which depends on the colour, and a term of v alone (its class's
// loss and its own gamma).  B[v], a lower bound of e(v, c) over c != col v, is
// kept with one colour bc[v] that attains it, if one is known: a move from class
// a to class b changes e in the columns a and b only, so B[v] = min(B[v], e(v, a),
// e(v, b)) stays a bound, and it stays attained unless bc[v] is one of the two
// and both rose above it.  A row whose bound is not known to be attained is
// rescanned only when its bound reaches the best key of the others.
//
// Vertex v = lane + 64 j lives in lane `lane`, slot j: weight, freeze, colour,
// own gamma, B, bc and the class's loss in registers; the adjacency of slot j to
// v* is one 64-bit scalar.  Class c lives in lane c % 64: largest weight, its
// multiplicity, second largest.  Only gamma (8 bits when no degree passes 255,
// else 16), the rows that wait for a pass and the passes' results are in LDS.
//
// One iteration: the slots' smallest key over attained bounds (registers, a DPP
// minimum); rows whose bound reaches it are staged and LPR lanes per row (four
// colours each) rescan them; the vertices at the smallest key are staged and the
// same way find and hash the tied moves; the slots take the move.
//
// What bounds it: the instructions of one wave's chain (810 vector and 370
// scalar ones a move on G(300, 0.3) of 38 colours, eight individuals per CU).
// 4096 x 10 x 300 iterations there: 144.2 ms with the scan of every one-move by
// 256 threads, 40.7 ms with exact bounds after every move (10 passes of rescans
// a move), 35 ms with bounds that are only made exact when they matter (0.7
// rows a move) and ties staged for one hash.
#pragma once

#include "wave_util.h"
#include "wvcp.h"

namespace dlm {

constexpr int kWvMaxN = 512, kWvMaxK = 128;
constexpr uint32_t kWvNone = 0x7fffffffu;  // e of a colour that is no candidate
constexpr int kWvTies = 128;               // tied moves waiting for their hash: up to 64, and 64 more
constexpr uint32_t kWvOpen = 0xffffu;      // bc of a bound that is not known to be attained

struct WvLayout {
  uint32_t gam, rec, tie, res_b, res_c, bytes;
};

// nj slots, rows of kp = 4 * ceil(k / 4) gammas
__host__ __device__ inline WvLayout wv_layout(int nj, int k, int gamma_bytes) {
  WvLayout L;
  const uint32_t rows = 64u * (uint32_t)nj;
  uint32_t o = 0;
  L.gam = o;
  o += rows * 4u * (uint32_t)((k + 3) / 4) * (uint32_t)gamma_bytes;
  L.rec = o;  // also the class statistics while a round starts
  o += 8u * rows > 12u * kWvMaxK ? 8u * rows : 12u * kWvMaxK;
  L.tie = o;  // one entry more than kWvTies: where lanes without a tied move write
  o += 8u * (kWvTies + 1);
  L.res_b = o;
  o += 4u * rows;
  L.res_c = o;
  o += 2u * rows;
  L.bytes = (o + 15u) & ~15u;
  return L;
}

template <int NJ, int LPR, class GT>
__global__ __launch_bounds__(64) void wvcp_wave_kernel(WvcpArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kRows = kWave / LPR;  // rows of one pass
  const int lane = threadIdx.x, li = blockIdx.x;
  const uint32_t ind = (uint32_t)(a.ind_base + li);
  const int n = a.n, k = a.k, S = a.shift;
  const uint32_t kp = 4u * (uint32_t)((k + 3) >> 2);
  const WvLayout L = wv_layout(NJ, k, (int)sizeof(GT));
  GT* gam = reinterpret_cast<GT*>(smem + L.gam);
  uint2* rec = reinterpret_cast<uint2*>(smem + L.rec);  // {v | colour << 9 | own gamma << 16, weight}
  uint2* tie = reinterpret_cast<uint2*>(smem + L.tie);  // {v << 16 | c, colour of v | own gamma << 7 | gamma << 16}
  uint32_t* res_b = reinterpret_cast<uint32_t*>(smem + L.res_b);
  uint16_t* res_c = reinterpret_cast<uint16_t*>(smem + L.res_c);
  const uint32_t adj_words = 2u * (((uint32_t)n >> 6) + 1u);
  const __attribute__((address_space(4))) uint32_t* adj = (const __attribute__((address_space(4))) uint32_t*)a.adj;
  const __attribute__((address_space(4))) int32_t* row_c = (const __attribute__((address_space(4))) int32_t*)a.row_ptr;
  const RoundKeys rk = round_keys(a.key);
  const int lj = lane & (LPR - 1), lrow = lane / LPR;  // this lane's colours 4 lj .. 4 lj + 3 and row in a pass
  // slot state
  uint32_t w[NJ], col[NJ], own[NJ], bc[NJ], bestc[NJ];  // weights and class weights << S: below 2^31
  int32_t frz[NJ], B[NJ], base[NJ];
  {
    uint32_t bad = 0u;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int v = lane + 64 * j;
      const int c = v < n ? a.colors[(size_t)li * n + v] : 0;
      bad |= (c < 0) | (c >= k);
      bestc[j] = (uint32_t)c;
      w[j] = v < n ? (uint32_t)a.weights[v] << S : 0u;
    }
    if (__ballot(bad != 0u)) {
      if (lane == 0) a.best_legal[li] = -1;
      return;
    }
  }

  const int64_t phi_max = 1ll << 30;
  int64_t phi = ((int64_t)k * a.max_w << S) / (2 * (int64_t)n);
  int64_t best_legal = INT64_MAX;
  int t = 0;
  uint64_t st_deg = 0, fp = kFnvOffset;
  uint32_t st_noops = 0, st_ties = 0, st_legal_rounds = 0, Lreg = 0;
  uint32_t m1[2], c1[2], m2[2];  // class lane + 64 s
  uint32_t mq[4];                // largest weights of the classes 4 lj .. 4 lj + 3
  uint32_t no_colour[4];         // kWvNone for a colour past k (every e is below it)
#pragma unroll
  for (int b = 0; b < 4; ++b) no_colour[b] = 4 * lj + b < k ? 0u : kWvNone;

  for (int r = 0; r < a.R; ++r) {
    if (r == a.R - 1) phi = (int64_t)(2 * a.max_w) << S;
    const int32_t phi32 = (int32_t)phi;  // phi <= 2^30, and every key of the round fits 32 bits
    // e of the four colours of this lane in the row of a staged vertex
    auto row_costs = [&](uint32_t v, uint32_t cv, uint32_t wv, uint32_t (&e)[4], uint32_t (&g)[4]) {
      const GT* p = gam + v * kp + 4u * (uint32_t)lj;
      if constexpr (sizeof(GT) == 1) {
        const uint32_t x = *reinterpret_cast<const uint32_t*>(p);
#pragma unroll
        for (int b = 0; b < 4; ++b) g[b] = (x >> (8 * b)) & 0xffu;
      } else {
        const uint2 x = *reinterpret_cast<const uint2*>(p);
        g[0] = x.x & 0xffffu;
        g[1] = x.x >> 16;
        g[2] = x.y & 0xffffu;
        g[3] = x.y >> 16;
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint32_t c = 4u * (uint32_t)lj + (uint32_t)b;
        e[b] = (max(mq[b], wv) - mq[b] + (uint32_t)phi32 * g[b]) | no_colour[b];
        e[b] = c == cv ? kWvNone : e[b];
      }
    };
    // rows past the row's end read the next vertex's gammas or the record area: masked by c >= k
    auto rescan = [&](int cnt) {
      wave_sync();
      for (int p0 = 0; p0 < cnt; p0 += kRows) {
        const uint2 x = rec[min(p0 + lrow, cnt - 1)];
        const uint32_t v = x.x & 0x1ffu;
        uint32_t e[4], g[4];
        row_costs(v, (x.x >> 9) & 0x7fu, x.y, e, g);
        uint32_t m = min(e[0], e[1]), c = e[1] < e[0] ? 1u : 0u;
        c = e[2] < m ? 2u : c;
        m = min(m, e[2]);
        c = e[3] < m ? 3u : c;
        m = min(m, e[3]);
        uint32_t q = m;
        q = min(q, dpp_mov<dpp::kXor1>(q));
        q = min(q, dpp_mov<dpp::kXor2>(q));
        q = min(q, dpp_mov<dpp::kHalfMirror>(q));
        if constexpr (LPR > 8) q = min(q, dpp_mov<dpp::kMirror>(q));
        if constexpr (LPR > 16) q = min(q, (uint32_t)__shfl_xor((int)q, 16));
        if (m == q) {  // any colour at the minimum
          res_b[v] = q;
          res_c[v] = (uint16_t)(4u * (uint32_t)lj + c);
        }
      }
      wave_sync();
    };
    auto class_base = [&](uint32_t wv, uint32_t x1, uint32_t y1, uint32_t x2) {
      return wv == x1 && y1 == 1u ? (int32_t)(x2 - x1) : 0;
    };

    // ---- fresh round state from the best-g colouring of the previous round
    wave_sync();
    for (uint32_t i = lane; i < 64u * NJ * kp * sizeof(GT) / 4u; i += kWave) reinterpret_cast<uint32_t*>(gam)[i] = 0u;
    uint32_t* cm = reinterpret_cast<uint32_t*>(rec);  // class m1, c1, m2
    for (int i = lane; i < 3 * kWvMaxK; i += kWave) cm[i] = 0u;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      col[j] = bestc[j];
      res_c[lane + 64 * j] = (uint16_t)bestc[j];
    }
    wave_sync();
    const int nnz = row_c[n];
    for (int e = lane; e < nnz; e += kWave) {
      const uint32_t ix = (uint32_t)a.erow[e] * kp + (uint32_t)res_c[a.col_idx[e]];
      constexpr uint32_t per = 4u / sizeof(GT);
      atomicAdd(reinterpret_cast<uint32_t*>(gam) + ix / per, 1u << (8u * sizeof(GT) * (ix % per)));
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (lane + 64 * j < n) atomicMax(&cm[col[j]], w[j]);
    wave_sync();
    uint32_t twice = 0u;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int v = lane + 64 * j;
      own[j] = v < n ? (uint32_t)gam[(uint32_t)v * kp + col[j]] : 0u;
      twice += own[j];
      frz[j] = v < n ? 0 : INT32_MAX;
      if (v < n) {
        if (w[j] == cm[col[j]])
          atomicAdd(&cm[kWvMaxK + col[j]], 1u);
        else
          atomicMax(&cm[2 * kWvMaxK + col[j]], w[j]);
      }
    }
    wave_sync();
    uint32_t fwp = 0u;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      m1[s] = cm[lane + 64 * s];
      c1[s] = cm[kWvMaxK + lane + 64 * s];
      m2[s] = cm[2 * kWvMaxK + lane + 64 * s];
      fwp += m1[s] >> S;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) mq[b] = cm[4 * lj + b];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      base[j] = lane + 64 * j < n ? class_base(w[j], cm[col[j]], cm[kWvMaxK + col[j]], cm[2 * kWvMaxK + col[j]]) : 0;
    wave_sync();
    int64_t conf = (int64_t)(wave_sum_u32(twice) >> 1), fw = (int64_t)wave_sum_u32(fwp);
    int64_t G = (fw << S) + phi * conf, G_best = G, conf_best = conf;
    auto keep_legal = [&]() {
      best_legal = fw;
      int16_t* gcol = late_args<WvcpArgs>()->colors + (size_t)li * n;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (lane + 64 * j < n) gcol[lane + 64 * j] = (int16_t)col[j];
      lanes_joined();
    };
    if (conf == 0 && fw < best_legal) keep_legal();
    {
      int cnt = 0;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        rec[lane + 64 * j] = make_uint2((uint32_t)(lane + 64 * j) | (col[j] << 9), w[j]);
        cnt = min(n, 64 * (j + 1));
      }
      rescan(cnt);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const bool in = lane + 64 * j < n;
        B[j] = in ? (int32_t)res_b[lane + 64 * j] : (int32_t)kWvNone;
        bc[j] = in ? (uint32_t)res_c[lane + 64 * j] : 0u;
      }
    }

    for (int it = 0; it < a.T; ++it, ++t) {
      if ((t & 63) == 0)
        Lreg = lemire(philox_w0_rk(ind, (uint32_t)(t + lane), 0u, kDomTenure, rk), (uint32_t)a.ten_rand);
      // aspiration: G + dg < G_best, so dg <= -1 at most
      const int32_t asp = (int32_t)max<int64_t>(G_best - G - 1, (int64_t)INT32_MIN);

      // ---- the smallest admissible dg: over the attained bounds first, then
      // the rows whose bound reaches it are rescanned
      uint32_t kv[NJ], best = 0xffffffffu, open = 0xffffffffu;
      auto vertex_key = [&](int j) {
        const int32_t d = B[j] + base[j] - phi32 * (int32_t)own[j];
        // no other colour (k = 1), or no vertex: nothing to move
        return (frz[j] <= t || d <= asp) && B[j] != (int32_t)kWvNone ? (uint32_t)d ^ 0x80000000u : 0xffffffffu;
      };
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        kv[j] = vertex_key(j);
        best = min(best, bc[j] != kWvOpen ? kv[j] : 0xffffffffu);
        open = min(open, bc[j] == kWvOpen ? kv[j] : 0xffffffffu);
      }
      uint32_t cur = wave_min_u32(best);
      int cnt = 0, seen = 0;
      if (__ballot(open <= cur && open != 0xffffffffu)) {
        uint32_t again = 0u;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const bool need = bc[j] == kWvOpen && kv[j] <= cur && kv[j] != 0xffffffffu;
          const uint64_t M = __ballot(need);
          if (need) rec[cnt + (int)lane_rank(M)] = make_uint2((uint32_t)(lane + 64 * j) | (col[j] << 9), w[j]);
          lanes_joined();
          again |= need ? 1u << j : 0u;
          cnt += __popcll(M);
        }
        rescan(cnt);
        best = 0xffffffffu;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const bool need = ((again >> j) & 1u) != 0u;
          const uint32_t nbv = res_b[lane + 64 * j], ncv = res_c[lane + 64 * j];
          B[j] = need ? (int32_t)nbv : B[j];
          bc[j] = need ? ncv : bc[j];
          kv[j] = need ? vertex_key(j) : kv[j];
          best = min(best, bc[j] != kWvOpen ? kv[j] : 0xffffffffu);
        }
        cur = wave_min_u32(best);
        cnt = 0;
      }
      if (cur == 0xffffffffu) {  // nothing admissible
        ++st_noops;
        fp = fnv_step(fp, 0xffffu, 0xffffu, (int32_t)(G >> S));
        continue;
      }
      // ---- every admissible move at it, hashed
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const uint64_t M = __ballot(kv[j] == cur);
        if (kv[j] == cur) {
          rec[cnt + (int)lane_rank(M)] = make_uint2((uint32_t)(lane + 64 * j) | (col[j] << 9) | (own[j] << 16), w[j]);
          res_b[lane + 64 * j] = (uint32_t)B[j];
        }
        lanes_joined();
        cnt += __popcll(M);
      }
      uint64_t hk = ~0ull;  // hash << 32 | v << 16 | c of this lane's smallest
      uint32_t hx = 0u;     // colour of its vertex | own gamma << 7 | gamma[v][c] << 16
      int nt = 0;           // tied moves staged
      auto hash_staged = [&]() {
        wave_sync();
        for (int b0 = 0; b0 < nt; b0 += kWave) {
          const bool in = b0 + lane < nt;
          const uint2 x = tie[in ? b0 + lane : 0];
          const uint64_t y = ((uint64_t)philox_w0_rk(ind, (uint32_t)t, x.x >> 16, x.x & 0xffffu, rk) << 32) | x.x;
          const bool lt = in && y < hk;
          hk = lt ? y : hk;
          hx = lt ? x.y : hx;
        }
        seen += nt;
        nt = 0;
        wave_sync();
      };
      wave_sync();
      for (int p0 = 0; p0 < cnt; p0 += kRows) {
        const bool ok = p0 + lrow < cnt;
        const uint2 x = rec[ok ? p0 + lrow : 0];
        const uint32_t v = x.x & 0x1ffu;
        uint32_t e[4], g[4];
        row_costs(v, (x.x >> 9) & 0x7fu, x.y, e, g);
        const uint32_t target = res_b[v];
        uint32_t z = 0u;
#pragma unroll
        for (int b = 0; b < 4; ++b) z |= e[b] == target ? 1u << b : 0u;
        z = ok ? z : 0u;
        for (uint64_t m = __ballot(z != 0u); m; m = __ballot(z != 0u)) {
          const uint32_t b = (uint32_t)__builtin_ctz(z | 16u);
          const uint32_t gb = b == 0u ? g[0] : b == 1u ? g[1] : b == 2u ? g[2] : g[3];
          tie[z ? nt + (int)lane_rank(m) : kWvTies] = make_uint2((v << 16) | (4u * (uint32_t)lj + b), (x.x >> 9) | (gb << 16));
          nt += __popcll(m);
          z &= z - 1u;
          if (nt > kWvTies - kWave) hash_staged();
        }
      }
      hash_staged();
      const uint32_t h = wave_min_u32((uint32_t)(hk >> 32));
      uint64_t at = __ballot((uint32_t)(hk >> 32) == h);
      if (at & (at - 1ull)) {  // equal hashes: the smallest (v, c)
        const uint32_t lo = wave_min_u32((uint32_t)(hk >> 32) == h ? (uint32_t)hk : 0xffffffffu);
        at = __ballot(hk == (((uint64_t)h << 32) | lo));
      }
      const int wl = __builtin_ctzll(at);
      const uint32_t win = readlane((uint32_t)hk, wl), xs = readlane(hx, wl);
      const uint32_t vs = win >> 16, cs = win & 0xffffu, old = xs & 0x7fu, gnew = xs >> 16;
      const int32_t dg = (int32_t)(cur ^ 0x80000000u), dcf = (int32_t)gnew - (int32_t)((xs >> 7) & 0x1ffu);
      // the adjacency of every slot to v*
      uint64_t nb[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const uint32_t o = vs * adj_words + 2u * j;
        nb[j] = (uint64_t)adj[o] | ((uint64_t)adj[o + 1] << 32);
      }
      const int deg = row_c[vs + 1] - row_c[vs];
      // gammas in the two columns, of every vertex
      uint32_t go[NJ], gc[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const GT* p = gam + (uint32_t)(lane + 64 * j) * kp;
        go[j] = p[old];
        gc[j] = p[cs];
      }

      // ---- classes: c* gains v* in O(1); the one it left is looked over only
      // when v* held its largest weight alone or its second largest
      uint32_t wv;
      {
        uint32_t x = 0u;
#pragma unroll
        for (int j = 0; j < NJ; ++j) x = (int)(vs >> 6) == j ? w[j] : x;
        wv = readlane(x, vs & 63);
      }
      auto class_get = [&](const uint32_t (&x)[2], uint32_t c) { return readlane(c < 64u ? x[0] : x[1], c & 63); };
      uint32_t o1 = class_get(m1, old), oc = class_get(c1, old), o2 = class_get(m2, old);
      const uint32_t b1 = class_get(m1, cs), bn = class_get(c1, cs), b2 = class_get(m2, cs);
      const uint32_t n1 = max(b1, wv), nc = wv > b1 ? 1u : bn + (wv == b1 ? 1u : 0u);
      const uint32_t n2 = wv > b1 ? b1 : (wv == b1 ? b2 : max(b2, wv));
      if (wv == o1 && oc > 1u) {
        --oc;
      } else if (wv == o1 || wv == o2) {
        uint32_t x = 0u;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          x = max(x, col[j] == old && lane + 64 * j != (int)vs ? w[j] : 0u);
        o1 = wave_max_u32(x);
        oc = 0u;
        x = 0u;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const bool in = col[j] == old && lane + 64 * j != (int)vs && w[j] != 0u;
          oc += (uint32_t)__popcll(__ballot(in && w[j] == o1));
          x = max(x, in && w[j] < o1 ? w[j] : 0u);
        }
        o2 = wave_max_u32(x);
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bool is_o = (uint32_t)(lane + 64 * s) == old, is_c = (uint32_t)(lane + 64 * s) == cs;
        m1[s] = is_c ? n1 : is_o ? o1 : m1[s];
        c1[s] = is_c ? nc : is_o ? oc : c1[s];
        m2[s] = is_c ? n2 : is_o ? o2 : m2[s];
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint32_t c = 4u * (uint32_t)lj + (uint32_t)b;
        mq[b] = c == cs ? n1 : c == old ? o1 : mq[b];
      }

      // ---- the slots: gammas, own gammas, class losses, best values
      const uint32_t Lt = readlane(Lreg, t & 63);
      const int32_t until = (int32_t)((uint32_t)t + Lt + (uint32_t)a.frz);
      const int32_t loss_o = class_base(o1, o1, oc, o2), loss_n = class_base(n1, n1, nc, n2);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        uint32_t one;  // this lane's bit of the mask
        asm("v_cndmask_b32_e64 %0, 0, 1, %1" : "=v"(one) : "s"(nb[j]));
        GT* p = gam + (uint32_t)(lane + 64 * j) * kp;
        go[j] -= one;
        gc[j] += one;
        p[old] = (GT)go[j];  // the row is this lane's alone
        p[cs] = (GT)gc[j];
        const bool moved = lane + 64 * j == (int)vs;
        own[j] = moved ? gnew : col[j] == old ? go[j] : col[j] == cs ? gc[j] : own[j];
        col[j] = moved ? cs : col[j];
        frz[j] = moved ? until : frz[j];
        const bool in_old = col[j] == old, in_new = col[j] == cs;
        base[j] = in_new ? (w[j] == n1 ? loss_n : 0) : in_old ? (w[j] == o1 ? loss_o : 0) : base[j];
        uint32_t eo = max(o1, w[j]) - o1 + (uint32_t)phi32 * go[j];
        uint32_t ec = max(n1, w[j]) - n1 + (uint32_t)phi32 * gc[j];
        eo = in_old ? kWvNone : eo;
        ec = in_new ? kWvNone : ec;
        uint32_t m = min(eo, ec);
        if (j == NJ - 1) m = lane + 64 * j < n ? m : kWvNone;
        const bool attained = m <= (uint32_t)B[j] && m != kWvNone;
        bc[j] = attained ? (eo <= ec ? old : cs) : (bc[j] == old || bc[j] == cs ? kWvOpen : bc[j]);
        B[j] = attained ? (int32_t)m : B[j];
      }
      conf += dcf;
      G += dg;
      fw = (G - phi * conf) >> S;
      st_deg += (uint64_t)deg;
      st_ties += seen > 1 ? 1u : 0u;
      fp = fnv_step(fp, vs, cs, (int32_t)(G >> S));
      if (G < G_best) {
        G_best = G;
        conf_best = conf;
#pragma unroll
        for (int j = 0; j < NJ; ++j) bestc[j] = col[j];
      }
      if (conf == 0 && fw < best_legal) keep_legal();
    }
    const bool legal = conf_best == 0;
    st_legal_rounds += legal ? 1u : 0u;
    if (r < a.R - 1) phi = legal ? (phi >> 1) : min(phi << 1, phi_max);
  }
  const WvcpArgs* o = late_args<WvcpArgs>();
  if (best_legal == INT64_MAX) {
    int16_t* gcol = o->colors + (size_t)li * n;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (lane + 64 * j < n) gcol[lane + 64 * j] = (int16_t)bestc[j];
  }
  if (lane == 0) {
    o->best_legal[li] = best_legal == INT64_MAX ? 0x7fffffff : (int32_t)best_legal;
    if (o->stats) {
      int64_t* s = o->stats + (size_t)li * DLM_NSTATS;
      s[0] = (int64_t)(t - (int)st_noops);
      s[1] = (int64_t)st_noops;
      s[2] = (int64_t)st_deg;
      s[3] = (int64_t)st_ties;
      s[4] = (int64_t)st_legal_rounds;
      s[5] = phi;
      s[6] = 0;
      s[7] = 0;
    }
    if (o->hash) o->hash[li] = fp;
  }
}

template <int NJ, int LPR, class GT>
static int launch_wv(const WvcpArgs& a, int pop, size_t lds, hipStream_t s) {
  auto kern = wvcp_wave_kernel<NJ, LPR, GT>;
  DLM_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kern, dim3(pop), dim3(kWave), lds, s, a);
  DLM_HIP(hipGetLastError());
  return DLM_OK;
}

template <class GT>
static int launch_wv_gamma(const WvcpArgs& a, int pop, size_t lds, hipStream_t s) {
  const int nj = (a.n + 63) / 64;
#define DLM_WV(J)                                                    \
  case J:                                                            \
    return a.k <= 32   ? launch_wv<J, 8, GT>(a, pop, lds, s)         \
           : a.k <= 64 ? launch_wv<J, 16, GT>(a, pop, lds, s)        \
                       : launch_wv<J, 32, GT>(a, pop, lds, s);
  switch (nj) {
    DLM_WV(1) DLM_WV(2) DLM_WV(3) DLM_WV(4) DLM_WV(5) DLM_WV(6) DLM_WV(7) DLM_WV(8)
  }
#undef DLM_WV
  return set_error(DLM_E_UNSUPPORTED, "dlm_wvcp_batch: n=%d too large for the wave search", a.n);
}

}  // namespace dlm
