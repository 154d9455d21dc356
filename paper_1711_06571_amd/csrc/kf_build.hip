// Combinatorial Kalman-filter track building (sections 2, 3.1, 4.3).
//
// Layout of the work: one lane per candidate slot, S = cand_cap consecutive
// lanes per seed, floor(64 / S) seeds per wave (lanes beyond the last seed
// idle).  One persistent launch: each wave takes groups of seeds from an
// atomic queue until the queue is empty, so uneven events and seeds balance
// across the chip.
//
// Per layer, per wave:
//   1. every live slot predicts its candidate (FP32 or FP64 arithmetic);
//   2. the search windows are computed and the hits in the phi-sorted rows of
//      bins that cover them are tested, (candidate, hit) pairs shared by all
//      lanes; wide windows only where a hit that can survive may lie;
//   3. accepted hits go to a pool of their seed in LDS;
//   4. the seed's children (hits and holes) are ranked by counting, best
//      first by (nhits, chi2, parent slot, hit chi2, hit index); the best cap
//      take the slots 0..cap-1;
//   5. the new slots pull the parent's predicted state and apply the Kalman
//      update with their hit;
//   6. back-pointers (parent slot, hit) go to the wave's history table in the
//      workspace; the best hit list is recovered at the end by walking it
//      backwards.
// Candidates with no child compete for a per-seed best-finished record (LDS).
#include <stdint.h>
#include <stdio.h>

#include <mutex>

#include "kfdev.h"
#include "kfhost.h"
#include "kfmlp.h"
#include "kfplan.h"
#include "kfwave.h"

using namespace kfdev;
using namespace kfreach;

namespace {

struct BuildArgs {
  // geometry
  int n_layers;
  float r[32];
  float z_half, bz, x_over_x0, mass;
  // cuts
  float chi2_cut;
  int max_holes, cap;
  float nsigma, win_sig_rphi, win_sig_z;
  int first_layer;
  int window_mode;
  const float* mlp;
  // hits
  int n_events, n_phi, n_z;
  const int32_t* offsets;
  // the hits packed per sorted position, three float4 each:
  // (phi, x, y, z), (cov 0..3), (cov 4, cov 5, orig bits, 0)
  const float4* hpack;
  int n_hits;
  int refine;            // sub-bins per phi bin in the fine index
  const int32_t* fine;   // [events][layers][n_z][n_phi * refine + 1]
  uint32_t* hist;        // [resident waves][searched layers][64] back-pointers
  // seeds
  int n_seeds, ld, n_groups;
  const float *seed_par, *seed_cov;
  const int8_t* q;
  const int32_t* seed_event;
  const int32_t* seed_order;
  // outputs
  int32_t* out_hits;
  float *out_par, *out_cov, *out_chi2;
  int32_t *out_nhits, *out_status;
  // extras
  const int32_t* event_n_seeds;
  int64_t* event_done_ticks;
  int64_t* start_tick;
  const int32_t* true_hits;
  const float* true_xyz;
  float* dump;
  int32_t* dump_count;
  int dump_capacity;
  unsigned long long* counters;
  // workspace
  int32_t* queue;
  int32_t* event_done;
};

// ku / kv in FP64 builds only: there, kernel arguments and per-seed values
// that the layer loop uses are recomputed where they are used instead of
// being hoisted out of the loop and spilled (the FP32 build spills 28 to 68 B a
// lane; with them 24 to 32, and its times stay within 1 %)
template <typename T, typename U> __device__ inline U ku64(U v) {
  if constexpr (sizeof(T) == 8) return ku(v);
  else return v;
}
template <typename T, typename U> __device__ inline U kv64(U v) {
  if constexpr (sizeof(T) == 8) return kv(v);
  else return v;
}

// The bounds of a Reach over sorted positions [p0, p1): the packing chunks
// that overlap them.
__device__ inline void reach_bounds(const float4* pack, int n_hits, int p0, int p1, Reach& q) {
  uint32_t l = 0, z = 0, lo = 0x7F800000u, hi = 0;
  for (int c = p0 / kPackChunk; c * kPackChunk < p1; ++c) {
    const uint32_t* w = (const uint32_t*)(pack + (size_t)c * kPackChunk * 3 + 2) + 3;
    const uint32_t u = w[0], r = c * kPackChunk + 1 < n_hits ? w[12] : 0x7F80u;
    l = (u & 0xFFFF0000u) > l ? (u & 0xFFFF0000u) : l;  // (non-negative floats order as integers)
    z = (u & 0xFFFFu) > z ? (u & 0xFFFFu) : z;
    lo = (r & 0xFFFF0000u) < lo ? (r & 0xFFFF0000u) : lo;
    hi = (r & 0xFFFFu) > hi ? (r & 0xFFFFu) : hi;
  }
  q.v = l | z;
  q.rad = lo | hi;
}

// The lanes of a candidate's seed.
struct Group {
  int sidx, base, slot, S;
  bool used;
};

// A seed's accepted hits of a layer: a pool of kPoolPerCap * cap entries in
// LDS, in no order (a candidate's own list is never needed: only the seed's
// best cap children survive), and room for the holes of its candidates.
//   e    [SEEDS][stride] {chi2, (slot << 24) | sorted position in the event}
//   cnt  [SEEDS] entries
//   seen [64] whether a candidate accepted a hit
constexpr int kPoolPerCap = 7;  // (with the holes a seed has at most 8 cap <= 64 children)
constexpr uint32_t kNoHit = 0xFFFFFFu;  // the position of a hole
struct Pool {
  uint2* e;
  int32_t* cnt;
  uint8_t* seen;
  int stride, full;
};

__device__ inline uint64_t readlane64(uint64_t v, int j) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, j);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), j);
  return ((uint64_t)hi << 32) | lo;
}

// chi2 that a hit of the candidate may have to reach the seed's best cap,
// `worst` the rank key of cap-th child known: such that the sum, rounded to
// FP32, does not exceed the key's.
template <typename T> __device__ inline float useful_chi2(uint64_t worst, T chi2, int nhits) {
  const int n = 31 - (int)(worst >> 59);
  const float sum = __uint_as_float((uint32_t)(worst >> 27));
  if (nhits + 1 > n) return __builtin_inff();
  return nhits + 1 < n ? -1.f : (float)((T)sum - chi2) + 1.3e-7f * sum;
}

// Cuts the pool of seed s (the same in every lane) to its best cap entries,
// in rank order: one entry per lane (a pool holds at most 64), each ranked
// against all others by the exact order of children (nhits, chi2, slot, hit
// chi2, hit index).  Where more than cap entries were held, sets the chi2 bound
// thr of the seed's candidates, and `cut`.
template <typename T>
__device__ inline void pool_cut(const BuildArgs& A, const Pool& po, const Group& gr, int s, int lane, T chi2, int nhits,
                                int e0, float& thr, bool& cut) {
  const int held = __builtin_amdgcn_readfirstlane(po.cnt[s]);
  const int m = held < po.full ? held : po.full;
  const bool in = lane < m;
  uint2* pe = po.e + s * po.stride;
  uint2 e = pe[in ? lane : 0];
  const float c2 = __uint_as_float(e.x);
  const int slot = in ? (int)(e.y >> 24) : 0, src = s * gr.S + slot;
  const T pc = shfl_t(chi2, src);
  const int pn = __shfl(nhits, src, 64), pe0 = __shfl(e0, src, 64);
  const uint32_t orig =
      in ? __float_as_uint(A.hpack[(size_t)(pe0 + (int)(e.y & 0xFFFFFFu)) * 3 + 2].z) : 0xFFFFFFFFu;
  const uint64_t key = in ? make_key(pn + 1, (float)(pc + (T)c2), slot, 0) : kInfKey;
  int rank = 0;
  for (int i = 0; i < m; ++i) {
    const uint64_t ki = readlane64(key, i);
    const float ci = readlane_t(c2, i);
    const uint32_t oi = (uint32_t)__builtin_amdgcn_readlane((int)orig, i);
    rank += ki < key || (ki == key && top_before(ci, oi, c2, orig)) ? 1 : 0;
  }
  lds_order();
  if (in && rank < A.cap) pe[rank] = e;
  if (lane == 0) po.cnt[s] = m < A.cap ? m : A.cap;
  lds_order();
  if (m > A.cap) {
    const uint64_t worst = readlane64(key, (int)__builtin_ctzll(__ballot(in && rank == A.cap - 1)));
    if (gr.used && gr.sidx == s) {
      thr = useful_chi2<T>(worst, chi2, nhits);
      cut = true;
    }
  }
}

// A candidate is wide when its window may hold more pairs than kWidePairs and
// kWideRow for each row of its bounded search, whose four intervals a row are
// an iteration each, however few hits they hold; it then first searches
// where its kProbeHits best hits should lie.
// Measured (us; the macros allow a rebuild to compare):
//                                 row 0   16   32  512 | probe 8   16   32
//   400 events of 100, 8 x 64 bins 1224  607  528  528 |     596  607  559
//   20 events of 20 000, FP64      4781 4787 4778 5281 |    4705 4787 4932
//   one event of 20 000, FP32       454  451  452  613 |     417  451  504
//   its windows 1 x 3 cm at least  2078 2093 2175 3581 |    1975 2093 2282
// kWidePairs of 96, 192, 384: 1 913, 2 093, 2 547 us with the 1 x 3 cm windows, 488,
// 437, 360 with 400 events of 100 tracks in 63 x 16 bins, the others within 1 %.
#ifndef KF_WIDE_PAIRS
#define KF_WIDE_PAIRS 192
#endif
#ifndef KF_WIDE_ROW
#define KF_WIDE_ROW 32
#endif
#ifndef KF_PROBE_HITS
#define KF_PROBE_HITS 8
#endif
constexpr float kWidePairs = KF_WIDE_PAIRS, kWideRow = KF_WIDE_ROW, kProbeHits = KF_PROBE_HITS;

// Hit search of every candidate of the wave, shared by all 64 lanes.
//
// Each live candidate's window covers, per z row it overlaps and per phi
// interval (two where the window wraps at 2 pi), one range of sorted hit
// positions bracketed by the fine phi index.  Range r of every candidate is
// taken in turn; the (candidate, hit) pairs of all candidates' ranges r are
// numbered through a wave prefix sum and handed out 64 NP at a time, NP
// pairs per lane, so a candidate with a wide window no longer holds up the
// wave while the others wait.  A lane finds the pair's candidate from the
// marks the candidates set where their pairs start and reads what that
// candidate's tests share by lane shuffles.  Every hit whose stored phi lies
// in the candidate's interval gets the exact window test (z first, then the
// angle about the axis); in-window hits get their chi2; accepted hits
// (chi2 < cut) go to their seed's pool (the slot from an LDS counter).  A
// pool that is full is cut to its best cap entries, and from then on only
// hits that can still be among them are added.
//
// Wide windows.  Few candidates hold most pairs (20 events of 20 000 tracks:
// 0.04 % of the candidate-layers, their windows whole layers, half of all
// pairs), and of all they accept only the seed's best cap children survive.
// A wide candidate first searches where hits of chi2 <= c2 lie (Reach), c2
// chosen to hold kProbeHits of them at the density of the window's middle
// row.  The seed's pool then bounds the chi2 of a hit that can still be among
// the survivors; where that bound is within c2 the search is complete, else
// the seed is searched again up to the bound (or the chi2 cut).  What is left
// out cannot survive; it would only have been counted, and the counts matter
// to "any child" (known from the accepted hits or the hole) and to "cut to
// cap" (known once the seed accepted more than cap).  Work counters ask for
// every hit: no bound then.  Pairs, same events: 462 M -> 123 M.
//
// The tests and chi2 run in FP32 in both arithmetic modes, from the
// prediction rounded to FP32: their rounding (chi2 ~ 3e-5 at the cut,
// positions ~ 1e-5 cm) stays far below the chi2 gaps (1e-3) and window-edge
// distances (1e-4 cm) that separate decisions; the Kalman update of a
// chosen hit runs in the arithmetic of the mode.  NP (pairs per lane and
// round at most) is defined with the LDS plan.
//
// seen: the candidate has a hit child; cut: the seed has more children than
// cap; scanned, tested: work counters of the hits this lane examined.
template <typename T, int NPT>
__device__ inline void coop_scan(const BuildArgs& A, int ev, int e0, int l, bool pok, const T Xp[6], const T Pp[21],
                                 T dphi_w, T dz_w, T chi2, int nhits, bool hole_ok, const Group& gr, const Pool& po,
                                 int8_t* start, int lane, bool& seen, bool& cut, unsigned& scanned,
                                 unsigned& tested) {
  static_assert(NPT >= 1 && NPT <= NP, "pairs per lane");
  const int nz = A.n_z, nf = A.n_phi * A.refine;
  // this lane's window as conservative stored-value intervals (the exact
  // test decides): a half-width half() about phip (3.14159 and more: the whole
  // circle), z rows taken from the middle one outwards
  float phip = 0.f;
  Rows rw = {0, -1, 0};
  // Per candidate, what every hit test shares: for dphi < pi/2 the angle
  // test |atan2(cross, dot)| <= dphi is dot > 0 and |cross| <= tan(dphi) dot
  // (ftan < 0 marks a wider window, which keeps the angle); the measurement
  // frame (tangent t = (-y, x) / r at the predicted point, from 1 / r) and
  // H P H^T of the prediction.
  float fx = 0.f, fy = 0.f, fz = 0.f, fdz = 0.f, fdphi = 0.f, ftan = 0.f;
  float firr = 0.f, suu = 0.f, suw = 0.f, sww = 0.f;
  auto half = [&]() { return fdphi + kEpsPhi; };
  if (pok) {
    fx = (float)Xp[0];
    fy = (float)Xp[1];
    fz = (float)Xp[2];
    fdz = (float)dz_w;
    fdphi = (float)dphi_w;
    phip = wrap_2pi(atan2f(fy, fx));
    rw = rows_of(fz, fdz + kEpsZ, ku64<T>(A.z_half), ku64<T>(A.n_z));
    // (the angle test runs in FP32: so does the tangent of its bound)
    ftan = !(dphi_w < T(1.5707963267948966)) ? -1.f : tanf((float)dphi_w);
    const T rr = k_sqrt(Xp[0] * Xp[0] + Xp[1] * Xp[1]);
    const T irr = k_rcp(rr);
    const T tx = -Xp[1] * irr, ty = Xp[0] * irr;
    firr = (float)irr;
    suu = (float)(tx * tx * Pp[ut(0, 0)] + T(2) * tx * ty * Pp[ut(0, 1)] + ty * ty * Pp[ut(1, 1)]);
    suw = (float)(tx * Pp[ut(0, 2)] + ty * Pp[ut(1, 2)]);
    sww = (float)Pp[ut(2, 2)];
  }
  const int32_t* frow = A.fine + ((size_t)ev * A.n_layers + l) * nz * (nf + 1);
  // ranges: (row, interval) for every row, 1 << sh intervals per row (two
  // where the window wraps at 2 pi, four of a Reach)
  Reach rq = {0.f, 0.f, 0u, 0u};
  float al[2] = {1.f, 1.f}, ah[2] = {0.f, 0.f};  // the row's arcs
  int sh = phi_parts(phip, half());
  int R = pok ? rw.n() << sh : 0;
  const float chi2_cut = A.chi2_cut;
  float thr = __builtin_inff();  // chi2 of a hit that may enter the pool
  bool lim = false;              // any pool was cut: thr counts
  // Ranges of iteration r: one range, or, where a row is one interval, two
  // rows (most windows that cross a row edge are then done in one
  // iteration): the stored-value interval and the sorted positions from the
  // fine index (read one iteration ahead).
  auto iters = [&]() { return sh == 0 ? (R + 1) >> 1 : R; };
  auto range_of = [&](int it, float& a, float& b, int& q0, int& q1, int& q2, int& q3) {
    a = 1.f;
    b = 0.f;
    q0 = 0;
    q1 = 0;
    q2 = 0;
    q3 = 0;
    const int r = sh == 0 ? 2 * it : it;
    if (r < R) {
      const int nf = ku64<T>(A.n_phi) * ku64<T>(A.refine), nz = ku64<T>(A.n_z);
      const float inv = fine_inv(nf);
      const int row = rw.at(r >> sh), i = r & ((1 << sh) - 1);
      if (sh == 2) {
        if (i == 0)
          reach_arcs(rq, suu, suw, sww, k_sqrt(fx * fx + fy * fy), fz, half(), fdz + kEpsZ, row, nz,
                     ku64<T>(A.z_half), al, ah);
        arc_part(phip, i & 2 ? al[1] : al[0], i & 2 ? ah[1] : ah[0], i & 1, a, b);
      } else {
        phi_part(phip, half(), i, a, b);
      }
      if (a <= b) {
        const int32_t* f = frow + (size_t)row * (nf + 1);
        const int ka = fine_key(a, inv, nf), kb = fine_key(b, inv, nf) + 1;
        q0 = f[ka];
        q1 = f[kb];
        if (sh == 0 && r + 1 < R) {
          const int32_t* f2 = frow + (size_t)rw.at(r + 1) * (nf + 1);
          q2 = f2[ka];
          q3 = f2[kb];
        }
      }
    }
  };
  const int inv_s = 65536 / gr.S + 1;  // lane / S = lane * inv_s >> 16 (lanes < 64)
  po.seen[lane] = 0;
  if (gr.used && gr.slot == 0) po.cnt[gr.sidx] = 0;

  float an = 1.f, bn = 0.f;
  int p0n = 0, p1n = 0, p2n = 0, p3n = 0;
  bool wide = false, pruned = false;
  bool look = A.counters == nullptr;  // wide windows still to be looked for
  bool again = false;                 // a wide candidate's bound still to be checked
  int Rmax = wave_max(iters());
  // (one call of range_of in the code: the pass over the ranges starts one
  // before the first, where only the first is read)
  for (int r = -1;;) {
    const float a = an, b = bn;
    const int p0 = p0n, p1 = p1n, p2 = p2n, p3 = p3n;
    range_of(r + 1, an, bn, p0n, p1n, p2n, p3n);
    if (r < 0 && look) {
      look = false;
      const int c0 = p1n - p0n;  // the middle row
      wide = pok && (float)c0 * (float)rw.n() > kWidePairs;
      if (__any(wide)) {
        if (wide) {
          const int32_t* of = A.offsets + ((size_t)ev * A.n_layers + l) * ((size_t)A.n_phi * nz + 1);
          reach_bounds(A.hpack, A.n_hits, of[rw.lo * A.n_phi], of[(rw.hi + 1) * A.n_phi], rq);
          wide = rq.usable(suu, sww);
          if (wide) {
            const float area = 4.f * fminf(half(), 3.1415927f) * k_sqrt(fx * fx + fy * fy) * A.z_half / (float)nz;
            const float s00 = fabsf(suu) + rq.lam(), s11 = sww + rq.vzz();
            const float s2 = fmaxf(s00 * s11 - suw * suw, 1e-6f * s00 * s11);
            const bool none = rq.none(suu, suw, sww);
            const float c2p =
                none ? chi2_cut : fminf(kProbeHits * area / (3.1415927f * k_sqrt(s2) * (float)c0), chi2_cut);
            rq.set(c2p, suu, suw, sww);
            Rows rb = rows_of(fz, fminf(fdz + kEpsZ, rq.dz(sww)), ku64<T>(A.z_half), nz);
            if (none) rb.hi = rb.lo - 1;
            wide = (float)c0 * (float)rw.n() > kWidePairs + kWideRow * (float)rb.n();
            if (wide) {
              rw = rb;
              sh = 2;
              R = rw.n() << sh;
            }
          }
        }
        again = __any(wide && rq.c2 < chi2_cut);
        Rmax = wave_max(iters());
        continue;
      }
    }
    const int cnt = r >= 0 && p1 > p0 ? p1 - p0 : 0;
    const int all = cnt + (r >= 0 && p3 > p2 ? p3 - p2 : 0);
    int total = 0;
    const int off = wave_excl_scan(all, lane, total);
    // sorted position of pair k of this candidate: pb + k, from pair `turn` on
    // (the second row) pb2 + k
    const int pb = p0 - off, turn = off + cnt, pb2 = p2 - turn;
    int carry = 0;  // candidate of the previous round's last pair
    // each lane takes NP pairs per round (pair base + 64 h + lane): their
    // loads share one round trip
    for (int base = 0; base < total; base += 64 * NPT) {
      // candidate of a pair: candidates mark the slot where their pairs start
      // in this round; the pair's candidate is the nearest mark at or below
      // its slot in its half, else the one whose pairs run on from before
#pragma unroll
      for (int h = 0; h < NPT; ++h) start[h * 64 + lane] = -1;
      if (all > 0 && off >= base && off - base < 64 * NPT) start[off - base] = (int8_t)lane;
      lds_order();
      int c[NPT], p[NPT];
      bool valid[NPT];
      float ca[NPT], cb[NPT], cx[NPT], cy[NPT], cz[NPT], cdz[NPT], cdphi[NPT], ctan[NPT], cirr[NPT], csuu[NPT], csuw[NPT],
          csww[NPT];
#pragma unroll
      for (int h = 0; h < NPT; ++h) {
        const int st = start[h * 64 + lane];
        const unsigned long long sm = __ballot(st >= 0) & ((2ull << lane) - 1ull);
        const int hb = sm ? 63 - (int)__builtin_clzll(sm) : 0;
        const int sc = __shfl(st, hb, 64);
        c[h] = sm ? sc : carry;
        carry = __builtin_amdgcn_readlane(c[h], 63);
        const int k = base + 64 * h + lane;
        valid[h] = k < total;
        const int c1 = __shfl(pb, c[h], 64), c2 = __shfl(pb2, c[h], 64);
        p[h] = (k < __shfl(turn, c[h], 64) ? c1 : c2) + k;
        ca[h] = __shfl(a, c[h], 64);
        cb[h] = __shfl(b, c[h], 64);
        cx[h] = __shfl(fx, c[h], 64);
        cy[h] = __shfl(fy, c[h], 64);
        cz[h] = __shfl(fz, c[h], 64);
        cdz[h] = __shfl(fdz, c[h], 64);
        cdphi[h] = __shfl(fdphi, c[h], 64);
        ctan[h] = __shfl(ftan, c[h], 64);
        cirr[h] = __shfl(firr, c[h], 64);
        csuu[h] = __shfl(suu, c[h], 64);
        csuw[h] = __shfl(suw, c[h], 64);
        csww[h] = __shfl(sww, c[h], 64);
      }
      // everything each pair can need, in one round trip for all NP pairs
      // (a pair past the end reads the round's first pair, which exists)
      float ph[NPT], hx[NPT], hy[NPT], hz[NPT], V[NPT][6];
      const int p_first = __builtin_amdgcn_readfirstlane(__shfl(p[0], 0, 64));
#pragma unroll
      for (int h = 0; h < NPT; ++h) {
        const int ps = valid[h] ? p[h] : p_first;
        const float4* hp = A.hpack + (size_t)ps * 3;
        const float4 u0 = hp[0], u1 = hp[1], u2 = hp[2];
        ph[h] = u0.x;
        hx[h] = u0.y;
        hy[h] = u0.z;
        hz[h] = u0.w;
        V[h][0] = u1.x;
        V[h][1] = u1.y;
        V[h][2] = u1.z;
        V[h][3] = u1.w;
        V[h][4] = u2.x;
        V[h][5] = u2.y;
      }
      // all loads in flight before the first test (the compiler would
      // otherwise wait for phi and issue the rest behind the phi test)
#pragma unroll
      for (int h = 0; h < NPT; ++h)
        asm volatile("" ::"v"(ph[h]), "v"(hx[h]), "v"(hy[h]), "v"(hz[h]), "v"(V[h][0]), "v"(V[h][1]), "v"(V[h][2]),
                     "v"(V[h][3]), "v"(V[h][4]), "v"(V[h][5]));
      bool acc[NPT];
      float c2[NPT];
#pragma unroll
      for (int h = 0; h < NPT; ++h) {
        acc[h] = false;
        c2[h] = 0.f;
        if (valid[h] && ph[h] >= ca[h] && ph[h] <= cb[h]) {
          scanned += 1;
          const float cr = cx[h] * hy[h] - cy[h] * hx[h], dt = cx[h] * hx[h] + cy[h] * hy[h];
          const bool in_phi =
              ctan[h] < 0.f ? fabsf(atan2f(cr, dt)) <= cdphi[h] : (dt > 0.f && fabsf(cr) <= ctan[h] * dt);
          if (fabsf(hz[h] - cz[h]) <= cdz[h] && in_phi) {
            // innovation in the tangent-plane frame and its chi2 (2 dof)
            tested += 1;
            const float ctx = -cy[h] * cirr[h], cty = cx[h] * cirr[h];
            const float r0 = ctx * (hx[h] - cx[h]) + cty * (hy[h] - cy[h]), r1 = hz[h] - cz[h];
            const float s00 = csuu[h] + ctx * ctx * V[h][0] + 2.f * ctx * cty * V[h][1] + cty * cty * V[h][3];
            const float s01 = csuw[h] + ctx * V[h][2] + cty * V[h][4];
            const float s11 = csww[h] + V[h][5];
            const float det = s00 * s11 - s01 * s01;
            if (s00 > 0.f && det > 0.f) {
              // (the hardware reciprocal: within a few ulp, no division sequence)
              c2[h] = (s11 * r0 * r0 - 2.f * s01 * r0 * r1 + s00 * r1 * r1) * k_rcp(det);
              acc[h] = c2[h] < chi2_cut;
            }
          }
        }
      }
      // the accepted hits into their seeds' pools
      bool pend[NPT], any = false;
#pragma unroll
      for (int h = 0; h < NPT; ++h) {
        pend[h] = acc[h];
        any = any || acc[h];
      }
      if (!__any(any)) continue;
      int sd[NPT];
      uint32_t ref[NPT];
#pragma unroll
      for (int h = 0; h < NPT; ++h) {
        if (acc[h]) po.seen[c[h]] = 1;
        sd[h] = c[h] * inv_s >> 16;
        ref[h] = ((uint32_t)(c[h] - sd[h] * gr.S) << 24) | (uint32_t)(p[h] - __shfl(e0, c[h], 64));
      }
      for (;;) {
        if (lim) {
#pragma unroll
          for (int h = 0; h < NPT; ++h) {
            const float ct = __shfl(thr, c[h], 64);  // (by all lanes)
            pend[h] = pend[h] && c2[h] <= ct;
          }
        }
        int at[NPT];
#pragma unroll
        for (int h = 0; h < NPT; ++h) at[h] = pend[h] ? atomicAdd(&po.cnt[sd[h]], 1) : po.full;
        unsigned long long pm = 0ull;
        int over = 0;  // a seed whose pool is full
#pragma unroll
        for (int h = 0; h < NPT; ++h) {
          if (at[h] < po.full) {
            po.e[sd[h] * po.stride + at[h]] = make_uint2(__float_as_uint(c2[h]), ref[h]);
            pend[h] = false;
          }
          const unsigned long long q = __ballot(pend[h]);
          if (q) over = __builtin_amdgcn_readlane(sd[h], (int)__builtin_ctzll(q));
          pm |= q;
        }
        if (!pm) break;
        pool_cut<T>(A, po, gr, over, lane, chi2, nhits, e0, thr, cut);
        lim = true;
      }
    }
    if (++r < Rmax) continue;
    if (!again) break;
    // the bounds of the wide candidates
    again = false;
    unsigned long long wm = __ballot(wide && rq.c2 < chi2_cut);
    unsigned long long redo = 0ull;  // lanes of the seeds to be searched again
    const unsigned long long gm = ((1ull << gr.S) - 1ull);
    while (wm) {
      const int s = __builtin_amdgcn_readlane(gr.sidx, (int)__builtin_ctzll(wm));
      const unsigned long long sm = gm << (s * gr.S);
      wm &= ~sm;
      pool_cut<T>(A, po, gr, s, lane, chi2, nhits, e0, thr, cut);
      lim = true;
      bool miss = false;
      if (gr.sidx == s && wide && rq.c2 < chi2_cut) {
        pruned = cut && thr < chi2_cut && (po.seen[lane] != 0 || hole_ok);
        miss = !pruned || thr > rq.c2;
        if (miss) rq.c2 = pruned ? thr : chi2_cut;
      }
      if (__any(miss)) redo |= sm;
    }
    const int R0 = rw.n();
    R = 0;
    if (!redo) break;
    if (redo >> lane & 1ull) {
      if (gr.slot == 0) po.cnt[gr.sidx] = 0;
      if (!pruned) po.seen[lane] = 0;
      if (wide && R0 > 0) {
        rq.set(rq.c2, suu, suw, sww);
        rw = rows_of(fz, fminf(fdz + kEpsZ, rq.dz(sww)), ku64<T>(A.z_half), nz);
      }
      R = pok ? rw.n() << sh : 0;
    }
    Rmax = wave_max(iters());
    r = -1;
  }
  __builtin_amdgcn_s_waitcnt(0);
  lds_order();
  seen = po.seen[lane] != 0;
}

// The seeds' best cap children (section 4.3): pool entries and holes ranked
// by one pass of comparisons.  Every child gets a 64-bit key (nhits, chi2,
// slot as in make_key, then the upper bits of its hit's chi2 and its place in
// the pool); lane `slot` of a seed takes every S-th child of the seed, counts
// the keys below each, and places those within the best cap + 1 in win.
// Keys that differ only in the place are a tie the key cannot order: such a
// seed's pool is put in exact order (pool_cut) and ranked again, where the
// place decides.  keys: [SEEDS][stride] u64, win: [SEEDS][cap + 1] u64.
//
// Ranking against every child of the seed costs some 2 instructions per
// comparison and no chain of dependent steps; popping the best of the
// candidates' sorted lists cap times was a chain of cap times three shuffle
// round trips and an LDS read (8 800 of a layer's 49 000 cycles, beside 2 500
// for sorting the lists and 8 500 for keeping them sorted).
// With the bounded search: 20 events of 20 000 tracks, build kernel FP64
// 8.87 -> 4.67 ms, FP32 one event 3.69 -> 0.42 ms (20 000 tracks, its slowest
// wave).
//
// Returns the number of children kept; n_all: children before the cut.
template <typename T, int NI>
__device__ inline void rank_items(const Pool& po, const Group& gr, const uint2* pe, uint64_t* kv, uint64_t* wv, int m,
                                  int mmax, int cap, T chi2, int nhits) {
  uint2 e[NI];
  T pc[NI];
  int pn[NI], rank[NI];
  uint64_t key[NI];
  // (each stage for all of the lane's children, so that its LDS operations
  // are in flight together)
#pragma unroll
  for (int t = 0; t < NI; ++t) {
    const int j = gr.slot + t * gr.S;
    e[t] = pe[gr.used && j < m ? j : 0];
  }
#pragma unroll
  for (int t = 0; t < NI; ++t) {
    const int src = gr.base + (gr.used && gr.slot + t * gr.S < m ? (int)(e[t].y >> 24) : gr.slot);
    pc[t] = shfl_t(chi2, src);
    pn[t] = __shfl(nhits, src, 64);
  }
#pragma unroll
  for (int t = 0; t < NI; ++t) {
    const int j = gr.slot + t * gr.S;
    const bool hit = (e[t].y & 0xFFFFFFu) != kNoHit;
    const float c2 = __uint_as_float(e[t].x);
    key[t] = ((uint64_t)(31 - pn[t] - (hit ? 1 : 0)) << 59) | ((uint64_t)chi2_bits((float)(pc[t] + (T)c2)) << 28) |
             ((uint64_t)(e[t].y >> 24) << 25) | ((uint64_t)(chi2_bits(c2) >> 12) << 6) | (uint64_t)j;
    if (!gr.used || j >= m) key[t] = kInfKey;
    if (gr.used && j < po.stride) kv[j] = key[t];
    rank[t] = 0;
  }
  lds_order();
  // (the keys past m are infinite up to NI S >= mmax, and the rest of the
  // stride is not read: both are multiples of 4 apart from the last round)
  for (int i = 0; i < mmax; i += 4) {
    uint64_t k[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) k[u] = kv[i + u];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (i + u >= NI * gr.S) k[u] = kInfKey;
#pragma unroll
      for (int t = 0; t < NI; ++t) rank[t] += k[u] < key[t] ? 1 : 0;
    }
  }
#pragma unroll
  for (int t = 0; t < NI; ++t)
    if (key[t] != kInfKey && rank[t] <= cap) wv[rank[t]] = key[t];
}
template <typename T>
__device__ inline int best_children(const BuildArgs& A, const Pool& po, const Group& gr, uint64_t* keys, uint64_t* win,
                                    int lane, T chi2, int nhits, int e0, bool hole_ok, bool& cut, uint2& child) {
  constexpr int NT = kPoolPerCap + 1;
  const int cap = A.cap, S = gr.S, sx = gr.used ? gr.sidx : 0;
  const unsigned long long gm = ((1ull << S) - 1ull) << gr.base;
  const unsigned long long hm = __ballot(hole_ok && gr.used) & gm;
  uint2* pe = po.e + sx * po.stride;
  uint64_t* kv = keys + sx * po.stride;
  uint64_t* wv = win + sx * (cap + 1);
  for (bool exact = false;;) {
    const int held = po.cnt[sx], m0 = held < po.full ? held : po.full;
    const int m = gr.used ? m0 + __builtin_popcountll(hm) : 0;
    if (hole_ok && gr.used)
      pe[m0 + __builtin_popcountll(hm & ((1ull << lane) - 1ull))] = make_uint2(0u, ((uint32_t)gr.slot << 24) | kNoHit);
    lds_order();
    const int mmax = wave_max(m);
    if (mmax <= 2 * S) rank_items<T, 2>(po, gr, pe, kv, wv, m, mmax, cap, chi2, nhits);
    else if (mmax <= 4 * S) rank_items<T, 4>(po, gr, pe, kv, wv, m, mmax, cap, chi2, nhits);
    else rank_items<T, NT>(po, gr, pe, kv, wv, m, mmax, cap, chi2, nhits);
    lds_order();
    const bool kept = gr.used && gr.slot < m;  // (slot < cap)
    const uint64_t k0 = wv[kept ? gr.slot : 0];
    const bool tie = kept && gr.slot + 1 < m && (k0 >> 6) == (wv[kept ? gr.slot + 1 : 0] >> 6);
    unsigned long long tm = exact ? 0ull : __ballot(tie);
    if (!tm) {
      child = pe[kept ? (int)(k0 & 63) : 0];
      cut = cut || m > cap;
      return m < cap ? m : cap;
    }
    while (tm) {
      const int s = __builtin_amdgcn_readlane(gr.sidx, (int)__builtin_ctzll(tm));
      tm &= ~(((1ull << S) - 1ull) << (s * S));
      float thr;
      pool_cut<T>(A, po, gr, s, lane, chi2, nhits, e0, thr, cut);
    }
    exact = true;
  }
}

// Waves per SIMD the register allocation aims at.  The build waits on
// memory and LDS most of the time, so a second resident wave pays even where
// it costs register spills (FP64: measured 26 % faster than one wave).  The
// macros allow a rebuild to compare.
#ifndef KF_BUILD_F32_WAVES
#define KF_BUILD_F32_WAVES 2
#endif
#ifndef KF_BUILD_F64_WAVES
#define KF_BUILD_F64_WAVES 2
#endif
#ifndef KF_BUILD_F64_LEARNED_WAVES
#define KF_BUILD_F64_LEARNED_WAVES 2
#endif

// Pairs per lane and round: NP in every build (learned FP64 builds of 32 events
// 11.45 ms with one, 10.79 with two, hybrid state 11.40 and 11.04; the plain
// hybrid FP64 build of 20 events 5.21 and 5.00).  The macro allows a rebuild to
// compare.
#ifndef KF_LEARNED_F64_NPT
#define KF_LEARNED_F64_NPT 2
#endif
template <typename T, bool LEARNED>
constexpr int NPT_OF = (sizeof(T) == 8 && LEARNED) ? KF_LEARNED_F64_NPT : NP;

template <typename T, bool LEARNED, bool HYB>
__global__ void __launch_bounds__(256, (sizeof(T) == 4 ? KF_BUILD_F32_WAVES
                                                       : (LEARNED ? KF_BUILD_F64_LEARNED_WAVES : KF_BUILD_F64_WAVES)))
    build_kernel(BuildArgs A) {
  const int S = A.cap;           // lanes per seed
  const int SEEDS = 64 / S;      // seeds per wave
  extern __shared__ __align__(16) uint32_t lds[];
  const int lane = threadIdx.x & 63;
  // the wave index as a uniform value in FP64 builds: the per-wave addresses
  // derived from it then stay in scalar registers (the FP32 build measured from
  // 1 % faster to 2 % slower with it)
  const int wave = sizeof(T) == 8 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : (int)(threadIdx.x >> 6);
  const int nwaves = blockDim.x >> 6;
  const int LB = A.n_layers - A.first_layer;  // searched layers
  const LdsPlan lp = lds_plan(LB, nwaves, S, (int)sizeof(T), LEARNED, HYB);
  constexpr int NPL = xs_npl((int)sizeof(T), LEARNED, HYB);
  constexpr bool XS = NPL >= 0;  // xs in LDS
  char* base = (char*)lds;
  // this wave's back-pointer table (written once per new candidate and layer,
  // read once per seed at the end)
  uint32_t* hist = A.hist + ((size_t)blockIdx.x * nwaves + wave) * LB * 64;
  // the state before a layer's prediction, in the output precision, for the
  // finished record: entry k of 27 (the stash, then the first half of xs);
  // after the records of a layer the same memory holds the children's keys
  constexpr int NST = XS ? 21 - NPL : 27, NX2 = XS ? 6 + NPL : 0;
  float* stash = (float*)(base + lp.stash) + (size_t)wave * NST * 64;
  T* xs = (T*)(base + lp.xs) + (size_t)wave * NX2 * 64;
  auto before = [&](int k) -> float& { return k < NST ? stash[k * 64 + lane] : ((float*)xs)[(k - NST) * 64 + lane]; };
  uint64_t* keys = XS && !LEARNED ? (uint64_t*)xs : (uint64_t*)stash;
  uint64_t* win = !XS || HYB ? (LEARNED && XS ? (uint64_t*)xs : keys + 512) : (LEARNED ? (uint64_t*)xs : (uint64_t*)stash);
  // the last NXL covariance entries of the prediction, in FP64 builds kept in
  // the second half of xs during the hit search
  constexpr int NXL = NX2 / 2;
  T* xp = xs + NXL * 64;
  float* fin = (float*)(base + lp.rec) + (size_t)wave * SEEDS * 27;
  int32_t* finm = (int32_t*)(base + lp.recf) + (size_t)wave * SEEDS * 5;
  // per wave: the network buffer, or (after the network has run) the pools
  char* wave_tl = base + lp.tl + (size_t)wave * lp.tl_stride;
  uint16_t* mlp_buf = (uint16_t*)wave_tl;
  Pool po;
  po.e = (uint2*)wave_tl;
  po.cnt = (int32_t*)(base + lp.pub + (size_t)wave * pub_bytes(S));
  po.seen = (uint8_t*)(po.cnt + SEEDS);
  po.stride = (kPoolPerCap + 1) * S;
  po.full = kPoolPerCap * S;
  int8_t* start = (int8_t*)(base + lp.acc) + (size_t)wave * 64 * NP;
  (void)mlp_buf;
  const int sidx = lane / S, slot = lane - (lane / S) * S, sbase = sidx * S;
  const bool lane_used = sidx < SEEDS;
  const Group gr = {sidx, sbase, slot, S, lane_used};

  if (A.start_tick && lane == 0) atomicMin((unsigned long long*)A.start_tick, (unsigned long long)wall_clock64());

  for (;;) {
    int grp = 0;
    if (lane == 0) grp = atomicAdd(A.queue, 1);
    grp = __shfl(grp, 0, 64);
    if (grp >= A.n_groups) break;
    const int gi = grp * SEEDS + sidx;
    int seed = (lane_used && gi < A.n_seeds) ? (A.seed_order ? A.seed_order[gi] : gi) : -1;
    int ev = (seed >= 0 && seed < A.n_seeds && A.seed_event) ? A.seed_event[seed] : 0;
    // caller-supplied indices outside their ranges: the seed is skipped
    const bool seed_ok = seed >= 0 && seed < A.n_seeds && ev >= 0 && ev < A.n_events;
    if (!seed_ok) { seed = 0; ev = 0; }
    const int q = seed_ok ? A.q[seed] : 1;
    // first sorted position of the event
    const int e0 = A.offsets[(size_t)ev * A.n_layers * ((size_t)A.n_phi * A.n_z + 1)];
    // candidate state
    T X[6], P[21];
#pragma unroll
    for (int k = 0; k < 6; ++k) X[k] = seed_ok ? (T)A.seed_par[(size_t)k * A.ld + seed] : T(0);
#pragma unroll
    for (int k = 0; k < 21; ++k) P[k] = seed_ok ? (T)A.seed_cov[(size_t)k * A.ld + seed] : T(0);
    if constexpr (HYB) {  // the seed in the hybrid state
      if (seed_ok) {
        T Y[6], B[9];
        hyb_from_cart(X, q, Y, B);
        congruence_mom(P, B);
#pragma unroll
        for (int k = 0; k < 6; ++k) X[k] = Y[k];
      }
    }
    T chi2 = 0;
    int nhits = 0, holes = 0;
    bool ontrack = true;
    int n_active = seed_ok ? 1 : 0;
    int seed_status = 0;
    if (lane_used && slot == 0) finm[sidx * 5 + 0] = 0;
    // a non-finite seed, or one whose event holds more hits than 24-bit
    // event-local indices can name, is its own (finished) result
    const int bad = !seed_ok ? 0
                    : event_too_large(A.offsets, ev, A.n_layers, A.n_phi * A.n_z) ? KF_EVENT_TOO_LARGE
                    : !(all_finite(X, 6) && all_finite(P, 21))                     ? KF_NONFINITE
                                                                                   : 0;
    if (bad) {
      if (slot == 0) {
        finm[sidx * 5 + 0] = 1; finm[sidx * 5 + 1] = 0; finm[sidx * 5 + 2] = bad;
        finm[sidx * 5 + 3] = A.first_layer - 1; finm[sidx * 5 + 4] = 0;
        for (int k = 0; k < 6; ++k) fin[sidx * 27 + k] = (float)X[k];
        for (int k = 0; k < 21; ++k) fin[sidx * 27 + 6 + k] = (float)P[k];
      }
      n_active = 0;
    }
    T fin_chi2_reg = 0;  // chi2 of the finished record, kept by slot 0 of the seed
    unsigned cnt_pred = 0, cnt_scan = 0, cnt_chi2 = 0, cnt_upd = 0;
    int last_l = A.first_layer - 1;
    for (int l = A.first_layer; l < A.n_layers; ++l) {
      // all seeds of the wave done?
      if (!__any(n_active > 0)) break;
      last_l = l;
      const bool live = slot < n_active;
      if (live) {
#pragma unroll
        for (int k = 0; k < 6; ++k) before(k) = (float)X[k];
#pragma unroll
        for (int k = 0; k < 21; ++k) before(6 + k) = (float)P[k];
      }
      T Xp[6], Pp[21];
      int rc = 1;
      if (live) {
        if constexpr (HYB)
          rc = predict_hyb<T>(X, P, (T)A.r[l], (T)ku64<T>(A.bz), (T)ku64<T>(A.z_half), (T)ku64<T>(A.x_over_x0),
                              (T)ku64<T>(A.mass), Xp, Pp);
        else
          rc = predict<T>(X, P, kv64<T>(q), (T)A.r[l], (T)ku64<T>(A.bz), (T)ku64<T>(A.z_half),
                          (T)ku64<T>(A.x_over_x0), (T)ku64<T>(A.mass), Xp, Pp);
      }
      else {
#pragma unroll
        for (int k = 0; k < 6; ++k) Xp[k] = T(0);
#pragma unroll
        for (int k = 0; k < 21; ++k) Pp[k] = T(0);
      }
      const bool pok = live && rc == 0;
      // plain window from the predicted covariance
      T w_rphi = T(0), w_z = T(0);
      const T R = (T)A.r[l];
      if (pok) {
        const T rr = k_sqrt(Xp[0] * Xp[0] + Xp[1] * Xp[1]);
        const T tx = -Xp[1] / rr, ty = Xp[0] / rr;
        const T Suu = tx * tx * Pp[ut(0, 0)] + T(2) * tx * ty * Pp[ut(0, 1)] + ty * ty * Pp[ut(1, 1)] +
                      sq((T)ku64<T>(A.win_sig_rphi));
        const T Sww = Pp[ut(2, 2)] + sq((T)ku64<T>(A.win_sig_z));
        w_rphi = (T)ku64<T>(A.nsigma) * k_sqrt(Suu);
        w_z = (T)ku64<T>(A.nsigma) * k_sqrt(Sww);
        if (A.dump && ontrack && A.true_hits) {
          const int th = A.true_hits[(size_t)l * A.ld + seed];
          if (th >= 0) {
            const int row = atomicAdd(A.dump_count, 1);
            if (row < A.dump_capacity) {
              float* d = A.dump + (size_t)row * KFMLP_DUMP_ROW;
              if constexpr (HYB) {
                // the features the network reads: the Cartesian prediction
                T Xc[6], Am[9], Pc[21];
                (void)cart_from_hyb(Xp, Xc, Am);
                for (int k = 0; k < 21; ++k) Pc[k] = Pp[k];
                congruence_mom(Pc, Am);
                for (int k = 0; k < 6; ++k) d[k] = (float)Xc[k];
                for (int k = 0; k < 21; ++k) d[6 + k] = (float)Pc[k];
              } else {
                for (int k = 0; k < 6; ++k) d[k] = (float)Xp[k];
                for (int k = 0; k < 21; ++k) d[6 + k] = (float)Pp[k];
              }
              const T mx = (T)A.true_xyz[((size_t)l * 3 + 0) * A.ld + seed];
              const T my = (T)A.true_xyz[((size_t)l * 3 + 1) * A.ld + seed];
              const T mz = (T)A.true_xyz[((size_t)l * 3 + 2) * A.ld + seed];
              const T dph = k_atan2(Xp[0] * my - Xp[1] * mx, Xp[0] * mx + Xp[1] * my);
              d[27] = (float)(R * fabs(dph));
              d[28] = (float)fabs(mz - Xp[2]);
              // the plain half-widths this candidate's window has (the gates
              // of the learned window are set from them)
              d[29] = (float)w_rphi;
              d[30] = (float)w_z;
              d[31] = __int_as_float((int)(((uint32_t)seed << 8) | ((uint32_t)l << 3) | (uint32_t)slot));
            }
          }
        }
      }
      if constexpr (LEARNED) {
        // learned window where the plain one is wide (either half-width above
        // its gate): the wave evaluates the network on those slots only
        const bool gated = pok && (w_rphi > (T)A.mlp[KFMLP_OFF_GATE] || w_z > (T)A.mlp[KFMLP_OFF_GATE + 1]);
        // the features rounded to FP32 first and pinned there by an empty
        // asm: converted inside the row writes instead, the FP64 build's
        // register allocation spilled twice as much
        float feat[27];
        if constexpr (HYB) {
          // the network reads the Cartesian prediction: convert the hybrid
          // one (state, and covariance through d(X)/d(Y))
          T Xc[6], Am[9], Pc[21];
          (void)cart_from_hyb(Xp, Xc, Am);
#pragma unroll
          for (int k = 0; k < 21; ++k) Pc[k] = Pp[k];
          congruence_mom(Pc, Am);
#pragma unroll
          for (int k = 0; k < 27; ++k) feat[k] = (float)(k < 6 ? Xc[k] : Pc[k - 6]);
        } else {
#pragma unroll
          for (int k = 0; k < 27; ++k) feat[k] = (float)(k < 6 ? Xp[k] : Pp[k - 6]);
        }
#pragma unroll
        for (int k = 0; k < 27; ++k) asm volatile("" : "+v"(feat[k]));
        const uint64_t act = kfmlp::wave_stage(A.mlp, mlp_buf, [&](int k) { return feat[k]; }, gated);
        float o[2] = {0.f, 0.f};
        if (act) kfmlp::wave_tiles(A.mlp, mlp_buf, act, o);
        if (gated) {
          const float kap = A.mlp[KFMLP_OFF_KAPPA];
          float wl[2] = {A.mlp[KFMLP_OFF_SCALE] * kfmlp::softplus(o[0]),
                         A.mlp[KFMLP_OFF_SCALE + 1] * kfmlp::softplus(o[1])};
          wl[0] *= kap;
          wl[1] *= kap;
          if (!(wl[0] < A.mlp[KFMLP_OFF_FLOOR])) w_rphi = (T)wl[0];
          if (!(wl[1] < A.mlp[KFMLP_OFF_FLOOR + 1])) w_z = (T)wl[1];
        }
      }
      const T dphi_w = pok ? w_rphi / R : T(0), dz_w = pok ? w_z : T(0);
      const bool hole_ok = pok && holes < A.max_holes;
      bool seen = false, cut = false;
#pragma unroll
      for (int k = 0; k < NXL; ++k) xp[k * 64 + lane] = Pp[21 - NXL + k];
      coop_scan<T, NPT_OF<T, LEARNED>>(A, kv64<T>(ev), e0, l, pok, Xp, Pp, dphi_w, dz_w, chi2, nhits, hole_ok, gr, po,
                                       start, lane, seen, cut, cnt_scan, cnt_chi2);
      const int nchild = (seen ? 1 : 0) + (hole_ok ? 1 : 0);
      // Finished candidates of this layer (live, no child) compete for the
      // record.  Slot 0 has the seed's most hits; where a candidate with as
      // many found a hit, the seed ends with more than any that stops here
      // has, which then need not compete.
      const int top_hits = __shfl(nhits, sbase, 64);
      const unsigned long long ahead = __ballot(live && seen && nhits == top_hits) & (((1ull << S) - 1ull) << sbase);
      const bool stopped = live && nchild == 0 && ahead == 0ull;
      if (__any(stopped)) {
        uint64_t fk = stopped ? make_key(nhits, (float)chi2, slot, 0) : kInfKey;
        const uint64_t best = group_min(fk, sbase, slot, S, lane_used);
        const int ws = (int)((best >> 24) & 7);
        const int wl_ = sbase + ws;
        // winner's chi2 in T and its fields
        const T wc2 = shfl_t(chi2, wl_);
        const int wn = __shfl(nhits, wl_, 64);
        const int wst = __shfl(live && rc ? rc : 0, wl_, 64);
        const T fc2 = shfl_t(fin_chi2_reg, sbase);
        if (best != kInfKey) {
          const int fvalid = finm[sidx * 5 + 0];
          const int fn = finm[sidx * 5 + 1];
          const bool take = !fvalid || wn > fn || (wn == fn && wc2 < fc2);
          if (take) {
            if (slot == ws) {
              for (int k = 0; k < 27; ++k) fin[sidx * 27 + k] = before(k);
              finm[sidx * 5 + 0] = 1; finm[sidx * 5 + 1] = wn; finm[sidx * 5 + 2] = wst;
              finm[sidx * 5 + 3] = l - 1; finm[sidx * 5 + 4] = ws;
            }
            if (slot == 0) fin_chi2_reg = wc2;
          }
        }
      }
      // the seed's best children into slots 0..cap-1
      lds_order();
      uint2 child;
      const int n_new =
          best_children<T>(A, po, gr, keys, win, lane, chi2, nhits, e0, hole_ok, cut, child);
      const bool is_hole = (child.y & 0xFFFFFFu) == kNoHit;
      const int my_parent = lane_used && slot < n_new ? (int)(child.y >> 24) : -1;
      if (lane_used && cut) seed_status |= KF_CAP_TRUNC;
      // new slots pull the parent's predicted state
      const int src = sbase + (my_parent >= 0 ? my_parent : slot);
#pragma unroll
      for (int k = 0; k < 6; ++k) X[k] = shfl_t(Xp[k], src);
#pragma unroll
      for (int k = 0; k < 21; ++k) P[k] = k < 21 - NXL ? shfl_t(Pp[k], src) : xp[(k - 21 + NXL) * 64 + src];
      const T pchi2 = shfl_t(chi2, src);
      const int pnh = __shfl(nhits, src, 64), pho = __shfl(holes, src, 64);
      const bool pon = __shfl((int)ontrack, src, 64) != 0;
      // (slots without a child keep values that nothing reads again: the
      // state need not be held through the layer for them)
      uint32_t my_orig = kHoleIdx;
      if (my_parent >= 0) {
        if (!is_hole) {
          const float4* hp = A.hpack + (size_t)(e0 + (int)(child.y & 0xFFFFFFu)) * 3;
          const float4 u0 = hp[0], u1 = hp[1], u2 = hp[2];
          const T hx = (T)u0.y, hy = (T)u0.z, hz = (T)u0.w;
          const T V[6] = {(T)u1.x, (T)u1.y, (T)u1.z, (T)u1.w, (T)u2.x, (T)u2.y};
          my_orig = __float_as_uint(u2.z);
          Innov<T> in;
          innovation<T>(X, P, hx, hy, hz, V, in);
          apply_update<T>(X, P, in);
        }
        chi2 = is_hole ? pchi2 : pchi2 + (T)__uint_as_float(child.x);
        nhits = is_hole ? pnh : pnh + 1;
        holes = is_hole ? pho + 1 : pho;
        if (A.dump && A.true_hits) {
          const int th = seed_ok ? A.true_hits[(size_t)l * A.ld + seed] : -1;
          ontrack = pon && (is_hole || (int)my_orig == th);
        }
        hist[(l - A.first_layer) * 64 + lane] = pack_hist(my_parent, my_orig);
      }
      cnt_pred += live ? 1u : 0u;
      cnt_upd += my_parent >= 0 && !is_hole ? 1u : 0u;
      n_active = n_new;
    }
    if (A.counters) {
      unsigned long long c[4] = {cnt_pred, cnt_scan, cnt_chi2, cnt_upd};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        unsigned long long v = c[k];
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m, 64);
        if (lane == 0) atomicAdd(&A.counters[k], v);
      }
    }
    // final choice: best active (slot order), then the finished record
    {
      const bool act = slot < n_active;
      const uint64_t k = act ? make_key(nhits, (float)chi2, slot, 0) : kInfKey;
      const uint64_t best = group_min(k, sbase, slot, S, lane_used);
      const int blane = sbase + (best != kInfKey ? (int)((best >> 24) & 7) : 0);
      const int bslot = best != kInfKey ? blane - sbase : -1;
      const T bc2 = shfl_t(chi2, blane);
      const int bn = __shfl(nhits, blane, 64);
      const T fc2 = shfl_t(fin_chi2_reg, sbase);
      const int fvalid = lane_used ? finm[sidx * 5 + 0] : 0;
      const int fn = lane_used ? finm[sidx * 5 + 1] : 0;
      const bool use_fin = fvalid && (bslot < 0 || fn > bn || (fn == bn && fc2 < bc2));
      if (seed_ok) {
        // state: the best lane writes its own; slot 0 writes the record
        if (!use_fin && slot == bslot) {
          for (int k2 = 0; k2 < 6; ++k2) A.out_par[(size_t)k2 * A.ld + seed] = (float)X[k2];
          for (int k2 = 0; k2 < 21; ++k2)
            A.out_cov[(size_t)k2 * A.ld + seed] = (float)P[k2];
          A.out_chi2[seed] = (float)chi2;
          A.out_nhits[seed] = nhits;
          A.out_status[seed] = seed_status;
        }
        if (use_fin && slot == 0) {
          for (int k2 = 0; k2 < 6; ++k2) A.out_par[(size_t)k2 * A.ld + seed] = fin[sidx * 27 + k2];
          for (int k2 = 0; k2 < 21; ++k2) A.out_cov[(size_t)k2 * A.ld + seed] = fin[sidx * 27 + 6 + k2];
          A.out_chi2[seed] = (float)fin_chi2_reg;
          A.out_nhits[seed] = fn;
          A.out_status[seed] = finm[sidx * 5 + 2] | seed_status;
        }
        // hit list: walk the history backwards (one lane per seed)
        if (slot == 0) {
          int from_l = use_fin ? finm[sidx * 5 + 3] : last_l;
          int s = use_fin ? finm[sidx * 5 + 4] : bslot;
          if (bslot < 0 && !use_fin) from_l = A.first_layer - 1;
          for (int l = A.n_layers - 1; l > from_l; --l) A.out_hits[(size_t)(l - A.first_layer) * A.ld + seed] = -1;
          for (int l = from_l; l >= A.first_layer; --l) {
            const uint32_t h = hist[(l - A.first_layer) * 64 + sbase + s];
            const uint32_t o = h & 0xFFFFFFu;
            A.out_hits[(size_t)(l - A.first_layer) * A.ld + seed] = o == 0xFFFFFFu ? -1 : (int32_t)o;
            s = (int)(h >> 24);
          }
        }
        // per-event completion
        if (slot == 0 && A.event_done_ticks) {
          const int done = atomicAdd(&A.event_done[ev], 1);
          if (done == A.event_n_seeds[ev] - 1) A.event_done_ticks[ev] = (int64_t)wall_clock64();
        }
      }
    }
  }
}

int refine_of(const kf_build_params* bp) { return bp->phi_refine > 0 ? bp->phi_refine : 64; }

// the launch shape of the last kf_build call of this host thread
thread_local kf_build_launch_info g_last_launch = {};

template <typename T, bool LEARNED, bool HYB>
int launch(const BuildArgs& A, int lanes, int blocks, int hist_waves, hipStream_t s) {
  const int LB = A.n_layers - A.first_layer;
  int dev = 0, max_lds = 0;
  if (kf_check(hipGetDevice(&dev))) return KF_E_HIP;
  if (kf_check(hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev))) return KF_E_HIP;
  auto plan = [&](int ln) { return lds_plan(LB, ln / 64, A.cap, (int)sizeof(T), LEARNED, HYB).total; };
  if (lanes == 0) {  // automatic
    lanes = plan_lanes(LB, A.cap, (int)sizeof(T), LEARNED, HYB, (size_t)max_lds);
    if (lanes == 0) return KF_E_UNSUPPORTED;
  }
  const int nwaves = lanes / 64;
  const size_t lds = plan(lanes);
  if (lds > (size_t)max_lds) return KF_E_UNSUPPORTED;
  if (lds > (size_t)64 * 1024 &&
      kf_check(hipFuncSetAttribute((const void*)build_kernel<T, LEARNED, HYB>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)))
    return KF_E_HIP;
  int cus = 0, per = 0;
  if (kf_check(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev))) return KF_E_HIP;
  if (kf_check(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, build_kernel<T, LEARNED, HYB>, lanes, lds)))
    return KF_E_HIP;
  if (blocks <= 0) blocks = cus * (per > 0 ? per : 1);
  const int need = (A.n_groups + nwaves - 1) / nwaves;
  if (blocks > need) blocks = need;
  if (blocks > hist_waves / nwaves) blocks = hist_waves / nwaves;  // history tables in the workspace
  if (blocks < 1) return KF_E_WORKSPACE;
  g_last_launch.lanes_per_block = lanes;
  g_last_launch.blocks = blocks;
  g_last_launch.lds_bytes = (int32_t)lds;
  g_last_launch.resident_blocks_per_cu = per;
  g_last_launch.max_lds_per_block = max_lds;
  hipLaunchKernelGGL((build_kernel<T, LEARNED, HYB>), dim3(blocks), dim3(lanes), lds, s, A);
  return kf_check_launch();
}

}  // namespace

extern "C" int kf_build_last_launch(kf_build_launch_info* info) {
  if (!info) return KF_E_INVALID_ARG;
  *info = g_last_launch;
  return KF_OK;
}

extern "C" size_t kf_build_workspace_bytes(const kf_build_params* bp, const kf_hits* hits, int32_t n_seeds) {
  (void)n_seeds;
  if (!bp || !hits || hits->n_events < 1 || hits->n_layers < 1 || hits->n_phi < 1 || hits->n_z < 1) return 0;
  if (bp->first_layer < 1 || bp->first_layer >= hits->n_layers) return 0;
  const size_t LB = (size_t)(hits->n_layers - bp->first_layer);
  if (hits->n_hits < 0) return 0;
  return ws_head_bytes(hits->n_events) +
         ((fine_bytes(hits->n_events, hits->n_layers, hits->n_phi, hits->n_z, refine_of(bp)) + 255) & ~(size_t)255) +
         pack_bytes(hits->n_hits) + (size_t)hist_waves_of_device() * LB * 64 * 4;
}

extern "C" int kf_build(const kf_geometry* g, const kf_build_params* bp, const kf_hits* hits, int32_t n_seeds,
                        int32_t ld, const float* seed_par, const float* seed_cov, const int8_t* q, int32_t* out_hits,
                        float* out_par, float* out_cov, float* out_chi2, int32_t* out_nhits, int32_t* out_status,
                        const kf_build_extra* extra, void* ws, size_t ws_bytes, void* stream) {
  if (kf_check_geometry(g) || !bp || !hits) return KF_E_INVALID_ARG;
  if (n_seeds < 0 || ld < n_seeds) return KF_E_INVALID_ARG;
  if (bp->first_layer < 1 || bp->first_layer >= g->n_layers) return KF_E_INVALID_ARG;
  if (bp->cand_cap < 1 || bp->max_holes < 0 || !(bp->nsigma > 0.f) || !(bp->win_sig_rphi > 0.f) ||
      !(bp->win_sig_z > 0.f))
    return KF_E_INVALID_ARG;
  if (bp->cand_cap > 8) return KF_E_UNSUPPORTED;
  if (bp->phi_refine < 0 || bp->phi_refine > 64) return KF_E_INVALID_ARG;
  if (bp->arith != KF_ARITH_F32 && bp->arith != KF_ARITH_F64) return KF_E_INVALID_ARG;
  if (bp->window_mode != 0 && bp->window_mode != 1) return KF_E_INVALID_ARG;
  if (bp->window_mode == 1 && !bp->mlp) return KF_E_INVALID_ARG;
  if (bp->state != 0 && bp->state != 1) return KF_E_INVALID_ARG;
  if (hits->n_layers != g->n_layers || hits->n_events < 1 || hits->n_phi < 1 || hits->n_z < 1 || hits->n_hits < 0)
    return KF_E_INVALID_ARG;
  if (n_seeds == 0) return KF_OK;
  if (!seed_par || !seed_cov || !q || !out_hits || !out_par || !out_cov || !out_chi2 || !out_nhits || !out_status)
    return KF_E_INVALID_ARG;
  if (!hits->offsets || (hits->n_hits > 0 && (!hits->x || !hits->y || !hits->z || !hits->phi || !hits->cov ||
                                               !hits->orig)))
    return KF_E_INVALID_ARG;
  kf_build_extra ex = {};
  if (extra) ex = *extra;
  if (hits->n_events > 1 && !ex.seed_event) return KF_E_INVALID_ARG;
  if (ex.event_done_ticks && !ex.event_n_seeds) return KF_E_INVALID_ARG;
  if (ex.dump && (!ex.dump_count || !ex.true_hits || !ex.true_xyz || ex.dump_capacity < 0)) return KF_E_INVALID_ARG;
  const int refine = refine_of(bp);
  if ((int64_t)hits->n_phi * refine > (1 << 20)) return KF_E_UNSUPPORTED;
  const size_t need = kf_build_workspace_bytes(bp, hits, n_seeds);
  if (!ws || ws_bytes < need || ((uintptr_t)ws & 255)) return KF_E_WORKSPACE;
  const int lanes = bp->lanes_per_block;
  if (lanes != 0 && lanes != 64 && lanes != 128 && lanes != 256) return KF_E_UNSUPPORTED;

  BuildArgs A;
  A.n_layers = g->n_layers;
  for (int i = 0; i < 32; ++i) A.r[i] = g->r[i];
  A.z_half = g->z_half; A.bz = g->bz; A.x_over_x0 = g->x_over_x0; A.mass = g->mass;
  A.chi2_cut = bp->chi2_cut; A.max_holes = bp->max_holes; A.cap = bp->cand_cap;
  A.nsigma = bp->nsigma; A.win_sig_rphi = bp->win_sig_rphi; A.win_sig_z = bp->win_sig_z;
  A.first_layer = bp->first_layer; A.window_mode = bp->window_mode; A.mlp = (const float*)bp->mlp;
  A.n_events = hits->n_events; A.n_phi = hits->n_phi; A.n_z = hits->n_z; A.offsets = hits->offsets;
  A.n_hits = hits->n_hits;
  A.refine = refine;
  const size_t fine_off = ws_head_bytes(hits->n_events);
  A.fine = (const int32_t*)((char*)ws + fine_off);
  const size_t pack_off =
      fine_off + ((fine_bytes(hits->n_events, hits->n_layers, hits->n_phi, hits->n_z, refine) + 255) & ~(size_t)255);
  A.hpack = (const float4*)((char*)ws + pack_off);
  const size_t hist_off = pack_off + pack_bytes(hits->n_hits);
  A.hist = (uint32_t*)((char*)ws + hist_off);
  const size_t LBw = (size_t)(g->n_layers - bp->first_layer) * 64 * 4;
  const int hist_waves = (int)((ws_bytes - hist_off) / LBw);
  const int seeds_per_wave = 64 / bp->cand_cap;
  A.n_seeds = n_seeds; A.ld = ld; A.n_groups = (n_seeds + seeds_per_wave - 1) / seeds_per_wave;
  A.seed_par = seed_par; A.seed_cov = seed_cov; A.q = q;
  A.seed_event = ex.seed_event; A.seed_order = ex.seed_order;
  A.out_hits = out_hits; A.out_par = out_par; A.out_cov = out_cov; A.out_chi2 = out_chi2;
  A.out_nhits = out_nhits; A.out_status = out_status;
  A.event_n_seeds = ex.event_n_seeds; A.event_done_ticks = ex.event_done_ticks; A.start_tick = ex.start_tick;
  A.true_hits = ex.true_hits; A.true_xyz = ex.true_xyz; A.dump = ex.dump; A.dump_count = ex.dump_count;
  A.dump_capacity = ex.dump_capacity;
  A.counters = (unsigned long long*)ex.counters;
  A.queue = (int32_t*)ws;
  A.event_done = (int32_t*)((char*)ws + 256);
  hipStream_t s = (hipStream_t)stream;
  if (int rc = launch_prep(hits, refine, A.fine, A.hpack, A.queue, A.event_done, A.start_tick, s)) return rc;
  if (bp->arith == KF_ARITH_F64)
    return bp->state == 1
               ? (bp->window_mode == 1 ? launch<double, true, true>(A, lanes, bp->persistent_blocks, hist_waves, s)
                                       : launch<double, false, true>(A, lanes, bp->persistent_blocks, hist_waves, s))
               : (bp->window_mode == 1 ? launch<double, true, false>(A, lanes, bp->persistent_blocks, hist_waves, s)
                                       : launch<double, false, false>(A, lanes, bp->persistent_blocks, hist_waves, s));
  return bp->state == 1
             ? (bp->window_mode == 1 ? launch<float, true, true>(A, lanes, bp->persistent_blocks, hist_waves, s)
                                     : launch<float, false, true>(A, lanes, bp->persistent_blocks, hist_waves, s))
             : (bp->window_mode == 1 ? launch<float, true, false>(A, lanes, bp->persistent_blocks, hist_waves, s)
                                     : launch<float, false, false>(A, lanes, bp->persistent_blocks, hist_waves, s));
}

// ------------------------------------------------- allocation-free variant
//
// kf_build_noalloc runs kf_build with its workspace in `scratch`, a static
// device array of this library: every GPU the library runs on holds its own
// copy (kScratchBytes) until the process ends.  In host code the array's
// name stands for a host-side shadow, not a device address: the device
// address is looked up once per device (hipGetSymbolAddress, with that
// device current) and only that pointer is handed to kernels.  What the
// build needs zeroed (queue head, per-event counters) is cleared by a kernel
// of every call; the fine index and the packed hits are rebuilt by every
// call; so the contents left by the previous call do not matter.  Calls that
// overlap on one GPU share the array and race.

static constexpr size_t kScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

// device address of this device's copy of `scratch`
int scratch_of_current_device(void** out) {
  int dev = 0;
  if (kf_check(hipGetDevice(&dev))) return KF_E_HIP;
  if (dev < 0 || dev >= kMaxDevices) return kf_fail(KF_E_UNSUPPORTED, "kf_build_noalloc: device index above 63");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    if (kf_check(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)))) return KF_E_HIP;
    if (!p) return kf_fail(KF_E_HIP, "kf_build_noalloc: no device address for the scratch array");
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return KF_OK;
}

}  // namespace

extern "C" size_t kf_build_noalloc_max_bytes(void) { return kScratchBytes; }

extern "C" int kf_build_noalloc(const kf_geometry* g, const kf_build_params* bp, const kf_hits* hits,
                                int32_t n_seeds, int32_t ld, const float* seed_par, const float* seed_cov,
                                const int8_t* q, int32_t* out_hits, float* out_par, float* out_cov, float* out_chi2,
                                int32_t* out_nhits, int32_t* out_status, const kf_build_extra* extra, void* stream) {
  if (kf_check_geometry(g) || !bp || !hits) return KF_E_INVALID_ARG;
  const size_t need = kf_build_workspace_bytes(bp, hits, n_seeds);
  if (need == 0) return KF_E_INVALID_ARG;
  if (need > kScratchBytes) {
    char msg[160];
    snprintf(msg, sizeof(msg), "kf_build_noalloc: this call needs %zu workspace bytes, the static scratch holds %zu",
             need, kScratchBytes);
    return kf_fail(KF_E_WORKSPACE, msg);
  }
  void* ws = nullptr;
  if (int rc = scratch_of_current_device(&ws)) return rc;
  return kf_build(g, bp, hits, n_seeds, ld, seed_par, seed_cov, q, out_hits, out_par, out_cov, out_chi2, out_nhits,
                  out_status, extra, ws, kScratchBytes, stream);
}
