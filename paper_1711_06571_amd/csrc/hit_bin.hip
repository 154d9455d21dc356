// Hit binning (the hit-selection structure of section 3.1): a counting sort
// of the hits of several events into (event, layer, z bin, phi bin), hits in
// a bin ordered by (phi, original index).  Deterministic: slots inside a bin
// are assigned by rank, never by atomic arrival order.
//
// Two paths with the same result, after a pass that gives every hit its bin
// and angle.  The grouped path sorts each (event, layer) range of input that
// holds each event's hits grouped by layer, all valid, in one or several
// blocks inside LDS; the general path takes any order and bad hits: count ->
// scan of the bin counts -> place (arbitrary order inside each bin, whole hit
// records) and offsets -> rank (exact order inside each bin) and write out.
// A device word selects the path, so the sequence has no host decision in it
// and can be captured in a graph.
#include <stdlib.h>
#include <string.h>

#include <algorithm>

#include "kfhost.h"
#include "kfranges.h"

using namespace kfranges;

namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr int kScanBlock = 1024;  // threads; each handles 2 elements
constexpr int kWideGrid = 2048;   // blocks of the grid-stride kernels: eight per CU
// Blocks of the rank kernel: twice as many, and no power of two, of which a
// wave's stride comes back to the same z rows, of the inner layers the fullest
// (200 000 shuffled tracks in 64 x 64 bins, 2 048 blocks 1 547 us, 4 093 1 330, 8 191
// 1 250; 50 000 in 63 x 16 bins 459, 419, 416; where the grouped path has sorted,
// each 2 048 blocks more take 0.3 us).
constexpr int kRankGrid = 4093;

// What the general path counts into, where the grouped path is not tried.
__global__ void clear_kernel(int32_t* __restrict__ count, int64_t n, int32_t* __restrict__ ctl,
                             int32_t* __restrict__ bad) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl[0] = ctl[1] = 1;
    ctl[2] = 0;
    if (bad) *bad = 0;
  }
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    count[i] = 0;
}

// The row coordinate of each layer: w = z on a barrel layer, w = r =
// sqrt(x^2 + y^2) on an endcap disk, binned over [lo, hi] in n_z rows.
struct RowGeom {
  int32_t disk[32];
  double lo[32], hi[32], inv[32];  // inv: 1 / (hi - lo)
};

// floor(a / d) for inv = 1 / d: the product is within 1e-15 of the quotient
// (relative), so where it is 1e-9 of its size from the next integer the
// quotient has the same floor; the division decides elsewhere.
__device__ inline double floor_div(double a, double d, double inv) {
  const double q = a * inv, f = floor(q), m = 1e-9 * (1.0 + fabs(q));
  if (q - f > m && f + 1.0 - q > m) return f;
  return floor(a / d);
}

// Bin of a hit inside its (event, layer) and its stored phi.  phi and the
// bin indices are computed in FP64 with the expression order of the
// definition, so the bin of a hit never depends on contraction or
// reassociation.
__device__ inline int bin_in_layer(double x, double y, double z, int l, const RowGeom& rg, int n_phi, int n_z,
                                   float* phf_out, int* ip_out) {
#pragma clang fp contract(off)
  double ph = atan2(y, x);
  if (ph < 0.0) ph += kTwoPi;
  const float phf = (float)ph;
  int ip = (int)floor_div((double)phf * (double)n_phi, kTwoPi, 1.0 / kTwoPi);
  ip = ip > n_phi - 1 ? n_phi - 1 : (ip < 0 ? 0 : ip);
  const double w = rg.disk[l] ? sqrt(x * x + y * y) : z;
  const double lo = rg.lo[l], hi = rg.hi[l];
  const double fz = floor_div((w - lo) * (double)n_z, hi - lo, rg.inv[l]);
  const int iz = fz < 0.0 ? 0 : (fz > (double)(n_z - 1) ? n_z - 1 : (int)fz);
  *phf_out = phf;
  *ip_out = ip;
  return iz * n_phi + ip;
}

__device__ inline bool finite3(float x, float y, float z) {
  return __builtin_isfinite(x) && __builtin_isfinite(y) && __builtin_isfinite(z);
}

// ---- Bins and angles ---------------------------------------------------------
//
// Every hit's bin ((event * L + layer) * nb + bin) * F + the piece of the bin
// its angle lies in, -1 for a hit on a layer outside [0, L) or with a
// non-finite coordinate, and its angle.  Where the grouped path is tried, the
// first hit of every (event, layer) range and, per block, whether its hits kept
// the order that path needs; otherwise the general path's counts and the
// arrival index among the bin's hits (the value the count's atomic returns; the
// rank pass fixes the order).  Blocks whose first hits are plainly not in order
// leave theirs to count_kernel, which bins and counts them in one pass, the
// atomics behind the arithmetic (8 events of 50 000 tracks in any order: 1.93 ms
// for the call with a pass for the counts alone, 1.70 without the attempt).
// The pass also clears what the kernels after it raise.  FP64 arithmetic bounds
// it (an arctangent and two quotients a hit): 8.16 M hits in 109 us, 24 B a hit.
constexpr int kBinGrid = 2048;

struct BinArgs {
  int n, E, L, n_phi, n_z;
  const int32_t* eoff;
  const int32_t* layer;
  const float* xyz;
  int32_t* gbin_of;  // bin * F + piece
  float* phi_of;
  int32_t* arrival;
  int32_t* count;
  int64_t NB;
  int32_t F;
  int32_t* seg;      // [E L + 1] first hit of every range
  // [kBinGrid] bit 0: the block's hits are not grouped or not all valid, or its
  // events do not tile the hits; bit 1: its hits are left to count_kernel
  uint8_t* blk_bad;
  int32_t* ctl;      // see BinWs
  int32_t* bad;      // may be null
  int32_t flag0, try_grouped;
};

// The hits [i0, i1) of this block: consecutive, so most need no search for
// their event, and a multiple of its threads.
__device__ inline void run_of_block(int n, int& i0, int& i1) {
  const int per = (int)((((int64_t)n + gridDim.x - 1) / gridDim.x + 255) & ~(int64_t)255);
  const int64_t at = (int64_t)blockIdx.x * per;
  i0 = at < n ? (int)at : n;
  i1 = at + per < n ? (int)(at + per) : n;
}

// Bins the block's hits, and counts them (COUNT) or writes the range starts.
// Returns the block's bits of blk_bad (of this thread's hits for bit 0).
template <bool COUNT>
__device__ inline int bin_run(const BinArgs& A, const RowGeom& rg, int i0, int i1) {
  const int n = A.n, E = A.E, L = A.L, nb = A.n_phi * A.n_z, t = threadIdx.x;
  const int32_t* eoff = A.eoff;
  int elo = 0, ehi = 1;
  if (eoff && i0 < i1) {
    elo = event_of(eoff, 0, E, i0);
    ehi = event_of(eoff, elo, E, i1 - 1) + 1;
  }
  const double turns = A.n_phi / kTwoPi;
  bool ok = true;
  int ln = 0, lpn = -1;
  float xn = 0.f, yn = 0.f, zn = 0.f;
  auto load = [&](int k) {
    if (k >= i1 - i0) return;
    const int i = i0 + k;
    ln = A.layer[i];
    if (!COUNT) lpn = i > 0 ? A.layer[i - 1] : -1;
    xn = A.xyz[i];
    yn = A.xyz[(size_t)n + i];
    zn = A.xyz[2 * (size_t)n + i];
  };
  load(t);
  // (a descent of the layer starts an event in ordered input; the check runs
  // behind the loads of the coordinates)
  if (!COUNT && __syncthreads_count(t < i1 - i0 && ln < lpn) > 64) return 3;
  for (int k = t; k < i1 - i0; k += 256) {
    const int i = i0 + k;
    const int l = ln, lp = lpn;
    const float xf = xn, yf = yn, zf = zn;
    load(k + 256);  // on its way during the arithmetic
    const int e = eoff ? event_of(eoff, elo, ehi, i) : 0;
    if (l < 0 || l >= L || !finite3(xf, yf, zf)) {
      A.gbin_of[i] = -1;
      if (COUNT && A.bad) atomicAdd(A.bad, 1);
      ok = false;
      continue;
    }
    float phf;
    int ip;
    const int gb = (e * L + l) * nb +
                   bin_in_layer((double)xf, (double)yf, (double)zf, l, rg, A.n_phi, A.n_z, &phf, &ip);
    // which of F pieces of the bin's angles: any function that never falls
    // with the angle will do
    const int pc = (int)(((double)phf * turns - (double)ip) * A.F);
    A.gbin_of[i] = gb * A.F + (pc < 0 ? 0 : (pc < A.F ? pc : A.F - 1));
    A.phi_of[i] = phf;
    if (COUNT) A.arrival[i] = atomicAdd(&A.count[gb], 1);
    else ok = range_starts(eoff, E, L, n, i, e, l, lp, A.seg) && ok;
  }
  return ok ? 0 : 1;
}

__global__ void __launch_bounds__(256) bin_kernel(BinArgs A, RowGeom rg) {
  const int n = A.n, E = A.E, EL = E * A.L, t = threadIdx.x;
  int i0, i1;
  run_of_block(n, i0, i1);
  if (!A.try_grouped) {
    (void)bin_run<true>(A, rg, i0, i1);
    return;
  }
  if (blockIdx.x == 0 && t == 0) {
    A.ctl[0] = A.flag0;
    A.ctl[1] = 0;
    A.ctl[2] = 0;
    if (A.bad) *A.bad = 0;
  }
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + t; k < A.NB; k += (int64_t)gridDim.x * blockDim.x) A.count[k] = 0;
  if (n == 0)
    for (int k = blockIdx.x * blockDim.x + t; k <= EL; k += gridDim.x * blockDim.x) A.seg[k] = 0;
  bool ok = true;
  if (A.eoff)
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + t; e < E; e += (int64_t)gridDim.x * blockDim.x)
      ok = ok && tiles(A.eoff, E, n, (int)e);
  const int bits = bin_run<false>(A, rg, i0, i1);
  const int any_bad = __syncthreads_or(!ok || (bits & 1));
  if (t == 0) A.blk_bad[blockIdx.x] = (any_bad ? 1 : 0) | (bits & 2);
}

// ---- Grouped path -----------------------------------------------------------
//
// When every event's hits come grouped by layer in ascending order, all on
// valid layers with finite coordinates (as detector readout and the
// generator deliver them), the hits of an (event, layer) are one contiguous
// input range and their sorted positions are that same range.  Blocks then
// sort the range in parts of at most `part` consecutive sorted positions (and
// the rest of a piece), each on its own:
//   1. an LDS histogram of the range's bins, each cut in F pieces of its
//      angles, and its scan: the starts, hence the part's pieces;
//   2. angle and input index of the part's hits into LDS, piece by piece
//      (arbitrary order inside a piece);
//   3. every hit counts the hits of its piece with a smaller (phi, input
//      index) key: its sorted position, to which the pair then moves;
//   4. one component after the other: the range read in input order into
//      LDS, picked from there in the sorted order, written out in one piece.
// So every byte is read and written coalesced.  The ranks are the largest
// phase, bounded by LDS reads, which is why a bin is cut in pieces of its
// angles and the angles alone are compared (5 hits a bin: 74 k cycles a block
// with (angle, index) pairs of whole bins, 17 k so; the components 46 k).
// 1 700 ranges of about 5 000 hits: 199 us here and 311 for the call, against
// 616 with one block per range that scattered whole records to their bins in
// memory and read them back (214 B a hit); 408 ranges of 20 000 in three
// parts each: 400 us for the call, against 876 by the general path then.  A
// longer prefetch (18 loads a thread) changed nothing.
constexpr int kSegPer = 8;                       // positions of a part per thread, at most
constexpr int kSegTile = 2048;                   // hits of a bin at most
constexpr int kSegPart = 6784;                   // leaves room for the rest of a piece
// One event of 20 000 tracks, the whole build call: 476 us with parts of 1 024,
// 481 with 2 048, 491 with 512 (each part reads the range's bins).
constexpr int kSegMinPart = 1024;
// Ranges of up to this many hits in the mean are sorted by blocks of 256
// threads, five to seven on a CU: 1 024 threads spend 25 us on a range of any
// size (17 408 ranges of 150 hits: 862 us, 286 with 256 threads; 1 088 ranges
// of 1 500: 100 and 79, of 3 000: 134 and 203).
constexpr int kSegSmall = 2000;
constexpr int kSegSmallPart = 1664;
constexpr int kSegMinCall = 64000;                // hits and a quarter of the bins of a call that tries the path
constexpr int kSegMaxBins = 4096;                // n_phi * n_z the grouped path takes: 12 bits
constexpr int kSegIdxBits = 20;                  // an index inside the range beside the bin
// Parts of a range up to which each stages the whole range; with more, a part
// reads its own hits alone.  Build call of 20 events (three parts a range): 5.35 ms
// staged, 5.74 not; of one event (20 parts): 476 us not staged, 500 staged.
constexpr int kSegStage = 4;
constexpr int kSegPieces = 3072;                 // pieces of all bins that leave two blocks their LDS

size_t seg_lds_bytes(int threads, int np) { return (size_t)(kSegPer * threads) * 8 + (size_t)(np + 1) * 4; }

struct SegArgs {
  int n, E, L, nb, F, part, n_blk;
  const int32_t* eoff;
  const int32_t* seg;
  const uint8_t* blk_bad;
  const int32_t* gbin_of;
  const float* phi_of;
  const float* xyz;
  const float* cov;
  int32_t* ctl;
  int32_t* offsets;
  float* sorted_xyzphi;
  float* sorted_cov;
  int32_t* sorted_orig;
};

// The 64-ary search for the last s in [0, EL) with seg[s] / part + s <= b.
__device__ inline int range_of_block(const int32_t* __restrict__ seg, int EL, int part, int b, int lane) {
  int lo = 0, hi = EL;  // answer in [lo, hi)
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) / 64, p = lo + lane * step;
    const bool le = p < hi && seg[p] / part + p <= b;
    const int c = __builtin_popcountll(__ballot(le));  // (monotone: the first c lanes)
    lo += (c > 0 ? c - 1 : 0) * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  return lo;
}

// Block b takes part b - (a / part + s) of the range s with the largest
// a / part + s at or below b (a: the range's first hit): the ranges tile the
// input, so every range owns at least as many blocks as it has parts, and
// n / part + E L blocks hold them all.
template <int T>
__global__ void __launch_bounds__(T, 8) seg_kernel(SegArgs A) {
  constexpr int kSegThreads = T, kSegCap = kSegPer * T;
  extern __shared__ __align__(16) int32_t sm[];
  float* key = (float*)sm;                 // [kSegCap] angle, then the staged component
  uint32_t* idx = (uint32_t*)sm + kSegCap; // [kSegCap] (piece, input index in the range), then the index alone
  int32_t* start = sm + 2 * kSegCap;       // [np + 1] counts and starts of the pieces; ends once placed
  __shared__ int32_t s_sum[kSegThreads / 64];
  __shared__ int s_sg;
  const int t = threadIdx.x, lane = t & 63, np = A.nb * A.F, EL = A.E * A.L;
  const size_t N = (size_t)A.n;
  // consecutive parts on one XCD, whose L2 then holds their range
  const int per_xcd = (int)gridDim.x / 8;
  const int b = (int)blockIdx.x < per_xcd * 8 ? (int)(blockIdx.x % 8) * per_xcd + (int)blockIdx.x / 8 : (int)blockIdx.x;
  bool bad = false;
  for (int k = t; k < (A.n_blk + 3) / 4; k += kSegThreads) {
    const int left = A.n_blk - 4 * k;
    const uint32_t w = ((const uint32_t*)A.blk_bad)[k];
    bad = bad || ((left >= 4 ? w : w & ((1u << (8 * left)) - 1)) & 0x01010101u) != 0;
  }
  if (t >= kSegThreads - 64) {
    const int r = range_of_block(A.seg, EL, A.part, b, lane);
    if (lane == 0) s_sg = r;
  }
  for (int k = t; k <= np; k += kSegThreads) start[k] = 0;
  // (without a bad block every entry of seg is written, ascending in [0, n])
  if (__syncthreads_or(bad)) {
    if (t == 0) A.ctl[0] = A.ctl[1] = 1;
    return;
  }
  const int sg = s_sg;
  const int a = A.seg[sg], len = A.seg[sg + 1] - a, k = b - (a / A.part + sg);
  const int parts = len > A.part ? (len + A.part - 1) / A.part : 1;
  if (k >= parts) return;
  if (len == 0) {
    int32_t* off = A.offsets + (size_t)sg * (A.nb + 1);
    for (int q = t; q <= A.nb; q += kSegThreads) off[q] = a;
    return;
  }
  if (len >= 1 << kSegIdxBits) {
    if (t == 0) A.ctl[0] = A.ctl[1] = 1;
    return;
  }
  const int32_t* gb = A.gbin_of + a;
  const int g0 = sg * np;
  constexpr int U = 5;
  for (int j0 = t; j0 < len; j0 += kSegThreads * U) {
    int g[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * kSegThreads < len) g[u] = gb[j0 + u * kSegThreads];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * kSegThreads < len) atomicAdd(&start[g[u] - g0], 1);
  }
  __syncthreads();
  // exclusive scan of the counts: a run of consecutive pieces per thread
  const int per = (np + kSegThreads - 1) / kSegThreads;
  const int c0 = t * per < np ? t * per : np, c1 = c0 + per < np ? c0 + per : np;
  int sum = 0;
  for (int q = c0; q < c1; ++q) sum += start[q];
  int inc = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(inc, d, 64);
    if (lane >= d) inc += v;
  }
  if (lane == 63) s_sum[t >> 6] = inc;
  __syncthreads();
  int run = inc - sum;
  for (int w = 0; w < (t >> 6); ++w) run += s_sum[w];
  for (int q = c0; q < c1; ++q) {
    const int c = start[q];
    start[q] = run;
    run += c;
  }
  if (t == 0) start[np] = len;
  __syncthreads();
  bad = false;
  for (int q = t; q < A.nb; q += kSegThreads) bad = bad || start[(q + 1) * A.F] - start[q * A.F] > kSegTile;
  if (__syncthreads_or(bad)) {
    if (t == 0) A.ctl[0] = A.ctl[1] = 1;
    return;
  }
  if (k == 0) {
    int32_t* off = A.offsets + (size_t)sg * (A.nb + 1);
    for (int q = t; q <= A.nb; q += kSegThreads) off[q] = a + start[q * A.F];
  }
  // this part: the pieces that start in [k len / parts, (k + 1) len / parts)
  auto first_piece = [&](int pos) {  // first piece with a start of pos or more
    int lo = 0, hi = np;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (start[mid] < pos) lo = mid + 1; else hi = mid;
    }
    return lo;
  };
  const int b0 = k == 0 ? 0 : first_piece((int)((int64_t)len * k / parts));
  const int b1 = k == parts - 1 ? np : first_piece((int)((int64_t)len * (k + 1) / parts));
  const int s0 = start[b0], m = b1 > b0 ? start[b1] - s0 : 0;
  __syncthreads();  // (the starts move below)
  if (m <= 0) return;
  if (m > kSegCap) {
    if (t == 0) A.ctl[0] = A.ctl[1] = 1;
    return;
  }
  for (int j0 = t; j0 < len; j0 += kSegThreads * U) {
    int g[U];
    float ph[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * kSegThreads < len) {
        g[u] = gb[j0 + u * kSegThreads] - g0;
        ph[u] = A.phi_of[a + j0 + u * kSegThreads];
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * kSegThreads < len && g[u] >= b0 && g[u] < b1) {
        const int s = atomicAdd(&start[g[u]], 1) - s0;
        key[s] = ph[u];
        idx[s] = (uint32_t)g[u] << kSegIdxBits | (uint32_t)(j0 + u * kSegThreads);
      }
  }
  __syncthreads();
  float kp[kSegPer];
  uint32_t ki[kSegPer];
  int at[kSegPer];
#pragma unroll
  for (int j = 0; j < kSegPer; ++j) {
    const int s = t + j * kSegThreads;
    at[j] = -1;
    if (s < m) {
      kp[j] = key[s];
      ki[j] = idx[s];
      const int pc = (int)(ki[j] >> kSegIdxBits);
      const int q0 = pc == b0 ? 0 : start[pc - 1] - s0, q1 = start[pc] - s0;
      // the angles alone; the indices only where two are equal
      int lt = 0, le = 0, q = q0;
      for (; q + 4 <= q1; q += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float pq = key[q + u];
          lt += pq < kp[j];
          le += pq <= kp[j];
        }
      }
      for (; q < q1; ++q) {
        const float pq = key[q];
        lt += pq < kp[j];
        le += pq <= kp[j];
      }
      if (le > lt + 1)
        for (q = q0; q < q1; ++q) lt += key[q] == kp[j] && idx[q] < ki[j];
      at[j] = q0 + lt;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSegPer; ++j)
    if (at[j] >= 0) {
      key[at[j]] = kp[j];
      idx[at[j]] = ki[j] & ((1u << kSegIdxBits) - 1);
    }
  __syncthreads();
  const size_t dst = (size_t)a + s0;
  const int first = A.eoff ? a - A.eoff[sg / A.L] : a;
  for (int q = t; q < m; q += kSegThreads) {
    A.sorted_xyzphi[3 * N + dst + q] = key[q];
    A.sorted_orig[dst + q] = first + (int)idx[q];
  }
  auto src_of = [&](int c) { return (c < 3 ? A.xyz + c * N : A.cov + (c - 3) * N) + a; };
  auto out_of = [&](int c) { return (c < 3 ? A.sorted_xyzphi + c * N : A.sorted_cov + (c - 3) * N) + dst; };
  if (parts > kSegStage) {
    // little of the range is this part's: its hits alone, from L2
    for (int q = t; q < m; q += kSegThreads) {
      const int i = (int)idx[q];
      float v[9];
#pragma unroll
      for (int c = 0; c < 9; ++c) v[c] = src_of(c)[i];
#pragma unroll
      for (int c = 0; c < 9; ++c) out_of(c)[q] = v[c];
    }
    return;
  }
  // chunks of kSegCap hits of a component, the next one on its way while
  // the present one is picked from
  const int chunks = (len + kSegCap - 1) / kSegCap;
  float in[kSegPer], val[kSegPer];
  auto load = [&](int c, int ch) {
    const float* p = src_of(c);
#pragma unroll
    for (int j = 0; j < kSegPer; ++j) {
      const int i = ch * kSegCap + t + j * kSegThreads;
      if (i < len) in[j] = p[i];
    }
  };
  load(0, 0);
  for (int c = 0; c < 9; ++c) {
    for (int ch = 0; ch < chunks; ++ch) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kSegPer; ++j) key[t + j * kSegThreads] = in[j];
      __syncthreads();
      if (ch + 1 < chunks) load(c, ch + 1);
      else if (c < 8) load(c + 1, 0);
#pragma unroll
      for (int j = 0; j < kSegPer; ++j) {
        const int q = t + j * kSegThreads;
        if (q < m) {
          const int i = (int)idx[q] - ch * kSegCap;
          if (i >= 0 && i < kSegCap) val[j] = key[i];
        }
      }
    }
    float* out = out_of(c);
#pragma unroll
    for (int j = 0; j < kSegPer; ++j)
      if (t + j * kSegThreads < m) out[t + j * kSegThreads] = val[j];
  }
}

// ---- General path: any order, bad hits --------------------------------------
// Every kernel of this path returns at once when the grouped path sorted the
// call (*go == 0).

// The count of every bin and every hit's arrival index after an attempt of the
// grouped path, by the blocks of bin_kernel; hits it left are binned too.
__global__ void __launch_bounds__(256) count_kernel(BinArgs A, RowGeom rg) {
  if (A.ctl[1] == 0) return;
  int i0, i1;
  run_of_block(A.n, i0, i1);
  if (A.blk_bad[blockIdx.x] & 2) {
    (void)bin_run<true>(A, rg, i0, i1);
    return;
  }
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    const int gb = A.gbin_of[i];
    if (gb >= 0) A.arrival[i] = atomicAdd(&A.count[gb / A.F], 1);
    else if (A.bad) atomicAdd(A.bad, 1);
  }
}

// Exclusive scan of 2 kScanBlock counts per block (in LDS); the last block to
// end scans the blocks' sums.  The start of bin g is
// out[g] + bsum[g / (2 kScanBlock)].
__global__ void __launch_bounds__(kScanBlock) scan_kernel(const int32_t* __restrict__ in, int32_t* __restrict__ out,
                                                          int32_t* __restrict__ bsum, int n,
                                                          const int32_t* __restrict__ go,
                                                          int32_t* __restrict__ ticket) {
  if (*go == 0) return;
  __shared__ int32_t s[kScanBlock / 64];
  __shared__ int s_last;
  const int t = threadIdx.x, lane = t & 63;
  // inclusive sum over the block's threads
  auto block_scan = [&](int v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(v, d, 64);
      if (lane >= d) v += o;
    }
    __syncthreads();
    if (lane == 63) s[t >> 6] = v;
    __syncthreads();
    for (int w = 0; w < (t >> 6); ++w) v += s[w];
    return v;
  };
  const int64_t i = (int64_t)blockIdx.x * 2 * kScanBlock + 2 * t;
  const int v0 = i < n ? in[i] : 0, v1 = i + 1 < n ? in[i + 1] : 0;
  const int inc = block_scan(v0 + v1);
  if (i < n) out[i] = inc - v1 - v0;
  if (i + 1 < n) out[i + 1] = inc - v1;
  if (t == kScanBlock - 1) {
    __hip_atomic_store(&bsum[blockIdx.x], inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // (the sum has reached memory before the ticket is taken; a release would
    // write back the whole L2 for it: 41 us against 9 with 837 blocks)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    s_last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  }
  __syncthreads();
  if (!s_last) return;
  int carry = 0;
  for (int c = 0; c < (int)gridDim.x; c += kScanBlock) {
    const int k = c + t;
    const int v = k < (int)gridDim.x ? __hip_atomic_load(&bsum[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const int w = block_scan(v);
    if (k < (int)gridDim.x) bsum[k] = carry + w - v;
    __syncthreads();
    int all = 0;
    for (int q = 0; q < kScanBlock / 64; ++q) all += s[q];
    carry += all;
  }
}

__device__ inline int bin_start(const int32_t* __restrict__ start, const int32_t* __restrict__ bsum, int64_t g) {
  return start[g] + bsum[g / (2 * kScanBlock)];
}

// Each hit takes the slot of its bin given by its arrival index and writes
// its whole record there: (x, y, z, phi), (cov 0..3), (cov 4, cov 5, input
// index, 0).  And offsets[el][b] = start of bin b of (event, layer) el; entry
// nb closes it.
__global__ void __launch_bounds__(256) place_kernel(int n, int F, const int32_t* __restrict__ gbin_of,
                                                    const float* __restrict__ phi_of,
                                                    const int32_t* __restrict__ arrival, const float* __restrict__ xyz,
                                                    const float* __restrict__ cov, const int32_t* __restrict__ start,
                                                    const int32_t* __restrict__ bsum,
                                                    const int32_t* __restrict__ count, int EL, int nb,
                                                    float4* __restrict__ rec, int32_t* __restrict__ offsets,
                                                    const int32_t* __restrict__ go) {
  if (*go == 0) return;
  const size_t N = (size_t)n;
  const int64_t first = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = first; i < n; i += stride) {
    const int gb = gbin_of[i];
    if (gb < 0) continue;
    const float4 r0 = make_float4(xyz[i], xyz[N + i], xyz[2 * N + i], phi_of[i]);
    const float4 r1 = make_float4(cov[i], cov[N + i], cov[2 * N + i], cov[3 * N + i]);
    const float4 r2 = make_float4(cov[4 * N + i], cov[5 * N + i], __int_as_float((int)i), 0.f);
    const int slot = bin_start(start, bsum, gb / F) + arrival[i];
    float4* r = rec + (size_t)slot * 3;
    r[0] = r0;
    r[1] = r1;
    r[2] = r2;
  }
  for (int64_t k = first; k < (int64_t)EL * (nb + 1); k += stride) {
    const int el = (int)(k / (nb + 1)), b = (int)(k % (nb + 1));
    const int64_t g = (int64_t)el * nb;
    offsets[k] = b < nb ? bin_start(start, bsum, g + b) : bin_start(start, bsum, g + nb - 1) + count[g + nb - 1];
  }
}

// Exact order inside a bin: rank = number of hits of the bin with a smaller
// (phi, original index) key.  W lanes (lane: this one's index among them) each
// hold one hit record of the bin and compare it with every hit of the bin,
// whose keys they pass around W at a time (larger bins loop over blocks of
// W).  The hit is then written to its slot in the sorted arrays.
template <int W>
__device__ inline void rank_bin(int lane, int b0, int cnt, int ev_base, size_t N, const float4* __restrict__ rec,
                                float* __restrict__ sorted_xyzphi, float* __restrict__ sorted_cov,
                                int32_t* __restrict__ sorted_orig) {
  for (int c0 = 0; c0 < cnt; c0 += W) {
    const bool mine = c0 + lane < cnt;
    const float4* r = rec + (size_t)(b0 + c0 + (mine ? lane : 0)) * 3;
    const float4 r0 = r[0], r1 = r[1], r2 = r[2];
    const int i = __float_as_int(r2.z);
    const float ph = r0.w;
    int rank = 0;
    // the keys of the next W hits are on their way during the comparisons
    float np = 0.f;
    int ni = 0;
    auto load = [&](int d0) {
      const float4* o = rec + (size_t)(b0 + (d0 + lane < cnt ? d0 + lane : 0)) * 3;
      ni = __float_as_int(o[2].z);
      np = o[0].w;
    };
    if (cnt > W) load(0);
    for (int d0 = 0; d0 < cnt; d0 += W) {
      const int oi = cnt > W ? ni : i;
      const float op = cnt > W ? np : ph;
      if (d0 + W < cnt) load(d0 + W);
      const int m = cnt - d0 < W ? cnt - d0 : W;
      int t = 0;
      for (; t + 2 <= m; t += 2) {  // (two steps' shuffles in flight)
        const float pj = __shfl(op, t, W), pk = __shfl(op, t + 1, W);
        const int j = __shfl(oi, t, W), k = __shfl(oi, t + 1, W);
        rank += (pj < ph || (pj == ph && j < i)) ? 1 : 0;
        rank += (pk < ph || (pk == ph && k < i)) ? 1 : 0;
      }
      for (; t < m; ++t) {
        const float pj = __shfl(op, t, W);
        const int j = __shfl(oi, t, W);
        rank += (pj < ph || (pj == ph && j < i)) ? 1 : 0;
      }
    }
    if (mine) {
      const int dst = b0 + rank;
      sorted_xyzphi[dst] = r0.x;
      sorted_xyzphi[N + dst] = r0.y;
      sorted_xyzphi[2 * N + dst] = r0.z;
      sorted_xyzphi[3 * N + dst] = ph;
      sorted_cov[dst] = r1.x;
      sorted_cov[N + dst] = r1.y;
      sorted_cov[2 * N + dst] = r1.z;
      sorted_cov[3 * N + dst] = r1.w;
      sorted_cov[4 * N + dst] = r2.x;
      sorted_cov[5 * N + dst] = r2.y;
      sorted_orig[dst] = i - ev_base;
    }
  }
}

// G lanes per bin, 64 / G bins at once; where one of these bins is so much
// the largest that the others' lanes would mostly wait for it, all 64 lanes
// take the bins one after another (85 000 shuffled hits, a bin of 1 000 a layer:
// 5 239 us with G lanes alone, 1 003 so; 20 bins of 100 a layer: 122 and 72).  A
// call of 6.5 M hits, 6 a bin: 872 us with 64 lanes a bin, 719 with 16; 24 a bin:
// 819 us with 32 lanes, 747 with 64.
template <int G>
__global__ void __launch_bounds__(256) rank_kernel(int NB, int n, int L, int nb_el,
                                                   const int32_t* __restrict__ eoff,
                                                   const float4* __restrict__ rec,
                                                   const int32_t* __restrict__ start,
                                                   const int32_t* __restrict__ bsum,
                                                   const int32_t* __restrict__ count,
                                                   float* __restrict__ sorted_xyzphi,
                                                   float* __restrict__ sorted_cov, int32_t* __restrict__ sorted_orig,
                                                   const int32_t* __restrict__ go) {
  if (*go == 0) return;
  const int lane = threadIdx.x & 63, sub = lane / G;
  const int64_t waves = gridDim.x * (int64_t)(blockDim.x / 64);
  for (int64_t g0 = (blockIdx.x * (int64_t)(blockDim.x / 64) + threadIdx.x / 64) * (64 / G); g0 < NB;
       g0 += waves * (64 / G)) {
    const int64_t gb = g0 + sub;
    const int cnt = gb < NB ? count[gb] : 0;
    if (!__any(cnt > 0)) continue;
    const int b0 = cnt > 0 ? bin_start(start, bsum, gb) : 0;
    // the event of the bin: bins are numbered (event * L + layer) * nb_el + bin
    const int ev_base = cnt > 0 && eoff ? eoff[gb / (L * nb_el)] : 0;
    // the steps of a wave: the largest bin's with G lanes a bin, the sum with 64
    float together = (float)((cnt + G - 1) / G) * (float)cnt, alone = (float)((cnt + 63) / 64) * (float)cnt;
#pragma unroll
    for (int d = G; d < 64; d <<= 1) {
      together = fmaxf(together, __shfl_xor(together, d, 64));
      alone += __shfl_xor(alone, d, 64);
    }
    if (G == 64 || together <= alone) {
      rank_bin<G>(lane % G, b0, cnt, ev_base, (size_t)n, rec, sorted_xyzphi, sorted_cov, sorted_orig);
    } else {
#pragma unroll 1
      for (int j = 0; j < 64; j += G)
        rank_bin<64>(lane, __builtin_amdgcn_readlane(b0, j), __builtin_amdgcn_readlane(cnt, j),
                     __builtin_amdgcn_readlane(ev_base, j), (size_t)n, rec, sorted_xyzphi, sorted_cov, sorted_orig);
    }
  }
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

struct BinWs {
  int32_t *gbin_of, *arrival, *count, *start, *bsum, *seg;
  uint8_t* blk_bad;
  // [0] the reported word, [1] the path: 1 where the general path runs, [2] the
  // scan's ticket
  int32_t* ctl;
  float* phi_of;
  float4* rec;  // [n][3] hit records in bin slots
};

size_t bin_ws_layout(int E, int L, int n_phi, int n_z, int n, char* base, BinWs* w) {
  const size_t NB = (size_t)E * L * n_phi * n_z;
  const size_t nblk = (NB + 2 * kScanBlock - 1) / (2 * kScanBlock);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += align256(bytes);
    return p;
  };
  char* a = take(sizeof(int32_t) * (size_t)n);
  char* b = take(sizeof(float4) * 3 * (size_t)n);
  char* c = take(sizeof(float) * (size_t)n);
  char* d = take(sizeof(int32_t) * NB);
  char* e = take(sizeof(int32_t) * (size_t)n);
  char* f = take(sizeof(int32_t) * NB);
  char* g = take(sizeof(int32_t) * (nblk + 1));
  char* k = take(sizeof(int32_t) * ((size_t)E * L + 1));
  char* m = take(kBinGrid);
  char* h = take(sizeof(int32_t) * 3);
  if (w) {
    w->ctl = (int32_t*)h;
    w->seg = (int32_t*)k;
    w->blk_bad = (uint8_t*)m;
    w->gbin_of = (int32_t*)a;
    w->rec = (float4*)b;
    w->phi_of = (float*)c;
    w->arrival = (int32_t*)e;
    w->count = (int32_t*)d;
    w->start = (int32_t*)f;
    w->bsum = (int32_t*)g;
  }
  return off;
}

int grid_for(int64_t n, int bs) { return (int)((n + bs - 1) / bs); }

int device_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  return cus;
}

}  // namespace

extern "C" size_t hit_bin_workspace_bytes(int32_t n_events, int32_t n_layers, int32_t n_phi, int32_t n_z,
                                          int32_t n_hits) {
  if (n_events < 1 || n_layers < 1 || n_phi < 1 || n_z < 1 || n_hits < 0) return 0;
  return bin_ws_layout(n_events, n_layers, n_phi, n_z, n_hits, nullptr, nullptr);
}

namespace {

int run_hit_bin(int L, const RowGeom& rg, int32_t n_events, const int32_t* event_offsets, int32_t n_phi,
                int32_t n_z, int32_t n_hits, const int32_t* layer, const float* xyz, const float* cov,
                int32_t* offsets, float* sorted_xyzphi, float* sorted_cov, int32_t* sorted_orig, int32_t* out_bad,
                void* ws, size_t ws_bytes, void* stream) {
  if (n_events < 1 || n_phi < 1 || n_z < 1 || n_hits < 0) return KF_E_INVALID_ARG;
  if (n_events > 1 && !event_offsets) return KF_E_INVALID_ARG;
  const int64_t NB = (int64_t)n_events * L * n_phi * n_z;
  if (NB >= (1ll << 31) - 1) return KF_E_UNSUPPORTED;
  if (!offsets) return KF_E_INVALID_ARG;
  if (n_hits > 0 && (!layer || !xyz || !cov || !sorted_xyzphi || !sorted_cov || !sorted_orig))
    return KF_E_INVALID_ARG;
  const size_t need = hit_bin_workspace_bytes(n_events, L, n_phi, n_z, n_hits);
  if (!ws || ws_bytes < need || ((uintptr_t)ws & 255)) return KF_E_WORKSPACE;
  BinWs w;
  bin_ws_layout(n_events, L, n_phi, n_z, n_hits, (char*)ws, &w);
  hipStream_t s = (hipStream_t)stream;
  const int bs = 256;
  const int nb = n_phi * n_z;
  const int EL = n_events * L;
  const char* path = getenv("KFTRACK_HIT_BIN_PATH");
  const int cus = device_cus();
  const int64_t mean = n_hits / EL;  // hits of a range
  const bool small = mean <= kSegSmall;
  const int threads = small ? 256 : 1024;
  // parts that give every CU about one and a half blocks, but not below
  // kSegMinPart (each part reads its range's bins: one event of 50 000 tracks 157
  // us with two blocks a CU, 128 with one and a half, 156 with one; 8 of 10 000 106,
  // 82 and 87); two where the ranges alone fill the chip (64 of 2 000: 111 and 118)
  // or the parts are near their largest (8 of 20 000: 186 and 192) or smallest
  // (4 of 5 000: 46 and 49)
  const int two = n_hits / (2 * cus), slots = EL >= 2 * cus || two >= 5000 || two < 900 ? 2 * cus : 3 * cus / 2;
  const int part = small ? kSegSmallPart : std::min(kSegPart, std::max(kSegMinPart, n_hits / slots));
  const int64_t seg_blocks = part_blocks(n_hits, part, EL, threads);
  // The grouped path is tried wherever its bins fit, but for the smallest
  // calls, which the general path's shorter kernels sort in 24 to 28 us against
  // 29 to 34 (one event of up to 2 000 tracks of 17 layers in 63 x 16 bins; 16
  // events of 100: 33 to 31; one of 5 000: 34 to 31, of 20 000: 108 to 60; 200 of
  // 500: 363 to 99; hits as events leave them, which fill few z rows of the
  // inner layers).  Large bins cost the general path most (one bin a layer,
  // 1 500 hits: 2 250 to 30).
  const bool forced = path && !strcmp(path, "grouped"), barred = path && !strcmp(path, "general");
  const bool tiny = (int64_t)n_hits + NB / 4 < kSegMinCall && n_hits < 16 * NB;
  // Ranges of few bins and few hits cost a block each more than the general path
  // its bins (765 000 ranges of 4 hits in 16 bins 7.5 ms to 1.2; 17 408 of 40 204 us
  // to 70, of 150 228 to 227, of 600 435 to 846; of 10 in 252 bins 198 to 150, of 40
  // 209 to 250).
  const bool thin = nb + 4 * mean < 640;
  const bool try_grouped = nb <= kSegMaxBins && seg_blocks > 0 && !barred && (forced || !(tiny || thin));
  // The reported word keeps the answers of a choice by ranges: 0 where the
  // grouped path sorts a call of six ranges and more per CU, or one it is
  // forced to try.  The word after it is the path.
  const int32_t flag0 = try_grouped && (forced || EL >= 6 * cus) ? 0 : 1;
  if (!try_grouped)
    hipLaunchKernelGGL(clear_kernel, dim3(std::min(grid_for(NB, bs), 4096)), dim3(bs), 0, s, w.count, NB, w.ctl,
                       out_bad);
  // pieces of a bin: a rank compares within a piece, two for every hit of the
  // mean bin (each piece costs a range its scan; all pieces of the call are
  // numbered in 32 bits)
  const int64_t pieces = std::min(std::min<int64_t>(kSegPieces / nb, ((1ll << 31) - 1) / NB), 2 * mean / nb + 1);
  const int F = try_grouped ? (int)std::max<int64_t>(1, pieces) : 1;
  const int blocks = std::max(1, std::min(grid_for(n_hits, bs), kBinGrid));
  BinArgs B{n_hits, n_events, L, n_phi, n_z, event_offsets, layer, xyz, w.gbin_of, w.phi_of, w.arrival, w.count, NB, F,
            w.seg, w.blk_bad, w.ctl, out_bad, flag0, try_grouped ? 1 : 0};
  hipLaunchKernelGGL(bin_kernel, dim3(blocks), dim3(bs), 0, s, B, rg);
  if (try_grouped) {
    SegArgs G{n_hits, n_events, L, nb, F, part, blocks, event_offsets, w.seg, w.blk_bad, w.gbin_of, w.phi_of, xyz, cov,
              w.ctl, offsets, sorted_xyzphi, sorted_cov, sorted_orig};
    hipLaunchKernelGGL(small ? seg_kernel<256> : seg_kernel<1024>, dim3((unsigned)seg_blocks), dim3(threads),
                       seg_lds_bytes(threads, nb * F), s, G);
    // general path from here (every kernel returns at once unless it is to run)
    if (n_hits > 0)
      hipLaunchKernelGGL(count_kernel, dim3(blocks), dim3(bs), 0, s, B, rg);
  }
  const int nblk = (int)((NB + 2 * kScanBlock - 1) / (2 * kScanBlock));
  hipLaunchKernelGGL(scan_kernel, dim3(nblk), dim3(kScanBlock), 0, s, w.count, w.start, w.bsum, (int)NB, w.ctl + 1,
                     w.ctl + 2);
  const int64_t items = std::max((int64_t)n_hits, (int64_t)EL * (nb + 1));
  hipLaunchKernelGGL(place_kernel, dim3((int)std::min<int64_t>((items + bs - 1) / bs, kWideGrid)), dim3(bs), 0, s,
                     n_hits, F, w.gbin_of, w.phi_of, w.arrival, xyz, cov, w.start, w.bsum, w.count, EL, nb, w.rec,
                     offsets, w.ctl + 1);
  if (n_hits > 0) {
    // lanes per bin by the mean bin, of which the fuller bins of the inner layers
    // hold several times as many, and a wave per bin where the waves suffice for
    // all (hits as events leave them, 16, 32 and 64 lanes, us: a mean of 2.4, 4
    // events 38, 39, 44; of 6, one event 38, 34, 33, 64 events 719, 737, 872; of 12,
    // 16 events 431, 374, 390; of 6 in 4 096 bins, 16 events 896, 915, 1 071, of
    // 15, 8 events 1 594, 1 274, 1 311)
    const int64_t in_bin = n_hits / NB;
    const int G = in_bin < 4 ? 16 : (in_bin < 16 && NB > 32768 ? 32 : 64);
    auto* rank = G == 16 ? rank_kernel<16> : (G == 32 ? rank_kernel<32> : rank_kernel<64>);
    hipLaunchKernelGGL(rank, dim3(std::min(grid_for(NB * G, bs), kRankGrid)), dim3(bs), 0, s, (int)NB, n_hits, L, nb,
                       event_offsets, w.rec, w.start, w.bsum, w.count, sorted_xyzphi, sorted_cov, sorted_orig,
                       w.ctl + 1);
  }
  return kf_check_launch();
}

}  // namespace

extern "C" int hit_bin(const kf_geometry* g, int32_t n_events, const int32_t* event_offsets, int32_t n_phi,
                       int32_t n_z, int32_t n_hits, const int32_t* layer, const float* xyz, const float* cov,
                       int32_t* offsets, float* sorted_xyzphi, float* sorted_cov, int32_t* sorted_orig,
                       int32_t* out_bad, void* ws, size_t ws_bytes, void* stream) {
  if (kf_check_geometry(g)) return KF_E_INVALID_ARG;
  // every layer binned in z over [-z_half, z_half]
  RowGeom rg = {};
  for (int l = 0; l < g->n_layers; ++l) {
    rg.disk[l] = 0;
    rg.lo[l] = -(double)g->z_half;
    rg.hi[l] = (double)g->z_half;
    rg.inv[l] = 1.0 / (rg.hi[l] - rg.lo[l]);
  }
  return run_hit_bin(g->n_layers, rg, n_events, event_offsets, n_phi, n_z, n_hits, layer, xyz, cov, offsets,
                     sorted_xyzphi, sorted_cov, sorted_orig, out_bad, ws, ws_bytes, stream);
}

extern "C" int hit_bin_det(const kf_detector* d, int32_t n_events, const int32_t* event_offsets, int32_t n_phi,
                           int32_t n_w, int32_t n_hits, const int32_t* layer, const float* xyz, const float* cov,
                           int32_t* offsets, float* sorted_xyzphi, float* sorted_cov, int32_t* sorted_orig,
                           int32_t* out_bad, void* ws, size_t ws_bytes, void* stream) {
  if (kf_check_detector(d)) return KF_E_INVALID_ARG;
  RowGeom rg = {};
  for (int l = 0; l < d->n_layers; ++l) {
    rg.disk[l] = d->kind[l] == KF_LAYER_DISK ? 1 : 0;
    rg.lo[l] = (double)d->lo[l];
    rg.hi[l] = (double)d->hi[l];
    rg.inv[l] = 1.0 / (rg.hi[l] - rg.lo[l]);
  }
  return run_hit_bin(d->n_layers, rg, n_events, event_offsets, n_phi, n_w, n_hits, layer, xyz, cov, offsets,
                     sorted_xyzphi, sorted_cov, sorted_orig, out_bad, ws, ws_bytes, stream);
}
