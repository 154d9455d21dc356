// Which event a hit belongs to and where the (event, layer) ranges of grouped
// input start (hit_bin.hip).  Host and device code (a CPU test runs it).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kfranges {

#define KFG __host__ __device__ inline

// The event e in [lo, hi) with eoff[e] <= i < eoff[e + 1] (for offsets that
// do not ascend: some e in [lo, hi)).
KFG int event_of(const int32_t* eoff, int lo, int hi, int i) {
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (eoff[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// Whether event e of E follows its predecessor: all of them do where the
// events tile [0, n) in order.
KFG bool tiles(const int32_t* eoff, int E, int n, int e) {
  return (e > 0 || eoff[0] == 0) && eoff[e] <= eoff[e + 1] && (e < E - 1 || eoff[E] == n);
}

// The ranges that start at hit i, on layer l of event e, its predecessor on
// layer lp (-1 for the first hit): seg[j] = i for every range j after the
// predecessor's up to its own, and n for those after the last hit's.  False
// where the hits are not in the order of their ranges.  If no hit returns
// false, every layer is in [0, L) and the events tile [0, n), all E L + 1
// entries of seg are written, ascending from 0 to n.
KFG bool range_starts(const int32_t* eoff, int E, int L, int n, int i, int e, int l, int lp, int32_t* seg) {
  const int f = e * L + l;
  int fp = -1;
  if (i > 0) {
    const int ep = eoff && i - 1 < eoff[e] ? event_of(eoff, 0, e + 1, i - 1) : e;
    fp = ep * L + lp;
  }
  if (lp < -1 || lp >= L || f < fp) return false;
  for (int j = fp + 1; j <= f; ++j) seg[j] = i;
  if (i == n - 1)
    for (int j = f + 1; j <= E * L; ++j) seg[j] = n;
  return true;
}

// Blocks of a grouped sort: every range owns at least as many as it has parts
// of `part` hits (the ranges tile the n hits).  -1 where the launch, of
// `threads` threads each, would reach the 2^32 threads a grid may have.
inline int64_t part_blocks(int n, int part, int64_t ranges, int threads) {
  const int64_t blocks = (int64_t)(n / part) + ranges;
  return blocks * threads < (int64_t)1 << 32 ? blocks : -1;
}

}  // namespace kfranges
