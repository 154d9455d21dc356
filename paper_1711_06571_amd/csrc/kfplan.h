// LDS plan of the build kernel (kf_build.hip): the per-wave regions of one
// block and their sizes.  Host code sizes the launch with it (two blocks of
// four waves per CU need at most 80 KB each), the kernel lays out its LDS
// with it.
#pragma once
#include <stddef.h>

#include "kfmlp.h"

// pairs per lane per round of the cooperative hit search (at most)
constexpr int NP = 2;

// LDS of one block (byte offsets), per wave:
//   stash    [27][64] f32      each slot's state before this layer's prediction
//                              (FP64: its first 21 - NPL values, the rest in
//                              the first half of xs)
//   record   [SEEDS][27] f32   best finished candidate of each seed
//   recfield [SEEDS][5] i32    valid, nhits, status, last layer, slot
//   starts   [64 NP] i8 run starts of the cooperative hit search
//   publish  [SEEDS] i32 entries of each seed's pool, [64] u8 whether one of a
//            candidate's hits was accepted
//   pool     [8 cap][SEEDS] of 8 B: a seed's accepted hits (chi2, position and
//            slot), ranked and cut to cap when an insertion finds it full, and
//            room for the holes of its candidates
//   mlp      activation buffer of the learned window (the network runs before
//            the hit search, so the pools of a learned build live in it)
//   xs       [6 + NPL][64] f64 FP64 builds: the rest of the state before the
//            prediction (FP32, first half), the last (6 + NPL) / 2 covariance
//            entries of the prediction during the hit search (second half)
// The state between layers stays in registers; what does not fit there is
// spilled (FP64: 280 B a lane, hybrid state 344, FP32 at most 68).  The children's
// keys take the stash or the first half of xs once the records are written.
// NPL: what fits two blocks of four waves per CU at cap 6 with the learned
// builds' network buffers (2) and in the hybrid state (20; 18 and 16 measured
// 0.7 and 1 % slower), 12 in the Cartesian state (14: 0.8 % slower).
__host__ __device__ constexpr int xs_npl(int tsize, bool learned, bool hyb) {
  return tsize == 8 ? (learned ? 2 : hyb ? 20 : 12) : -6;
}
struct LdsPlan {
  size_t stash, rec, recf, acc, pub, tl, tl_stride, mlp, xs, total;
};
__host__ __device__ inline size_t align16(size_t v) { return (v + 15) & ~(size_t)15; }
__host__ __device__ constexpr size_t pub_bytes(int cap) { return (size_t)(64 / cap) * 4 + 64; }
__host__ __device__ inline LdsPlan lds_plan(int LB, int nwaves, int cap, int tsize, bool learned, bool hyb) {
  const int seeds = 64 / cap;
  const int npl = xs_npl(tsize, learned, hyb);
  // FP32 values per lane in the stash: all 27 without the LDS state
  const int nst = npl < 0 ? 27 : 21 - npl;
  LdsPlan p;
  (void)LB;
  p.stash = 0;
  p.rec = align16(p.stash + (size_t)nwaves * nst * 64 * 4);
  p.recf = align16(p.rec + (size_t)nwaves * seeds * 27 * 4);
  const size_t tl_wave = (size_t)seeds * cap * 8 * 8;
  p.acc = align16(p.recf + (size_t)nwaves * seeds * 5 * 4);
  p.pub = align16(p.acc + (size_t)nwaves * 64 * NP);
  p.tl = align16(p.pub + (size_t)nwaves * pub_bytes(cap));
  if (learned) {
    const size_t per = tl_wave > KFMLP_LDS_BYTES ? tl_wave : (size_t)KFMLP_LDS_BYTES;
    p.mlp = p.tl;
    p.total = p.mlp + (size_t)nwaves * per;
    p.tl_stride = per;
  } else {
    p.mlp = p.total = align16(p.tl + (size_t)nwaves * tl_wave);
    p.tl_stride = tl_wave;
  }
  p.xs = p.total;
  if (npl >= 0) p.total = align16(p.xs + (size_t)nwaves * (6 + npl) * 64 * 8);
  return p;
}
// Lanes of a block (256, 128 or 64) with which the LDS of a CU holds the most
// waves, of which its registers allow eight; the widest of those, 0 if none
// fits.  FP64 builds at small caps, whose records or pools take more than half
// a CU's LDS for four waves: 20 events in the hybrid state at cap 2, 2.99 ms with
// four waves per CU, 2.21 with seven.
inline int plan_lanes(int LB, int cap, int tsize, bool learned, bool hyb, size_t lds) {
  int best = 0, most = 0;
  for (int lanes = 256; lanes >= 64; lanes /= 2) {
    const size_t waves = lds / lds_plan(LB, lanes / 64, cap, tsize, learned, hyb).total * (lanes / 64);
    if ((int)(waves < 8 ? waves : 8) > most) {
      most = (int)(waves < 8 ? waves : 8);
      best = lanes;
    }
  }
  return best;
}
