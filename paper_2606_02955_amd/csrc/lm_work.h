// lm_work.h -- how the LM head's tiles are shared by the workgroups: plain
// functions of the number of candidates, the vocabulary and the hidden size,
// evaluated on the device (the host does not know the number of candidates).
// Internal to libfdllm.so; compiled for the host as well, to be tested there.
#ifndef FDLLM_LM_WORK_H
#define FDLLM_LM_WORK_H

#include <stddef.h>

#ifdef __HIPCC__
#define FDLLM_HD __host__ __device__
#else
#define FDLLM_HD
#endif

namespace fdllm {

// The candidates are cut into the fewest position tiles of at most 256, and
// the tiles are as narrow (32, 64, 128, 192, 256 positions) as then still
// holds them: a narrow tile saves the matrix work and the reads of the hidden
// states of positions that are not there.  The vocabulary is cut into `k`
// ranges, the same for every position tile: a range's running maximum decides
// how its terms are rounded, so equal hidden rows have equal results only
// where they meet the same ranges.
//
// One position tile: a range per workgroup (one workgroup per compute unit),
// in steps of 16 rows, so every workgroup reads the same number of weight
// rows.  Several: ranges of whole weight tiles, each (position tile, range) a
// segment; the k with the shortest time of the workgroup with the most to do,
// among those of kLmRounds numbers of segments a workgroup from the smallest
// possible on.  More and shorter segments share the work more evenly, but each
// costs what kLmSegmentD hidden elements of a weight tile cost to fill and
// drain its stages and combine its states.  Against an even share of all
// (position tile, weight tile) pairs with ranges that differ from tile to
// tile: 13 position tiles at d = 4096, V = 126464 3140 -> 2466 us, 3 tiles
// 701 -> 600, 11 tiles at d = 1024, V = 50257 268 -> 250, 16 tiles the same;
// 38 tiles at d = 64, V = 16000, where 63 weight tiles leave no better k,
// 96 -> 100.
constexpr int kLmGroups = 256;
constexpr int kLmXcds = 8;                     // workgroup g runs on die g % 8
constexpr int kLmVt = 256;                     // vocabulary rows per tile (MFMA A operand)
constexpr int kLmMaxPt = 256;                  // positions per tile at most (MFMA B operand)
constexpr int kLmRounds = 8;
constexpr int kLmSegmentD = 192;

struct LmWork {
  int mt, pt;        // position tiles and their width
  int unit, nb;      // vocabulary rows per unit, units of the vocabulary
  int k;             // ranges of the vocabulary, at most kLmGroups
};

// Everything but k where there are several position tiles.
FDLLM_HD inline LmWork lm_work_tiles(int n, int V) {
  LmWork w;
  w.mt = (n + kLmMaxPt - 1) / kLmMaxPt;
  const int per = w.mt ? (n + w.mt - 1) / w.mt : 0;
  w.pt = per <= 32 ? 32 : per <= 64 ? 64 : per <= 128 ? 128 : per <= 192 ? 192 : 256;
  w.unit = w.mt > 1 ? kLmVt : 16;
  w.nb = (V + w.unit - 1) / w.unit;
  w.k = w.nb < kLmGroups ? w.nb : kLmGroups;
  return w;
}

// The ranges where workgroups have `round` + ceil(mt / kLmGroups) segments, and
// the time of the longest one (in hidden elements of a weight tile).
FDLLM_HD inline int lm_round_ranges(const LmWork& w, int round) {
  const long long r = (w.mt + kLmGroups - 1) / kLmGroups + round;
  const int k = (int)(r * kLmGroups / w.mt);
  const int most = w.nb < kLmGroups ? w.nb : kLmGroups;
  return k < most ? k : most;
}
FDLLM_HD inline unsigned long long lm_round_time(const LmWork& w, int k, int d) {
  const long long segments = ((long long)w.mt * k + kLmGroups - 1) / kLmGroups;
  const long long tiles = (w.nb + k - 1) / k;
  return (unsigned long long)segments * (unsigned long long)(tiles * d + kLmSegmentD);
}

FDLLM_HD inline LmWork lm_work(int n, int V, int d) {
  LmWork w = lm_work_tiles(n, V);
  if (w.mt <= 1) return w;
  unsigned long long best = ~0ull;
  for (int round = 0; round < kLmRounds; ++round) {
    const int k = lm_round_ranges(w, round);
    const unsigned long long t = lm_round_time(w, k, d);
    if (t < best) {
      best = t;
      w.k = k;
    }
  }
  return w;
}

// First unit of range s: floor(s nb / k).
FDLLM_HD inline int lm_first(const LmWork& w, int s) {
  const int q = w.nb / w.k, r = w.nb % w.k;
  return s * q + s * r / w.k;
}

// Segments of workgroup g: u = lm_seg_first(w, g), and every
// (kLmGroups / kLmXcds)-th from there below lm_seg_end(w, g); segment u is
// range u / mt of position tile u % mt.  With several position tiles the dies
// have contiguous ranges each, and a die's workgroups neighbouring segments at
// the same time, so the position tiles on the same weight rows, and the
// workgroups on the same hidden rows, share its L2, whatever the number of
// position tiles.
FDLLM_HD inline int lm_seg_first(const LmWork& w, int g) {
  if (w.mt == 1) return g;
  return (int)((long long)(g % kLmXcds) * w.mt * w.k / kLmXcds) + g / kLmXcds;
}
FDLLM_HD inline int lm_seg_end(const LmWork& w, int g) {
  if (w.mt == 1) return g < w.k ? g + 1 : g;
  return (int)((long long)(g % kLmXcds + 1) * w.mt * w.k / kLmXcds);
}

// Most partial results (one per candidate and range) of any number of
// candidates up to n.
inline size_t lm_max_partials(long long n, int V) {
  const long long one = (n < kLmMaxPt ? n : kLmMaxPt) * (long long)kLmGroups;
  const long long mt = (n + kLmMaxPt - 1) / kLmMaxPt;
  if (mt <= 1) return (size_t)one;
  // k <= kLmGroups, k <= the weight tiles, mt k <= kLmGroups (rounds of mt)
  const long long rounds = (mt + kLmGroups - 1) / kLmGroups + kLmRounds - 1;
  const long long tiles = (V + kLmVt - 1) / kLmVt;
  long long most = mt * (tiles < kLmGroups ? tiles : kLmGroups);
  if (most > rounds * kLmGroups) most = rounds * kLmGroups;
  most *= kLmMaxPt;
  return (size_t)(one > most ? one : most);
}

}  // namespace fdllm

#endif  // FDLLM_LM_WORK_H
