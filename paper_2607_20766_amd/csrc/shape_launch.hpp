// Launch rules that depend on sizes alone.  Plain host C++ without HIP, so that
// they can be checked at sizes no test would launch.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace shape {

// A launch takes fewer than 2^32 work-items (threads times workgroups) along x;
// more are refused as an invalid configuration.
constexpr int64_t kMaxWorkItems = ((int64_t)1 << 32) - 1;
inline int64_t max_workgroups(int threads) { return kMaxWorkItems / threads; }

// Waves (starts in flight) of an alignment's workgroup, one workgroup per pair
// and group of starts: eight share the samples of A where that leaves two
// workgroups per compute unit and their LDS fits (eight_fit), else four, the least
// a call is checked for.
constexpr int kAlignMinWaves = 4;
constexpr int kAlignMaxWaves = 8;
inline int align_waves(int64_t n_pairs, int n_starts, bool eight_fit, int n_cu) {
  const bool eight = n_pairs * n_starts >= (int64_t)2 * kAlignMaxWaves * n_cu &&
                     n_starts >= kAlignMaxWaves && eight_fit &&
                     n_pairs <= max_workgroups(kAlignMaxWaves * 64);
  return eight ? kAlignMaxWaves : kAlignMinWaves;
}

// Whether a workgroup's dynamic LDS and its kernel's own (rounded up to 16 bytes,
// the dynamic part's alignment) are within what the device allows.
inline bool align_split_fits(size_t dynamic, size_t own, size_t max_lds) {
  return dynamic + (own + 15) / 16 * 16 <= max_lds;
}

// Rounds of a pair that its workgroup works on at a time, a wave each, in screens
// that one wave per pair leaves short of waves: four rounds and two rounds fill the
// chip up to kFourRoundPairsPerCu (28 pairs per compute unit are fewer than eight
// waves per SIMD) and kTwoRoundPairsPerCu, or where a pair's LDS (lds bytes) leaves
// a compute unit few pairs.  Rounds drawn past an adaptive pair's stop are dropped,
// (R - 1)/2 on average, so R falls as a round grows; n_rounds is the most a pair
// takes.  One : two : four rounds, ms:
//   few pairs          5,000 molecules of 10-50 atoms, adaptive 0.58 : 0.51 :
//                      0.49; 8,000 0.78 : 0.71 : 0.72; 11,000 1.00 : 0.92 : 0.96;
//                      13,000 1.09 : 1.07 : 1.14; 16,000 1.29 : 1.30 : 1.37
//   LDS per pair       20,000 of 50-100 atoms (17 pairs' records in a compute
//                      unit's LDS) 3.04 : 2.63 : 2.78; 60,000 of 30-70 (25) 6.59
//                      : 6.53 : 6.90; of 30-60 (28) 6.49 : 6.52 : 6.88; 20,000
//                      of 100-150 (11) fixed 3.09 : 2.59 : 2.32, of 200-256 (6)
//                      6.98 : 5.03 : 3.99
//   long rounds        8,000 pairs, 1,024 samples per side and round 0.81 :
//                      0.77 : 0.88
// One workgroup per pair: R also falls until the launch holds them (2^24 pairs of
// four waves are too many).
constexpr int kSplitPairsPerCu = 3;  // up to here rounds of 256 samples: eight waves per pair
constexpr int kFourRoundPairsPerCu = 28;
constexpr int kTwoRoundPairsPerCu = 50;
inline int screen_rounds(bool adaptive, int64_t n_pairs, int64_t n_rounds, int round_side,
                         int64_t lds, int n_cu) {
  constexpr int64_t kLdsPerCu = 160 * 1024;
  const int64_t resident = kLdsPerCu / lds;
  int R = 1;
  if (n_pairs <= (int64_t)kTwoRoundPairsPerCu * n_cu || resident <= 25) R = 2;
  if (n_pairs <= (int64_t)kFourRoundPairsPerCu * n_cu || resident <= 11) R = 4;
  if (adaptive && n_pairs > (int64_t)kSplitPairsPerCu * n_cu)
    while (R > 1 && R * round_side > 1024) R /= 2;
  while (R > n_rounds || (R > 1 && n_pairs > max_workgroups(R * 64))) R /= 2;
  return R;
}

}  // namespace shape
