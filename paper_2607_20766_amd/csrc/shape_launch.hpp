// Launch rules that depend on sizes alone.  Plain host C++ without HIP, so that
// they can be checked at sizes no test would launch.
#pragma once

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

}  // namespace shape
