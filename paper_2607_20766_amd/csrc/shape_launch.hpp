// Launch rules that depend on sizes alone.  Plain host C++ without HIP, so that
// they can be checked at sizes no test would launch.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace shape {

// A launch takes fewer than 2^32 work-items (threads times workgroups) along x;
// more are refused as an invalid configuration.
constexpr int64_t kMaxWorkItems = ((int64_t)1 << 32) - 1;
inline int64_t max_workgroups(int threads) { return kMaxWorkItems / threads; }

// Whether two molecule sets, `blocks` workgroups of 256 threads together, are prepared in
// a launch each: too many for one, and neither is empty.
inline bool prepare_apart(int64_t blocks, int n_a, int n_b) {
  return blocks > max_workgroups(256) && n_a > 0 && n_b > 0;
}

// Alignments (k_align, k_align_split): how starts are spread over waves and
// workgroups.  Every shape gives the same bits.
//
// Whether every start runs by itself in a workgroup of sixteen waves.  Of these
// `busy` have samples (two slots of 64 each), and every workgroup draws A's samples,
// about the work of one evaluation: the fewer are busy, and the fewer evaluations
// there are, the fewer starts it takes for one wave per start to be as fast.  15-45
// atoms, split : four waves of a start each, us:
//   8 steps     256 samples (two busy), 400 starts 110 : 97, 800 184 : 99, 2,000 369 :
//               104; 512 (four) 800 194 : 165, 2,000 380 : 177; 1,000 (eight) 1,600 391
//               : 328; 2,048 (sixteen) 160 280 : 520, 2,000 720 : 610
//   none        256 samples, 550 starts 33 : 27; 512, 550 34 : 29; 1,000, 1,000 54 : 48;
//               2,048, 1,000 equal
// Steps of small molecules (mean_b atoms in B on average) are mostly the part that one
// wave takes by itself, so fewer starts still: 2,048 samples, 8 steps, 1,600 starts of 2-8
// atoms 286 : 172, 10-20 398 : 321.
// resident: waves of k_align with a start that a compute unit's LDS holds (the samples
// take 16 bytes each).  With one per SIMD or less (two per compute unit for small molecules
// and single evaluations) every wave waits for its own chain alone, however many starts
// there are: 5,000 pairs x 1 start, 8 steps of 4,096 samples 3.4 : 8.0 ms, of 2,048 1.8 :
// 2.2; 2,000 x 2 of 4,096 2.6 : 3.5 (x 4, 500 pairs 1.3 : 1.2); 20,000 x 1 of 2-8 atoms and
// 2,048 samples, 2 steps 1.5 : 1.3.
inline bool align_splits_starts(int64_t n_pairs, int n_starts, int n_steps, int busy,
                                int resident, double mean_b, int n_cu) {
  if (n_starts > 65535 || n_pairs > max_workgroups(1024)) return false;
  if (resident <= (n_steps > 0 && mean_b >= 12.0 ? 4 : 2)) return true;
  const double per_cu = n_steps > 0 ? std::min(7.0, 0.5 * (busy + 1))
                                    : std::min(4.0, 0.25 * (busy + 4));
  return (double)n_pairs * n_starts <= per_cu * std::min(1.0, 0.3 + mean_b / 43.0) * n_cu;
}

// Waves (starts in flight) of a workgroup: eight share the samples of A where that
// leaves two workgroups per compute unit and their LDS fits (eight_fit), else four, the
// least a call is checked for.  Four also where there are pairs enough and the last
// eight starts would fill half of the waves or less (eight : four, one evaluation of
// 3,000 pairs, 256 samples: 9 starts 158 : 131 us, 20 256 : 228; 16 201 : 203), unless
// LDS holds only two workgroups (crowded; 1,000 pairs x 9 of 4,096 569 : 655).
constexpr int kAlignMinWaves = 4;
constexpr int kAlignMaxWaves = 8;
inline int align_waves(int64_t n_pairs, int n_starts, bool eight_fit, bool crowded, int n_cu) {
  const int last = n_starts % kAlignMaxWaves;
  const bool full = last == 0 || last > kAlignMinWaves;
  const bool eight = n_pairs * n_starts >= (int64_t)2 * kAlignMaxWaves * n_cu &&
                     n_starts >= kAlignMaxWaves &&
                     (full || crowded || n_pairs < (int64_t)3 * n_cu) && eight_fit &&
                     n_pairs <= max_workgroups(kAlignMaxWaves * 64);
  return eight ? kAlignMaxWaves : kAlignMinWaves;
}

// Starts that a workgroup takes: with many pairs all of its pair's, so that A's samples
// are drawn once (3,000 pairs x 16 starts, one evaluation of 256 samples: 201 us with
// eight, 186 with all); with few as many as it has waves, so that there are more
// workgroups (300 x 16: 34 : 40), or eight (1,000 x 9: four 53, eight 50, all 47; 4 steps
// 187 : 187 : 194).
inline int align_starts_per_block(int64_t n_pairs, int n_starts, int waves, int n_cu) {
  if (n_pairs >= (int64_t)8 * n_cu) return n_starts;
  const int some = n_pairs >= (int64_t)3 * n_cu ? kAlignMaxWaves : waves;
  return std::max(some, (n_starts + 65534) / 65535);
}

// Whether a workgroup's dynamic LDS and its kernel's own (rounded up to 16 bytes,
// the dynamic part's alignment) are within what the device allows.
inline bool align_split_fits(size_t dynamic, size_t own, size_t max_lds) {
  return dynamic + (own + 15) / 16 * 16 <= max_lds;
}

// Sample points per lane that a screen evaluates together: four, or two where the last
// four of a lane's slots in a round (per_lane of them) would be half empty or more (one
// wave per pair, 40,000 pairs, four : two points, ms: 2 slots 2.37 : 1.31, 4 1.27 : 1.31, 5
// 1.96 : 1.56, 6 1.67 : 1.33, 7 1.47 : 1.54, 22 1.78 : 1.71).
inline int screen_points(int per_lane) {
  return per_lane % 4 == 1 || per_lane % 4 == 2 ? 2 : 4;
}

// Rounds that adaptive pairs take to SE(T) <= tau, on average and roughly: 17 rounds of
// 256 samples per side for 30 atoms against 10-50 at tau 0.005, going as 1/tau^2, fewer
// where the molecules differ in size (measured : this, tau 0.005, a query of 30 against 1-4
// atoms 2.2 : 2.5, 4-12 9.0 : 8.2, 50-100 11.9 : 12.2, 150-256 4.9 : 4.6).  Only kernels
// are chosen by it.
inline double screen_rounds_expected(double tau, int round_side, double query_atoms,
                                     double library_atoms) {
  const double large = std::max(query_atoms, library_atoms);
  const double alike = std::min(1.0, 1.75 * std::min(query_atoms, library_atoms) / large);
  return 0.112 / (tau * tau * round_side) * alike * std::pow(std::max(1.0, 25.0 / large), 0.6);
}

// Rounds of a pair that its workgroup works on at a time, a wave each, and those of its
// first pass: all of them, and then in every pass, or fewer (but what the pair's budget
// holds), and then as many as the pair still seems to need.
// Several rounds where one wave per pair leaves a compute unit short of waves:
//   LDS per pair       (lds bytes) for the rounds: 20,000 molecules of 50-100 atoms (17
//                      pairs in a compute unit's LDS), one : two : four rounds 3.04 : 2.63 :
//                      2.78 ms; 60,000 of 30-70 (25) 6.59 : 6.53 : 6.90, of 30-60 (28) 6.49 :
//                      6.52 : 6.88; 20,000 of 100-150 (11) fixed 3.09 : 2.59 : 2.32, of
//                      200-256 (6) 6.98 : 5.03 : 3.99
//   few pairs          fixed mode, four up to 28 pairs per compute unit (fewer than eight
//                      waves per SIMD), two up to 50; 2,048 samples per side, one : these:
//                      3,000 molecules 160 : 140 us, 7,100 308 : 280, 9,000 (two) 364 :
//                      350, 12,700 480 : 472; 512 samples equal from 5,000 on
// Adaptive pairs have to need them, or they leave their other waves idle, and a pass more
// costs about what two dropped rounds do.  Molecules of 10-50 atoms, 30-atom query (e:
// expected; one : two : two after a first of one : four : four after a first of one), us:
//   pairs  800  e 1.1    46 :   41 :   46 :   40 :   46
//         1500  e 2.2    74 :   61 :   66 :   56 :   66
//         3500  e 4.4   156 :  141 :  152 :  139 :  152
//         5000  e 4.4   177 :  166 :  181 :  180 :  195
//         7000  e 8.9   391 :  359 :  394 :  375 :  413
//         9000  e 8.9   452 :  435 :  479 :  466 :  513
//         9000  e 2.2   158 :  168 :  178 :  198 :  218
// of 50-100 atoms, 64-atom query:
//          800  e 1.1    69 :   51 :   69 :   62 :   68
//         9000  e 4.4   473 :  406 :  415 :  419 :  473
//         9000  e 2.2   295 :  261 :  289 :  365 :  343
//         9000  e 1.1   198 :  212 :  194 :  366 :  221
// and of 160-250 atoms, 200-atom query (e 2.2: four after a first of two 689):
//         9000  e 4.4  1536 : 1234 : 1322 : 1003 : 1210
//         9000  e 2.2   916 :  711 :  908 :  907 :  905
//         9000  e 1.1   567 :  645 :  553 :  909 :  542
// Over 906 such screens (1-250 atoms, 800-20,000 pairs, SE(T) 0.003 to 0.05) this rule
// takes 1.01 times the fastest of the six shapes and at most 1.06 times one wave per pair.
// Up to three pairs per compute unit (rounds of other sizes than 256) four from e 1: 700
// pairs of 150-256 atoms, 1,024 samples per side and round, e 1.2 263 us, two 306, one 480.
// Otherwise long rounds do not repay a dropped one (8,000 pairs, 1,024 samples per side and
// round 0.81 : 0.77 : 0.88 ms).
// A budget (seeded) only adds to what tau asks for, on the device: several rounds then by
// the number of pairs alone (budgets of 4.7 rounds on average, up to 37, tau 0.02, 3,000
// pairs of 10-50 atoms, one : two : four 517 : 268 : 158 us; all budgets one round 73 : 71 :
// 82), whole where tau alone needs many (a triage's best 8,385 of 167,696 molecules,
// 11-atom query, tau 0.005: 868 us, from the budgets 952).
// One workgroup per pair: the rounds fall until a launch holds them.  n_rounds is the most
// a pair takes, expected what tau asks for on average.
constexpr int kSplitPairsPerCu = 3;  // up to here rounds of 256 samples: eight waves per pair
struct ScreenShape {
  int rounds, first;
};
inline ScreenShape screen_shape(bool adaptive, bool seeded, int64_t n_pairs, int64_t n_rounds,
                                double expected, int round_side, int64_t lds, int n_cu) {
  constexpr int64_t kLdsPerCu = 160 * 1024;
  const int64_t resident = kLdsPerCu / lds;
  const auto up_to = [&](int per_cu) { return n_pairs <= (int64_t)per_cu * n_cu; };
  const double e = expected;
  int few = up_to(28) ? 4 : (up_to(50) ? 2 : 1);
  int room = resident <= 11 ? 4 : (resident <= 25 ? 2 : 1);
  if (adaptive && !seeded && !up_to(1)) {
    if (e < (up_to(kSplitPairsPerCu) ? 1.0 : (up_to(14) ? 1.9 : 10.0)))
      few = (up_to(8) && e >= 0.7) || (up_to(28) && e >= 2.5) || (up_to(50) && e >= 5.0) ? 2 : 1;
    if (e < 1.9) room = std::min(room, 2);
  }
  if (adaptive && !up_to(kSplitPairsPerCu))
    while (few > 1 && few * round_side > 1024) few /= 2;
  int R = std::max(few, room);
  while (R > n_rounds || (R > 1 && n_pairs > max_workgroups(R * 64))) R /= 2;
  int first = 1;
  // whole passes also where most pairs' waves run at once anyway
  const bool at_once = up_to(14) && 5 * n_pairs <= 3 * resident * n_cu;
  if (!adaptive || up_to(1) || e >= 3.5 || (e >= 1.9 && at_once) ||
      (e >= 1.0 && up_to(kSplitPairsPerCu)))
    first = R;
  else if (e >= 1.9 || (e >= 0.7 && up_to(8)))
    first = std::min(2, R);
  return {R, first};
}

}  // namespace shape
