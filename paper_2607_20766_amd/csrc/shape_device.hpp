// Device primitives of the IS shape-overlap engine (gfx950, wave64).
//
// Everything here runs in FP32 on the vector ALU except Philox (32-bit
// integer multiplies) and the per-molecule preparation (FP64).  Notation
// follows the paper: o_i = exp(-alpha_i |r - c_i|^2), m = sum o_i,
// u = 1 - prod (1 - o_i), w = u / m, Z = sum (pi/alpha_i)^(3/2).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "shape_normal_poly.hpp"

namespace shape {

constexpr int kWave = 64;

// Prepared atom record used by every hot loop: centre and the exponent scale
// for exp2, a2 = alpha * log2(e), so that o = exp2(-a2 |r - c|^2).
struct __align__(16) Atom {
  float x, y, z, a2;
};

// Sampling record of an atom: standard deviation 1/sqrt(2 alpha) of its
// mixture component and the component-selection threshold (word 0 of the
// Philox block selects component j = #{i < N-1 : word0 >= thr_i}).
struct __align__(8) AtomSampling {
  float sd;
  uint32_t thr;
};

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): ten rounds; each round multiplies
// words 0 and 2 by the two round constants and mixes high halves with the
// other words and the key; the key advances by the Weyl constants.  The
// products are written as 32x32->64-bit multiplies so that each is one
// v_mad_u64_u32 rather than a v_mul_hi_u32/v_mul_lo_u32 pair.
// ---------------------------------------------------------------------------
// The three-way XORs are one v_bitop3_b32 each (truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint2 k) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = make_uint4(xor3((uint32_t)(p1 >> 32), c.y, k.x), (uint32_t)p1,
                   xor3((uint32_t)(p0 >> 32), c.w, k.y), (uint32_t)p0);
    k.x += 0x9E3779B9u;
    k.y += 0xBB67AE85u;
  }
  return c;
}

// N transcendental operations f(0) .. f(N-1), issued back to back at raised
// wave priority.  gfx950 co-issues the FP32 operations of two waves of a SIMD
// (two cycles each) only while both stand at one; a transcendental takes the
// SIMD for eight cycles alone.  At equal priority the waves gather at their
// transcendentals and the FMAs around them go out one by one, four cycles
// each; with the transcendentals first, waves leave them at once and gather
// at their FMAs instead.  Measured for streams of one exponential per five
// FMAs: 24.8 -> 19.0 cycles with eight or four waves per SIMD (18.3 if every
// FMA were co-issued), one per twelve FMAs: 47.9 -> 33.4; groups of 4, 8 and
// 16 measure the same, single exponentials 20.0.
constexpr int kTransPrio = 3;
template <int N, class F>
__device__ __forceinline__ void trans_group(F f) {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(kTransPrio);
#pragma unroll
  for (int i = 0; i < N; ++i) f(i);
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
}

// o = exp2(-e) for a group of N exponents.
template <int N>
__device__ __forceinline__ void exp2_group(float (&e)[N]) {
  trans_group<N>([&](int i) { e[i] = __builtin_amdgcn_exp2f(-e[i]); });
}

// Atoms taken together by the evaluators below, so that a group holds eight
// exponentials (and one loop step) whatever the number of points per lane.
constexpr int exp_atoms(int S) { return S >= 8 ? 1 : 8 / S; }

// Standard normals from the top 24 bits b of N Philox words: u = (b + 1/2) 2^-24,
// z = Phi^-1(u) = sqrt(2) erfinv(x), x = 2u - 1 = b 2^-23 + (2^-24 - 1), which
// one FP32 fma forms exactly, so the tails are resolved to the last bit.
// erfinv after Giles (2011): z = x P(L), L = -log2(1 - x^2) (1 - x^2 >= 2^-24 (1 +
// 2^-24)), with one polynomial in L for L < kSplit and one in sqrt(L) above it
// (coefficients from gen_normal_poly.py; relative error below 3e-7 over every 24-bit u).
// The logarithms are issued as one group at raised priority (see exp2_group), and
// the tail is evaluated only where a lane of the wave needs it.
template <int N>
__device__ __forceinline__ void normals_from_bits(const uint32_t (&word)[N], float (&z)[N]) {
  using namespace normal_poly;
  float x[N], L[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    x[i] = fmaf((float)(word[i] >> 8), 0x1p-23f, 0x1p-24f - 1.0f);
    const float ax = fabsf(x[i]);
    L[i] = (1.0f - ax) * (1.0f + ax);
  }
  trans_group<N>([&](int i) { L[i] = -__builtin_amdgcn_logf(L[i]); });
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float t = fmaf(L[i], kCenScale, kCenOff);
    float p = kCen[8];
#pragma unroll
    for (int k = 7; k >= 0; --k) p = fmaf(p, t, kCen[k]);
    z[i] = x[i] * p;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (!(L[i] < kSplit)) {
      const float t = fmaf(__builtin_amdgcn_sqrtf(L[i]), kTailScale, kTailOff);
      float p = kTail[8];
#pragma unroll
      for (int k = 7; k >= 0; --k) p = fmaf(p, t, kTail[k]);
      z[i] = x[i] * p;
    }
  }
}

// Components of a molecule's mixture selected by D Philox words:
// j = #{i < n-1 : word >= thr_i}.  The thresholds are non-decreasing, so the
// count is found by binary lifting in ceil(log2(n)) steps (the step count is
// the same for every lane); every index read is below n-1.
template <int D>
__device__ __forceinline__ void select_components(const AtomSampling* samp, int n,
                                                  const uint32_t (&word)[D], int (&j)[D]) {
  const int last = n - 1;
#pragma unroll
  for (int d = 0; d < D; ++d) j[d] = 0;
  if (last <= 0) return;
  for (int step = 1 << (31 - __builtin_clz((unsigned)last)); step > 0; step >>= 1)
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int c = j[d] + step;
      const int idx = (c < last ? c : last) - 1;
      if (c <= last && word[d] >= samp[idx].thr) j[d] = c;
    }
}

// Guide table of a molecule's component choice, built once per molecule in
// LDS: guide[g] = #{i < n-1 : thr_i <= g 2^24} for the top eight bits g of
// a word.  Every threshold counted there lies at or below any word whose top
// bits are g, so that word's count starts at guide[g] and steps only over
// the thresholds inside its 2^24-wide bucket (on average (n-1)/256 of them):
// the same count as select_components', from one table read and a short
// scan instead of ceil(log2(n)) dependent reads.
constexpr int kGuideBits = 8;
constexpr int kGuideSize = 1 << kGuideBits;

__device__ __forceinline__ void build_guide(const AtomSampling* samp, int n, uint8_t* guide,
                                            int tid, int nthreads) {
  const int last = n - 1;
  for (int g = tid; g < kGuideSize; g += nthreads) {
    const uint32_t x = (uint32_t)g << (32 - kGuideBits);
    int c = 0;  // largest c <= last with thr_{c-1} <= x (thresholds non-decreasing)
    if (last > 0) {
      for (int step = 1 << (31 - __builtin_clz((unsigned)last)); step > 0; step >>= 1) {
        const int t = c + step;
        if (t <= last && samp[t - 1].thr <= x) c = t;
      }
    }
    guide[g] = (uint8_t)c;  // c <= last < 256
  }
}

// The components of D words together: each step reads one threshold per word,
// so the words' LDS latencies overlap.
template <int D>
__device__ __forceinline__ void select_components_guided(const AtomSampling* samp,
                                                         const uint8_t* guide, int n,
                                                         const uint32_t (&word)[D],
                                                         int (&j)[D]) {
  const int last = n - 1;
#pragma unroll
  for (int d = 0; d < D; ++d) j[d] = guide[word[d] >> (32 - kGuideBits)];
  for (bool more = true; more;) {
    more = false;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const bool step = word[d] >= samp[j[d]].thr && j[d] < last;  // j <= last: in range
      j[d] += step ? 1 : 0;
      more |= step;
    }
  }
}

// Samples of a molecule: exact draws from its normalised mixture.  Philox block k of
// the molecule's stream gives a component by integer thresholds and three normals, and
// the point r = c_j + z sd_j per axis.  Antithetic samples 2k and 2k + 1 share block k;
// the odd one is the reflection about its component's centre (z of opposite sign).
//
// Components and normals of D blocks x, the steps of all of them interleaved so that
// their latencies overlap; select(words, j) is select_components or its guided form.
template <int D, class Select>
__device__ __forceinline__ void draws_of(const uint4 (&x)[D], Select select, int (&j)[D],
                                         float (&z)[3 * D]) {
  uint32_t w0[D], wz[3 * D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    w0[d] = x[d].x;
    wz[3 * d] = x[d].y;
    wz[3 * d + 1] = x[d].z;
    wz[3 * d + 2] = x[d].w;
  }
  select(w0, j);
  normals_from_bits<3 * D>(wz, z);
}

__device__ __forceinline__ uint4 philox_block(uint64_t blk, uint32_t mol_id, uint2 key) {
  return philox4x32_10(make_uint4((uint32_t)blk, (uint32_t)(blk >> 32), mol_id, 0u), key);
}

// D draws together (blocks below 2^32) by binary lifting.
template <int D>
__device__ __forceinline__ void draws(const AtomSampling* samp, int n, uint32_t mol_id,
                                      const uint32_t (&blk)[D], uint2 key, int (&j)[D],
                                      float (&z)[3 * D]) {
  uint4 x[D];
#pragma unroll
  for (int d = 0; d < D; ++d) x[d] = philox_block(blk[d], mol_id, key);
  draws_of<D>(x, [&](const uint32_t (&w)[D], int (&c)[D]) { select_components<D>(samp, n, w, c); },
              j, z);
}

// The draws' points, or their reflections about the components' centres (sign = -1).
// atoms/samp point at the molecule's own records (LDS or global).
template <int D>
__device__ __forceinline__ void draw_points(const Atom* atoms, const AtomSampling* samp,
                                            const int (&j)[D], const float (&z)[3 * D],
                                            float sign, float (&rx)[D], float (&ry)[D],
                                            float (&rz)[D]) {
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const Atom c = atoms[j[d]];
    const float sd = samp[j[d]].sd;
    rx[d] = fmaf(sign * z[3 * d], sd, c.x);
    ry[d] = fmaf(sign * z[3 * d + 1], sd, c.y);
    rz[d] = fmaf(sign * z[3 * d + 2], sd, c.z);
  }
}

// First-order density m = sum o_i and union complement q = prod (1 - o_i) of a
// molecule at S points (the caller initialises m to 0 and q to 1; u = 1 - q),
// from the differences r - c_i.
template <int S>
__device__ __forceinline__ void eval_density(const Atom* __restrict__ atoms, int n,
                                             const float (&rx)[S], const float (&ry)[S],
                                             const float (&rz)[S], float (&m)[S],
                                             float (&q)[S]) {
  constexpr int U = exp_atoms(S);
  const auto group = [&](int i, auto count) {
    constexpr int V = decltype(count)::value;
    float o[V * S];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const Atom a = atoms[i + u];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float dx = rx[s] - a.x, dy = ry[s] - a.y, dz = rz[s] - a.z;
        o[u * S + s] = a.a2 * fmaf(dx, dx, fmaf(dy, dy, dz * dz));
      }
    }
    exp2_group(o);
#pragma unroll
    for (int u = 0; u < V; ++u)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        m[s] += o[u * S + s];
        q[s] = fmaf(-q[s], o[u * S + s], q[s]);
      }
  };
  int i = 0;
  for (; i + U <= n; i += U) group(i, std::integral_constant<int, U>{});
  if constexpr (U > 1)
    for (; i < n; ++i) group(i, std::integral_constant<int, 1>{});
}

// ---------------------------------------------------------------------------
// Expanded-quadratic atom records.  In a frame centred at `ref`, with
// c' = c - ref and r' = r - ref, the exponent of o = exp2(-e) is
//   e = a2 |r' - c'|^2 = a2 |r'|^2 + (-2 a2 c') . r' + a2 |c'|^2,
// four fused multiply-adds per atom once |r'|^2 is known for the point.
// Records are formed in FP64 and rounded once; frames keep |r'| at the size
// of a molecule so the cancellation in e stays at FP32 rounding level.
// ---------------------------------------------------------------------------
struct __align__(16) AtomRec {
  float bx, by, bz, c;  // -2 a2 c', a2 |c'|^2
};

__device__ __forceinline__ void make_rec(const Atom& a, float rx, float ry, float rz,
                                         AtomRec& rec, float& a2) {
  const double x = (double)a.x - (double)rx, y = (double)a.y - (double)ry,
               z = (double)a.z - (double)rz;
  const double k = (double)a.a2;
  rec.bx = (float)(-2.0 * k * x);
  rec.by = (float)(-2.0 * k * y);
  rec.bz = (float)(-2.0 * k * z);
  rec.c = (float)(k * (x * x + y * y + z * z));
  a2 = a.a2;
}

// Exponent e = a2 |r' - c'|^2 of an atom at a point, o = exp2(-e).
__device__ __forceinline__ float exponent_x(const AtomRec& b, float a2, float rx, float ry,
                                            float rz, float r2) {
  float e = fmaf(a2, r2, b.c);
  e = fmaf(b.bx, rx, e);
  e = fmaf(b.by, ry, e);
  return fmaf(b.bz, rz, e);
}

// Occupancies of n atoms at S points, folded in atom order:
// fold(s, o) is called for atom 0, 1, ... of each point s.
template <int S, class Fold>
__device__ __forceinline__ void eval_atoms_x(const AtomRec* __restrict__ rec,
                                             const float* __restrict__ a2, int n,
                                             const float (&rx)[S], const float (&ry)[S],
                                             const float (&rz)[S], const float (&r2)[S],
                                             Fold fold) {
  constexpr int U = exp_atoms(S);
  int i = 0;
  for (; i + U <= n; i += U) {
    float o[U * S];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const AtomRec b = rec[i + u];
      const float a = a2[i + u];
#pragma unroll
      for (int s = 0; s < S; ++s) o[u * S + s] = exponent_x(b, a, rx[s], ry[s], rz[s], r2[s]);
    }
    exp2_group(o);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < S; ++s) fold(s, o[u * S + s]);
  }
  if constexpr (U > 1) {
    for (; i < n; ++i) {
      const AtomRec b = rec[i];
      const float a = a2[i];
      float o[S];
#pragma unroll
      for (int s = 0; s < S; ++s) o[s] = exponent_x(b, a, rx[s], ry[s], rz[s], r2[s]);
      exp2_group(o);
#pragma unroll
      for (int s = 0; s < S; ++s) fold(s, o[s]);
    }
  }
}

// Two atoms' records in one 48-byte word, so that the inner loop needs one LDS
// address.  A molecule of odd size ends with a phantom atom: e = |r|^2 + 10^30,
// so o = 0 exactly at every point, also where |r|^2 overflows (a width of 0 would
// make that NaN), which changes no sum and no product.
struct __align__(16) AtomRec2 {
  AtomRec r[2];
  float a2[2];
  float pad[2];
};
__host__ __device__ constexpr int rec_pairs(int n) { return (n + 1) / 2; }

// Atom i of n of a molecule in the frame of (rx, ry, rz); the last atom of an
// odd molecule also writes the phantom.
__device__ __forceinline__ void make_rec2(const Atom& a, float rx, float ry, float rz,
                                          AtomRec2* rec, int i, int n) {
  AtomRec2& w = rec[i >> 1];
  make_rec(a, rx, ry, rz, w.r[i & 1], w.a2[i & 1]);
  if (i == n - 1 && (n & 1)) {
    w.r[1] = AtomRec{0.f, 0.f, 0.f, 1e30f};
    w.a2[1] = 1.f;
  }
}

// eval_atoms_x over such records: at least eight exponentials per group.  kAhead
// reads the next group's records before this one's terms, for kernels with too
// few waves to cover the LDS latency and registers to spare.
template <int S, bool kAhead, class Fold>
__device__ __forceinline__ void eval_pairs_x(const AtomRec2* __restrict__ rec, int n,
                                             const float (&rx)[S], const float (&ry)[S],
                                             const float (&rz)[S], const float (&r2)[S],
                                             Fold fold) {
  constexpr int U = S >= 4 ? 1 : 4 / S;  // records per group
  const auto group = [&](auto count, auto get) {
    constexpr int V = decltype(count)::value;
    float o[2 * V * S];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const AtomRec2 w = get(u);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < S; ++s)
          o[(2 * u + h) * S + s] = exponent_x(w.r[h], w.a2[h], rx[s], ry[s], rz[s], r2[s]);
    }
    exp2_group(o);
#pragma unroll
    for (int u = 0; u < 2 * V; ++u)
#pragma unroll
      for (int s = 0; s < S; ++s) fold(s, o[u * S + s]);
  };
  using Whole = std::integral_constant<int, U>;
  const int np = rec_pairs(n);
  int i = 0;
  if constexpr (kAhead) {
    const int whole = np / U * U;
    if (whole > 0) {
      AtomRec2 w0[U], w1[U];
      const auto read = [&](int j, AtomRec2 (&w)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = rec[j + u];
      };
      const auto first = [&](int u) { return w0[u]; };
      const auto second = [&](int u) { return w1[u]; };
      read(0, w0);
      for (; i + 2 * U <= whole; i += 2 * U) {
        read(i + U, w1);
        group(Whole{}, first);
        read(min(i + 2 * U, whole - U), w0);  // the last time read again, unused
        group(Whole{}, second);
      }
      if (i < whole) group(Whole{}, first);
      i = whole;
    }
  } else {
    for (; i + U <= np; i += U) group(Whole{}, [&](int u) { return rec[i + u]; });
  }
  if constexpr (U > 1)
    for (; i < np; ++i)
      group(std::integral_constant<int, 1>{}, [&](int u) { return rec[i + u]; });
}

// Union complement q = prod(1 - o_i) (the caller initialises q to 1, u = 1 - q),
// and the first-order density m with it, over pair records.
template <int S, bool kAhead = false>
__device__ __forceinline__ void eval_union_x2(const AtomRec2* rec, int n, const float (&rx)[S],
                                              const float (&ry)[S], const float (&rz)[S],
                                              const float (&r2)[S], float (&q)[S]) {
  eval_pairs_x<S, kAhead>(rec, n, rx, ry, rz, r2,
                  [&](int s, float o) { q[s] = fmaf(-q[s], o, q[s]); });
}
template <int S, bool kAhead = false>
__device__ __forceinline__ void eval_density_x2(const AtomRec2* rec, int n, const float (&rx)[S],
                                                const float (&ry)[S], const float (&rz)[S],
                                                const float (&r2)[S], float (&m)[S],
                                                float (&q)[S]) {
  eval_pairs_x<S, kAhead>(rec, n, rx, ry, rz, r2, [&](int s, float o) {
    m[s] += o;
    q[s] = fmaf(-q[s], o, q[s]);
  });
}

// First-order density m and union complement q at S points (expanded form).
template <int S>
__device__ __forceinline__ void eval_density_x(const AtomRec* __restrict__ rec,
                                               const float* __restrict__ a2, int n,
                                               const float (&rx)[S], const float (&ry)[S],
                                               const float (&rz)[S], const float (&r2)[S],
                                               float (&m)[S], float (&q)[S]) {
  eval_atoms_x<S>(rec, a2, n, rx, ry, rz, r2, [&](int s, float o) {
    m[s] += o;
    q[s] = fmaf(-q[s], o, q[s]);
  });
}

// First-order density m and union u itself at S points (expanded form), u
// by the cancellation-free recurrence u <- u + o - u o.  Slightly dearer than
// tracking q = 1 - u, but u keeps its relative precision where every o_i is
// small, so w = u/m stays accurate in a molecule's tails (where a moved
// partner can sit during alignment).
template <int S>
__device__ __forceinline__ void eval_density_u_x(const AtomRec* __restrict__ rec,
                                                 const float* __restrict__ a2, int n,
                                                 const float (&rx)[S], const float (&ry)[S],
                                                 const float (&rz)[S], const float (&r2)[S],
                                                 float (&m)[S], float (&u)[S]) {
  eval_atoms_x<S>(rec, a2, n, rx, ry, rz, r2, [&](int s, float o) {
    m[s] += o;
    u[s] = fmaf(-u[s], o, u[s] + o);
  });
}

// |r|^2 of a point.
__device__ __forceinline__ float norm2(float x, float y, float z) {
  return fmaf(x, x, fmaf(y, y, z * z));
}

// Bounded weight w = u/m in [0, 1] (m > 0 for every sampled point; guard 0).
// u times the hardware reciprocal of m: within 2 ulp of the quotient.
__device__ __forceinline__ float bounded_weight(float u, float m) {
  return m > 0.0f ? fminf(u * __builtin_amdgcn_rcpf(m), 1.0f) : 0.0f;
}

// ---------------------------------------------------------------------------
// Wave-level reductions (fixed butterfly order: deterministic).
// ---------------------------------------------------------------------------
// A butterfly over XOR partners 32, 16, 8, 4, 2, 1 on the vector ALU, without
// LDS round trips: the halves and the rows of 16 are exchanged by gfx950's
// permlane swaps; inside a row the partner of step d is reached by rotating
// the row by d places, since by then the values repeat every 2 d lanes.
// Every lane ends with the same bits (a sum of two does not depend on their
// order).
template <int Ctrl>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)b, Ctrl, 0xf, 0xf, true);
  const long long hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), Ctrl, 0xf, 0xf, true);
  return __longlong_as_double((hi << 32) | lo);
}
__device__ __forceinline__ double f64_of(unsigned lo, unsigned hi) {
  return __longlong_as_double(((long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
  {
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32),
                                                     false, false);
    v = f64_of(lo[0], hi[0]) + f64_of(lo[1], hi[1]);
  }
  {
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32),
                                                     false, false);
    v = f64_of(lo[0], hi[0]) + f64_of(lo[1], hi[1]);
  }
  v += dpp_f64<0x128>(v);  // row_ror:8
  v += dpp_f64<0x124>(v);  // row_ror:4
  v += dpp_f64<0x122>(v);  // row_ror:2
  v += dpp_f64<0x121>(v);  // row_ror:1
  return v;
}

// Wave sum by DPP: an inclusive scan inside each row of 16 lanes (shifts 1,
// 2, 4, 8), then lane 15 of rows 0 and 2 is added into rows 1 and 3 and lane
// 31 into rows 2 and 3, leaving the total in lane 63, which is returned to
// every lane.  Fixed order: deterministic.
template <int Ctrl, int RowMask>
__device__ __forceinline__ float dpp_step(float v) {
  const int s = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), Ctrl, RowMask, 0xf, true);
  return v + __builtin_bit_cast(float, s);
}
// Sum over each row of 16 lanes, returned to all 16 lanes of the row: XOR
// partners 1 and 2 inside each quad (quad_perm), then the mirror lane of the
// other quad (row_half_mirror) and of the other half row (row_mirror).  Each
// step adds two partials that the partner lane adds in the other order, and
// the sum of two floats does not depend on their order, so every lane of a
// row ends with the same bits.
__device__ __forceinline__ float row_sum16(float v) {
  v = dpp_step<0xB1, 0xf>(v);   // quad_perm [1,0,3,2]
  v = dpp_step<0x4E, 0xf>(v);   // quad_perm [2,3,0,1]
  v = dpp_step<0x141, 0xf>(v);  // row_half_mirror
  v = dpp_step<0x140, 0xf>(v);  // row_mirror
  return v;
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v = dpp_step<0x111, 0xf>(v);  // row_shr:1
  v = dpp_step<0x112, 0xf>(v);  // row_shr:2
  v = dpp_step<0x114, 0xf>(v);  // row_shr:4
  v = dpp_step<0x118, 0xf>(v);  // row_shr:8
  v = dpp_step<0x142, 0xa>(v);  // row_bcast:15 into rows 1, 3
  v = dpp_step<0x143, 0xc>(v);  // row_bcast:31 into rows 2, 3
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

__device__ __forceinline__ float wave_sumf(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Workgroups go to the chip's eight XCDs, each with its own L2, in
// round-robin order of blockIdx.  xcd_chunk(b, G) renumbers them so that
// tiles of kXcdTile consecutive items are each handled by one XCD (tile t on
// XCD t mod 8): neighbouring molecules, whose records share cache lines, then
// meet in one L2 instead of being fetched by two, and a tile's outputs fill
// whole lines.  Tiles, not one contiguous range per XCD, keep the XCDs evenly
// loaded when the work per item drifts along the index (a sorted library).
// A bijection on [0, G): below F = G - G mod (8 kXcdTile) block b = 8 k + x
// (XCD x, its k-th block) takes item (8 (k / T) + x) T + k mod T, which runs
// over [0, F) once; blocks from F on keep their index.
constexpr int kXcds = 8;
constexpr int kXcdTile = 64;
__device__ __forceinline__ int xcd_chunk(int b, int G) {
  const int F = G - G % (kXcds * kXcdTile);
  if (b >= F) return b;
  const int x = b % kXcds, k = b / kXcds;
  return ((k / kXcdTile) * kXcds + x) * kXcdTile + k % kXcdTile;
}

// Lane l's FP64 value, read by every lane (l wave-uniform).
__device__ __forceinline__ double readlane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, l);
  const long long hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double((hi << 32) | lo);
}

// Orders LDS writes of this wave before its later LDS reads (wave-private
// staging needs no workgroup barrier).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace shape
