// Hybrid pipeline (section "Differentiable alignment and the hybrid
// pipeline"): rigid alignment on the analytic first-order overlap (Eq. fo,
// exact and cheap) from multiple starts — the given pose, the four proper
// principal-axis alignments and random rotations — then scoring of the
// superposed pair by the union estimator (the screening kernels).
//
// Pose convention as in the IS alignment: c''_j = R(q/|q|) c_j + t for B's
// atoms, q = (w, x, y, z) unnormalised, rotation about B's coordinate origin.
//
//   T_FO = O / (O_AA + O_BB - O),  O = sum_ij K_ij,
//   K_ij = (pi/(a_i+a_j))^(3/2) exp(-k_ij |c_i - c''_j|^2), k_ij = a_i a_j/(a_i+a_j)
//   dO/dc''_j = sum_i 2 k_ij K_ij (c_i - c''_j)
//   dO/dt = sum_j dO/dc''_j,  dO/dtheta = sum_j (c''_j - t) x dO/dc''_j
// and dT/dq follows from dtheta = 2 (w dv - dw v + v x dv) for q = (w, v).
#include "shape_kernels.hpp"

#include <algorithm>
#include <type_traits>

#include <math.h>

namespace shape {

// ---------------------------------------------------------------------------
// Starts, FP64.
// ---------------------------------------------------------------------------

// Symmetric 3x3 eigen-decomposition by cyclic Jacobi rotations: eigenvalues
// descending, unit eigenvectors in the columns of V (row-major).
__device__ void jacobi3(double a[3][3], double V[9]) {
  double U[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
  for (int sweep = 0; sweep < 60; ++sweep) {
    // every remaining rotation is below 10^-30 and no two eigenvalues are so
    // close that it could change their order: no component of U changes at
    // FP64.  Rounding leaves off-diagonals of 10^-16 of the rotated terms, so
    // waiting for them to vanish took about twenty sweeps instead of six.
    const double d01 = fabs(a[1][1] - a[0][0]), d02 = fabs(a[2][2] - a[0][0]),
                 d12 = fabs(a[2][2] - a[1][1]);
    if (fmin(fmin(d01, d02), d12) > 1e-10 * (fabs(a[0][0]) + fabs(a[1][1]) + fabs(a[2][2])) &&
        fabs(a[0][1]) <= 1e-30 * d01 && fabs(a[0][2]) <= 1e-30 * d02 &&
        fabs(a[1][2]) <= 1e-30 * d12)
      break;
    const double off = fabs(a[0][1]) + fabs(a[0][2]) + fabs(a[1][2]);
    if (off < 1e-300) break;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = p + 1; q < 3; ++q) {
        if (a[p][q] == 0.0) continue;
        const double theta = (a[q][q] - a[p][p]) / (2.0 * a[p][q]);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
        const double c = 1.0 / sqrt(t * t + 1.0), s = t * c;
        for (int k = 0; k < 3; ++k) {
          const double akp = a[k][p], akq = a[k][q];
          a[k][p] = c * akp - s * akq;
          a[k][q] = s * akp + c * akq;
        }
        for (int k = 0; k < 3; ++k) {
          const double apk = a[p][k], aqk = a[q][k];
          a[p][k] = c * apk - s * aqk;
          a[q][k] = s * apk + c * aqk;
        }
        for (int k = 0; k < 3; ++k) {
          const double ukp = U[k][p], ukq = U[k][q];
          U[k][p] = c * ukp - s * ukq;
          U[k][q] = s * ukp + c * ukq;
        }
      }
  }
  // columns by descending eigenvalue (registers only: no indexed arrays)
  double ev[3] = {a[0][0], a[1][1], a[2][2]};
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = i + 1; j < 3; ++j) {
      const bool swap = ev[j] > ev[i];
      const double e = ev[i];
      ev[i] = swap ? ev[j] : e;
      ev[j] = swap ? e : ev[j];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const double u = U[r][i];
        U[r][i] = swap ? U[r][j] : u;
        U[r][j] = swap ? u : U[r][j];
      }
    }
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int r = 0; r < 3; ++r) V[3 * r + c] = U[r][c];
}

// Mixture mean and principal axes of one molecule (weights v_i / Z,
// v_i = (pi/alpha_i)^(3/2), given as t = pi/alpha_i and its root); axes as
// columns of U, descending variance, the largest-magnitude component of the
// first two positive, U right-handed.  get(i, xyz) gives atom i's t, root and
// position.
template <class Get>
__device__ __forceinline__ void principal_frame(Get get, int n, double mu[3], double U[9]) {
  double Z = 0.0, m0 = 0.0, m1 = 0.0, m2 = 0.0;
  for (int i = 0; i < n; ++i) {
    float c[3];
    const double2 t = get(i, c);
    const double v = t.x * t.y;
    Z = fma(t.x, t.y, Z);
    m0 = fma(v, (double)c[0], m0);
    m1 = fma(v, (double)c[1], m1);
    m2 = fma(v, (double)c[2], m2);
  }
  mu[0] = m0 / Z;
  mu[1] = m1 / Z;
  mu[2] = m2 / Z;
  double C[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  for (int i = 0; i < n; ++i) {
    float at[3];
    const double2 t = get(i, at);
    const double w = t.x * t.y / Z;
    const double x[3] = {(double)at[0] - mu[0], (double)at[1] - mu[1], (double)at[2] - mu[2]};
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) C[r][c] += w * x[r] * x[c];
  }
  jacobi3(C, U);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double big = U[c];
#pragma unroll
    for (int r = 1; r < 3; ++r)
      if (fabs(U[3 * r + c]) > fabs(big)) big = U[3 * r + c];
    if (big < 0)
#pragma unroll
      for (int r = 0; r < 3; ++r) U[3 * r + c] = -U[3 * r + c];
  }
  U[2] = U[3] * U[7] - U[6] * U[4];
  U[5] = U[6] * U[1] - U[0] * U[7];
  U[8] = U[0] * U[4] - U[3] * U[1];
}

__device__ void rot_of_quat(const double q[4], double R[9]) {
  const double w = q[0], x = q[1], y = q[2], z = q[3];
  R[0] = 1 - 2 * (y * y + z * z); R[1] = 2 * (x * y - w * z); R[2] = 2 * (x * z + w * y);
  R[3] = 2 * (x * y + w * z); R[4] = 1 - 2 * (x * x + z * z); R[5] = 2 * (y * z - w * x);
  R[6] = 2 * (x * z - w * y); R[7] = 2 * (y * z + w * x); R[8] = 1 - 2 * (x * x + y * y);
}

// Unit quaternion (w >= 0) of a rotation matrix, largest-diagonal branch.
__device__ void quat_of_rot(const double R[9], double q[4]) {
  const double tr = R[0] + R[4] + R[8];
  double w, x, y, z;
  if (tr >= R[0] && tr >= R[4] && tr >= R[8]) {
    const double s = sqrt(1.0 + tr) * 2.0;
    w = 0.25 * s; x = (R[7] - R[5]) / s; y = (R[2] - R[6]) / s; z = (R[3] - R[1]) / s;
  } else if (R[0] >= R[4] && R[0] >= R[8]) {
    const double s = sqrt(1.0 + R[0] - R[4] - R[8]) * 2.0;
    w = (R[7] - R[5]) / s; x = 0.25 * s; y = (R[1] + R[3]) / s; z = (R[2] + R[6]) / s;
  } else if (R[4] >= R[8]) {
    const double s = sqrt(1.0 + R[4] - R[0] - R[8]) * 2.0;
    w = (R[2] - R[6]) / s; x = (R[1] + R[3]) / s; y = 0.25 * s; z = (R[5] + R[7]) / s;
  } else {
    const double s = sqrt(1.0 + R[8] - R[0] - R[4]) * 2.0;
    w = (R[3] - R[1]) / s; x = (R[2] + R[6]) / s; y = (R[5] + R[7]) / s; z = 0.25 * s;
  }
  const double sg = w < 0 ? -1.0 : 1.0;
  q[0] = sg * w; q[1] = sg * x; q[2] = sg * y; q[3] = sg * z;
}

// Whether a molecule is valid, as in the preparation: offsets in range, 1 to
// max_atoms atoms (here), and every alpha > 0 and every value finite.
__device__ __forceinline__ bool fo_range_ok(const MolsDev& M, int a0, int a1) {
  return a0 >= 0 && (int64_t)a1 <= M.n_atoms && a1 - a0 >= 1 && a1 - a0 <= M.max_atoms;
}
__device__ __forceinline__ bool fo_atom_ok(const float4& c) {
  return c.w > 0.0f && isfinite(c.w) && isfinite(c.x) && isfinite(c.y) && isfinite(c.z);
}
__device__ __forceinline__ float4 fo_atom(const MolsDev& M, int i) {
  return make_float4(M.xyz[3 * (int64_t)i], M.xyz[3 * (int64_t)i + 1], M.xyz[3 * (int64_t)i + 2],
                     M.alpha[i]);
}

// kLanes lanes per pair: even lanes take A's frame, odd lanes B's (lanes of one
// molecule form the same sums in atom order), and each lane takes every kLanes-th
// start.  A chain of FP64 latencies (sums, Jacobi, quaternions) while there are few
// pairs: eight lanes share a molecule's weights' roots and divisions through LDS,
// 10,000 pairs 154 -> 28 us (one lane per pair took two frames and seven starts in
// turn, with arrays in scratch memory).  Many pairs are bound by FP64 issue, and large
// molecules by that LDS: two lanes repeat nothing and read the atoms from memory.
__host__ __device__ inline size_t fo_starts_lds_bytes(int lanes, int max_atoms) {
  return lanes == 2 ? 0
                    : (size_t)2 * (kWave / lanes) * max_atoms *
                          (sizeof(double2) + 3 * sizeof(float));
}

template <int kLanes>
__global__ __launch_bounds__(kWave) void k_fo_starts(MolsDev A, MolsDev B, int n_random, uint2 key,
                                                     int* __restrict__ flag,
                                                     float* __restrict__ pose) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr bool kStaged = kLanes > 2;
  constexpr int kPairs = kWave / kLanes;
  const int lane = threadIdx.x, l = lane % kLanes, half = l & 1;
  const int max_n = A.max_atoms > B.max_atoms ? A.max_atoms : B.max_atoms;
  const int set = 2 * (lane / kLanes) + half;
  double2* t_root = reinterpret_cast<double2*>(smem) + (size_t)set * max_n;
  float* xyz = reinterpret_cast<float*>(reinterpret_cast<double2*>(smem) +
                                        (size_t)2 * kPairs * max_n) +
               (size_t)set * 3 * max_n;
  const int p = blockIdx.x * kPairs + lane / kLanes;
  const bool live = p < B.n_mols;
  const MolsDev& M = half ? B : A;
  const auto root = [](float alpha) {
    const double t = M_PI / (double)alpha;
    return make_double2(t, sqrt(t));
  };
  int a0 = 0, n = 0;
  bool bad = false;
  if (live) {
    const int m = half ? p : (A.n_mols == 1 ? 0 : p);
    a0 = M.off[m];
    const int a1 = M.off[m + 1];
    bad = !fo_range_ok(M, a0, a1);
    n = bad ? 0 : a1 - a0;
    for (int i = l >> 1; i < n; i += kLanes / 2) {
      const float4 c = fo_atom(M, a0 + i);
      if (!fo_atom_ok(c)) bad = true;
      if constexpr (kStaged) {
        t_root[i] = root(c.w);
        xyz[3 * i] = c.x;
        xyz[3 * i + 1] = c.y;
        xyz[3 * i + 2] = c.z;
      }
    }
  }
  constexpr uint64_t kMine = (1ull << kLanes) - 1;
  bad = (__ballot(bad) & (kMine << (lane & ~(kLanes - 1)))) != 0;
  wave_lds_sync();
  double mu[3] = {0, 0, 0}, U[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
  if (live && !bad) {
    const auto get = [&](int i, float (&at)[3]) {
      if constexpr (kStaged) {
        at[0] = xyz[3 * i];
        at[1] = xyz[3 * i + 1];
        at[2] = xyz[3 * i + 2];
        return t_root[i];
      } else {
        const float4 c = fo_atom(M, a0 + i);
        at[0] = c.x;
        at[1] = c.y;
        at[2] = c.z;
        return root(c.w);
      }
    };
    principal_frame(get, n, mu, U);
  }
  double muA[3], UA[9], muB[3], UB[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    UA[k] = __shfl(U[k], lane & ~1, kWave);
    UB[k] = __shfl(U[k], lane | 1, kWave);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    muA[k] = __shfl(mu[k], lane & ~1, kWave);
    muB[k] = __shfl(mu[k], lane | 1, kWave);
  }
  if (!live) return;
  const int n_starts = 5 + n_random;
  float* out = pose + (size_t)p * n_starts * 7;
  if (bad) {
    for (int c = l; c < n_starts * 7; c += kLanes) out[c] = __builtin_nanf("");
    if (l == 0) atomicOr(flag, 1);
    return;
  }
  for (int c = l; c < 7; c += kLanes) out[c] = c == 0 ? 1.f : 0.f;
  for (int s = l; s < 4 + n_random; s += kLanes) {
    double R[9];
    if (s < 4) {
      // the proper sign matrices diag(1, 1, 1), (1, -1, -1), (-1, 1, -1), (-1, -1, 1)
      const double D[3] = {s < 2 ? 1.0 : -1.0, s == 0 || s == 2 ? 1.0 : -1.0,
                           s == 0 || s == 3 ? 1.0 : -1.0};
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          double acc = 0.0;
#pragma unroll
          for (int k = 0; k < 3; ++k) acc += UA[3 * r + k] * D[k] * UB[3 * c + k];
          R[3 * r + c] = acc;
        }
    } else {
      // uniform rotation (Shoemake) from three 24-bit uniforms
      const uint4 x = philox4x32_10(make_uint4((uint32_t)(s - 4), (uint32_t)p, 0x5157A27u, 0u),
                                    key);
      const double u1 = ((double)(x.x >> 8) + 0.5) * 0x1p-24;
      const double u2 = ((double)(x.y >> 8) + 0.5) * 0x1p-24;
      const double u3 = ((double)(x.z >> 8) + 0.5) * 0x1p-24;
      const double q[4] = {sqrt(u1) * cos(2 * M_PI * u3), sqrt(1 - u1) * sin(2 * M_PI * u2),
                           sqrt(1 - u1) * cos(2 * M_PI * u2), sqrt(u1) * sin(2 * M_PI * u3)};
      rot_of_quat(q, R);
    }
    double q[4];
    quat_of_rot(R, q);
    float* o = out + 7 * (1 + s);
    for (int i = 0; i < 4; ++i) o[i] = (float)q[i];
    for (int a = 0; a < 3; ++a)
      o[4 + a] = (float)(muA[a] - (R[3 * a] * muB[0] + R[3 * a + 1] * muB[1] +
                                   R[3 * a + 2] * muB[2]));
  }
}

// ---------------------------------------------------------------------------
// First-order alignment: Adam runs inside the kernel, poses and moments stay in
// registers.
// ---------------------------------------------------------------------------
// Row layout: at most kFoRowsStarts starts (rows of 16 lanes) per
// workgroup; moved-atom arrays of the rows at a stride of s float4 with
// s = 2 (mod 8), so the four rows of a wave read their broadcast atoms from
// four disjoint groups of LDS banks.
constexpr int kFoRowsStarts = 16;
constexpr size_t kFoRowsLdsMax = 48 * 1024;
__host__ __device__ inline int fo_rows_stride(int max_b) {
  return max_b + (((2 - max_b) % 8) + 8) % 8;
}

struct FoAlignArgs {
  MolsDev A, B;
  int* flag;        // raised on invalid data
  int n_starts, n_steps;
  float lr;
  float* pose;  // [pairs][starts][7], read and written
  float* T;     // [pairs][starts]
  float* grad;  // [pairs][starts][7] at the final pose, or nullptr
  const int* order;  // optional launch order of the row layout: block x takes pair order[x]
};

// v of lane c of this lane's row of 16.
__device__ __forceinline__ float row_lane(float v, int c) {
  const int b = __builtin_bit_cast(int, v);
  int r = 0;
  switch (c) {  // a constant at every use
    case 0: r = __builtin_amdgcn_mov_dpp(b, 0x150, 0xf, 0xf, true); break;
    case 1: r = __builtin_amdgcn_mov_dpp(b, 0x151, 0xf, 0xf, true); break;
    case 2: r = __builtin_amdgcn_mov_dpp(b, 0x152, 0xf, 0xf, true); break;
    case 3: r = __builtin_amdgcn_mov_dpp(b, 0x153, 0xf, 0xf, true); break;
    case 4: r = __builtin_amdgcn_mov_dpp(b, 0x154, 0xf, 0xf, true); break;
    case 5: r = __builtin_amdgcn_mov_dpp(b, 0x155, 0xf, 0xf, true); break;
    default: r = __builtin_amdgcn_mov_dpp(b, 0x156, 0xf, 0xf, true); break;  // row_newbcast:6
  }
  return __builtin_bit_cast(float, r);
}

// Both molecules into LDS (x, y, z, alpha) by the threads tid of n; whether
// the pair is valid, the same in every thread (any: an OR over the group,
// after which the staged atoms are visible to it if it is a barrier).
template <class Any>
__device__ __forceinline__ bool fo_stage(const FoAlignArgs& a, bool ok, float4* sA, int a0, int na,
                                         float4* sB, int b0, int nb, int tid, int n, Any any) {
  bool bad = !ok;  // then the counts are not trusted and nothing is read
  if (ok) {
    for (int i = tid; i < na; i += n) {
      const float4 c = fo_atom(a.A, a0 + i);
      if (!fo_atom_ok(c)) bad = true;
      sA[i] = c;
    }
    for (int j = tid; j < nb; j += n) {
      const float4 c = fo_atom(a.B, b0 + j);
      if (!fo_atom_ok(c)) bad = true;
      sB[j] = c;
    }
  }
  return !any(bad);
}

// (pi/(a_i+a_j))^(3/2) = pi^(3/2) rs^3 and k_ij = a_i a_j rs^2 of a pair of
// widths, from rs = 1/sqrt(a_i + a_j): kk = -log2(e) k_ij, pre = the
// prefactor, f2 = 2 k_ij.
__device__ __forceinline__ void fo_consts_rs(float ai, float aj, float rs, float& kk, float& pre,
                                             float& f2) {
  const float ir = rs * rs;
  const float k = ai * aj * ir;
  kk = -1.44269504088896f * k;
  pre = 5.56832799683170785f * ir * rs;
  f2 = 2.f * k;
}
__device__ __forceinline__ void fo_consts(float ai, float aj, float& kk, float& pre, float& f2) {
  fo_consts_rs(ai, aj, __builtin_amdgcn_rsqf(ai + aj), kk, pre, f2);
}

struct FoAcc {
  float O = 0.f, gx = 0.f, gy = 0.f, gz = 0.f, rx = 0.f, ry = 0.f, rz = 0.f;
  // the term pre exp of c''_j at distance d from c_i: O, dO/dc''_j, torque
  __device__ __forceinline__ void add(const float3& d, const float4& cj, float e, float pre,
                                      float f2) {
    O = fmaf(pre, e, O);
    const float f = f2 * (pre * e);
    const float fx = f * d.x, fy = f * d.y, fz = f * d.z;
    gx = fmaf(f, d.x, gx); gy = fmaf(f, d.y, gy); gz = fmaf(f, d.z, gz);
    rx = fmaf(cj.y, fz, fmaf(-cj.z, fy, rx));
    ry = fmaf(cj.z, fx, fmaf(-cj.x, fz, ry));
    rz = fmaf(cj.x, fy, fmaf(-cj.y, fx, rz));
  }
};

// One pass over the N_A x N_B atom pairs spread over the lanes (pair p = lane
// + 64 t is lane's term t; its row i and column j are stepped incrementally),
// for S poses of B at once: per pose the lane's part of O, dO/dt and the torque
// sum c''_j x f, its terms added in turn.  The pose-independent factors of a
// pair come from its widths (one rsqrt) and serve all S poses.  U terms go
// together; the last few are masked (prefactor 0: their terms add exactly 0).
template <int S, int U>
__device__ __forceinline__ void fo_pass(const float4* sA, int na, const float4* sM, int stride,
                                        int nb, FoAcc (&acc)[S]) {
  const int lane = threadIdx.x & (kWave - 1);
  const int di = kWave / nb, dj = kWave % nb;
  const int n = na * nb, terms = (n + kWave - 1) / kWave, whole = n / kWave / U * U;
  int i = lane / nb, j = lane % nb;
  const auto group = [&](int t, auto masked) {
    float4 ci[U], cj[U][S];
    float rs[U], kk[U], pre[U], f2[U], e[U * S];
    float3 d[U][S];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ci[u] = sA[decltype(masked)::value ? min(i, na - 1) : i];
#pragma unroll
      for (int s = 0; s < S; ++s) cj[u][s] = sM[s * stride + j];
      rs[u] = ci[u].w + cj[u][0].w;
      i += di;
      j += dj;
      if (j >= nb) {
        j -= nb;
        ++i;
      }
    }
    trans_group<U>([&](int u) { rs[u] = __builtin_amdgcn_rsqf(rs[u]); });
#pragma unroll
    for (int u = 0; u < U; ++u) {
      fo_consts_rs(ci[u].w, cj[u][0].w, rs[u], kk[u], pre[u], f2[u]);
      if constexpr (decltype(masked)::value)
        if (lane + kWave * (t + u) >= n) pre[u] = 0.f;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float dx = ci[u].x - cj[u][s].x, dy = ci[u].y - cj[u][s].y,
                    dz = ci[u].z - cj[u][s].z;
        d[u][s] = make_float3(dx, dy, dz);
        e[u * S + s] = kk[u] * fmaf(dx, dx, fmaf(dy, dy, dz * dz));
      }
    }
    trans_group<U * S>([&](int x) { e[x] = __builtin_amdgcn_exp2f(e[x]); });
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < S; ++s) acc[s].add(d[u][s], cj[u][s], e[u * S + s], pre[u], f2[u]);
  };
  int t = 0;
  for (; t < whole; t += U) group(t, std::false_type{});
  for (; t < terms; t += U) group(t, std::true_type{});
}

// sum_ij K_ij of a molecule with itself (pose invariant), over all lanes.
__device__ __forceinline__ float fo_self(const float4* s, int n) {
  const int lane = threadIdx.x & (kWave - 1);
  const int di = kWave / n, dj = kWave % n;
  int i = lane / n, j = lane % n;
  float acc = 0.f;
  for (; i < n;) {
    const float4 ci = s[i], cj = s[j];
    const float sa = ci.w + cj.w;
    const float ir = __builtin_amdgcn_rcpf(sa);
    const float dx = ci.x - cj.x, dy = ci.y - cj.y, dz = ci.z - cj.z;
    const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    const float t = 3.14159265358979f * ir;
    acc += t * __builtin_amdgcn_sqrtf(t) *
           __builtin_amdgcn_exp2f(-1.44269504088896f * ci.w * cj.w * ir * d2);
    i += di;
    j += dj;
    if (j >= n) {
      j -= n;
      ++i;
    }
  }
  return wave_sum_dpp(acc);
}

// One wave per pair and S of its starts, for molecules that the row layout below
// does not take.  VALU issue bounds it: per atom pair and pose 22 instructions and
// an exponential, shared by the poses 8 (widths), a reciprocal root, 8 (indices)
// and A's LDS read.  8,000 pairs of 75 x 50-100 atoms, 8 starts, 50 steps: 16.1 ms
// with one start per wave, a lane's first terms' factors kept in registers and one
// term at a time; 15.4 ms with the transcendentals of two terms grouped, 13.4 ms
// with two starts and 12.3 ms with four; 100 pairs 0.79 -> 0.62 ms.  All lanes walk the atom pairs for the
// S poses together (fo_pass); the steps between two passes are taken by S rows of
// 64/S lanes, each for its own start: every lane of a row holds its pose, and
// Adam's component c with its moments sits in lane c of the row.
template <int S, int U>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4)))
void k_fo_align(FoAlignArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kRow = kWave / S;
  const int lane = threadIdx.x, lr = lane % kRow, row = lane / kRow;
  const int groups = (a.n_starts + S - 1) / S;
  const int pair = blockIdx.x / groups;
  const int s_raw = (int)(blockIdx.x % groups) * S + row;
  const bool live = s_raw < a.n_starts;
  // spare rows repeat the last start
  const size_t item = (size_t)pair * a.n_starts + (live ? s_raw : a.n_starts - 1);
  const int ma = a.A.n_mols == 1 ? 0 : pair;
  const int a0 = a.A.off[ma], a1 = a.A.off[ma + 1], na = a1 - a0;
  const int b0 = a.B.off[pair], b_end = a.B.off[pair + 1], nb = b_end - b0;
  const int stride = a.B.max_atoms;
  float4* sA = reinterpret_cast<float4*>(smem);  // [max_a] x, y, z, alpha
  float4* sB = sA + a.A.max_atoms;               // [max_b] B as given
  float4* sM = sB + stride;                      // [S][max_b] B moved
  const bool ok = fo_range_ok(a.A, a0, a1) && fo_range_ok(a.B, b0, b_end);
  if (!fo_stage(a, ok, sA, a0, na, sB, b0, nb, lane, kWave, [](bool b) { return __any(b); })) {
    if (live && lr == 0) {
      a.T[item] = __builtin_nanf("");
      if (a.grad)
        for (int c = 0; c < 7; ++c) a.grad[item * 7 + c] = __builtin_nanf("");
      atomicOr(a.flag, 1);
    }
    return;
  }
  wave_lds_sync();
  const float S0 = fo_self(sA, na) + fo_self(sB, nb);  // O_AA + O_BB
  float x[7];
  float* ps = a.pose + item * 7;
#pragma unroll
  for (int c = 0; c < 7; ++c) x[c] = ps[c];
  const int mine = lr < 7 ? lr : 6;
  float m_l = 0.f, v_l = 0.f;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  float b1t = 1.f, b2t = 1.f;  // b1^t, b2^t as running products
  float T = 0.f, g[7];
  for (int it = 0; it <= a.n_steps; ++it) {
    // move B by the current pose
    const float n2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
    const float in = rsqrtf(n2);
    const float qw = x[0] * in, qx = x[1] * in, qy = x[2] * in, qz = x[3] * in;
    const float R0 = 1.f - 2.f * (qy * qy + qz * qz), R1 = 2.f * (qx * qy - qw * qz),
                R2 = 2.f * (qx * qz + qw * qy), R3 = 2.f * (qx * qy + qw * qz),
                R4 = 1.f - 2.f * (qx * qx + qz * qz), R5 = 2.f * (qy * qz - qw * qx),
                R6 = 2.f * (qx * qz - qw * qy), R7 = 2.f * (qy * qz + qw * qx),
                R8 = 1.f - 2.f * (qx * qx + qy * qy);
    for (int j = lr; j < nb; j += kRow) {
      const float4 c = sB[j];
      sM[row * stride + j] =
          make_float4(fmaf(R0, c.x, fmaf(R1, c.y, fmaf(R2, c.z, x[4]))),
                      fmaf(R3, c.x, fmaf(R4, c.y, fmaf(R5, c.z, x[5]))),
                      fmaf(R6, c.x, fmaf(R7, c.y, fmaf(R8, c.z, x[6]))), c.w);
    }
    wave_lds_sync();
    FoAcc acc[S];
    fo_pass<S, U>(sA, na, sM, stride, nb, acc);
    wave_lds_sync();  // sM is rewritten next step
    float r[7];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const float w[7] = {wave_sum_dpp(acc[s].O),  wave_sum_dpp(acc[s].gx),
                          wave_sum_dpp(acc[s].gy), wave_sum_dpp(acc[s].gz),
                          wave_sum_dpp(acc[s].rx), wave_sum_dpp(acc[s].ry),
                          wave_sum_dpp(acc[s].rz)};
#pragma unroll
      for (int c = 0; c < 7; ++c) r[c] = s == 0 || row == s ? w[c] : r[c];
    }
    // torque about B's origin: sum (c''_j - t) x f = sum c''_j x f - t x sum f
    r[4] -= x[5] * r[3] - x[6] * r[2];
    r[5] -= x[6] * r[1] - x[4] * r[3];
    r[6] -= x[4] * r[2] - x[5] * r[1];
    const float D = S0 - r[0];
    const float iD = __builtin_amdgcn_rcpf(D);
    const float dTdO = S0 * iD * iD;
    const float gth[3] = {dTdO * r[4], dTdO * r[5], dTdO * r[6]};
    // dT/dq = (2/|q|) [ -v.g ; w g - v x g ]
    const float vdg = qx * gth[0] + qy * gth[1] + qz * gth[2];
    g[0] = 2.f * in * (-vdg);
    g[1] = 2.f * in * (qw * gth[0] - (qy * gth[2] - qz * gth[1]));
    g[2] = 2.f * in * (qw * gth[1] - (qz * gth[0] - qx * gth[2]));
    g[3] = 2.f * in * (qw * gth[2] - (qx * gth[1] - qy * gth[0]));
    g[4] = dTdO * r[1];
    g[5] = dTdO * r[2];
    g[6] = dTdO * r[3];
    if (it == a.n_steps) {
      T = r[0] / D;  // only the final pose's T is returned
      break;
    }
    // Adam on -T (bias-corrected moments, betas 0.9 / 0.999), q renormalised;
    // reciprocals by the hardware (a step of length ~lr tolerates 1 ulp).
    // Lane c < 7 of the row updates component c; the row reads the new pose.
    b1t *= b1;
    b2t *= b2;
    const float ic1 = __builtin_amdgcn_rcpf(1.f - b1t), ic2 = __builtin_amdgcn_rcpf(1.f - b2t);
    float g_l = g[0], x_l = x[0];
#pragma unroll
    for (int c = 1; c < 7; ++c) {
      g_l = mine == c ? g[c] : g_l;
      x_l = mine == c ? x[c] : x_l;
    }
    const float gc = -g_l;
    m_l = fmaf(b1, m_l, (1.f - b1) * gc);
    v_l = fmaf(b2, v_l, (1.f - b2) * gc * gc);
    const float den = __builtin_amdgcn_sqrtf(v_l * ic2) + eps;
    const float xn_l = x_l - a.lr * (m_l * ic1) * __builtin_amdgcn_rcpf(den);
    float xn[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) xn[c] = __shfl(xn_l, lane - lr + c, kWave);
    const float inv = rsqrtf(xn[0] * xn[0] + xn[1] * xn[1] + xn[2] * xn[2] + xn[3] * xn[3]);
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = xn[c] * inv;
#pragma unroll
    for (int c = 4; c < 7; ++c) x[c] = xn[c];
  }
  if (live && lr == 0) {
#pragma unroll
    for (int c = 0; c < 7; ++c) ps[c] = x[c];
    a.T[item] = T;
    if (a.grad)
#pragma unroll
      for (int c = 0; c < 7; ++c) a.grad[item * 7 + c] = g[c];
  }
}

// ---------------------------------------------------------------------------
// First-order alignment, row layout: one workgroup per pair and up to 16
// starts, one start per 16-lane row of a wave, so the per-step work that
// does not scale with the atom pairs (rotation, reductions, Adam) is shared
// by four starts per wave instruction.  Lane l of a row owns A's atoms
// i = l + 16 r (r < RA; rows past N_A are padding whose terms add exactly
// 0) and walks all of B's moved atoms, read as LDS
// broadcasts.  The pose-independent constants of every atom pair,
// kk = -log2(e) k_ij and lq = log2((pi/(a_i+a_j))^(3/2)) + kk |c_i|^2 (A's
// atoms do not move), sit in an LDS table filled once per workgroup (padding
// rows: kk = 0, lq = -inf, so K = 0).  Per term, with d = c_i - c''_j and
// |d|^2 = |c_i|^2 + |c''_j|^2 + (-2 c_i) . c''_j:
//   K = exp2(kk (|c''_j|^2 + (-2 c_i) . c''_j) + lq)   (|c''_j|^2 stored
//       with the moved atom)
// (FP32 emulation on drug-sized molecules at random poses against FP64:
// relative error of O at most 7.7e-7, of its gradient 2.2e-6 (1.0e-6 and
// 3.3e-6 with |c_i|^2 added per term); 10 VALU + exp per term.)
// and the lane keeps O_i = sum_j K, W_i = sum_j kk K, P_i = sum_j kk K c''_j,
// so that F_i = sum_j kk K d = c_i W_i - P_i.  Since dO/dc''_j is parallel to d,
// c''_j x (s d) = c_i x (s d), so the torque about B's origin is
// sum_i c_i x F_i less t x sum F, formed once per lane instead of per term;
// dO/dc''_j = 2 k K d = -2 ln(2) kk K d scales F once at the end.
// Every lane of a row holds the same pose and gradient (row sums leave
// identical bits in all 16 lanes); Adam's seven components are updated one
// per lane (lanes 0-6 of the row, with their moments) and read back by the
// whole row, instead of all seven in every lane.
// ---------------------------------------------------------------------------
// VALU issue bounds it, at two thirds of its LDS bandwidth (a moved atom and RA
// constants per RA terms): of 952 instructions per wave and step (30 x 30 atoms)
// 657 are terms.  The terms of a few of B's atoms go together, their exponentials
// in one prioritised group (trans_group), while the next ones' data are read
// from LDS: 10,000 pairs x 8 starts x 50 steps (2 rows) 1.45 ms with four atoms
// unrolled, 1.41 with the group, 1.35 with the data read ahead.  Atoms per group:
// as many as the registers of four waves per SIMD hold twice (2 rows: two atoms
// 1.42 ms, three 1.35, four 1.35; 4 rows, 4,000 pairs of 64 x 20-64 atoms: one
// 2.23, two 2.16, four spilled 2.82, none read ahead 2.36; 1 row, 8,000 of 16 x
// 10-50: two 0.77, three 0.71, six 0.73, none read ahead 0.77).  More waves do
// not help: with the constants tabulated per distinct width of B, a third of the
// LDS, six waves per SIMD measured 3 % more.
constexpr int fo_term_atoms(int ra) { return ra == 4 ? 2 : 3; }
template <int N, int RA>
struct FoTermGroup {
  static constexpr int V = N;
  float4 cj[V];        // moved atoms
  float2 kp[V * RA];   // their constants with the lane's atoms of A
};
template <int RA>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
void k_fo_align_rows(FoAlignArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int sBad[kFoRowsStarts / 4];  // per wave: an invalid atom
  constexpr int RA16 = RA * 16;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int l16 = lane & 15, row = lane >> 4;
  const int pair = a.order ? a.order[blockIdx.x] : xcd_chunk(blockIdx.x, gridDim.x);
  const int s_raw = blockIdx.y * kFoRowsStarts + wave * 4 + row;
  const bool live = s_raw < a.n_starts;
  const int s = live ? s_raw : a.n_starts - 1;  // spare rows repeat the last start
  const size_t item = (size_t)pair * a.n_starts + s;
  const int ma = a.A.n_mols == 1 ? 0 : pair;
  const int a0 = a.A.off[ma], a1 = a.A.off[ma + 1], na = a1 - a0;
  const int b0 = a.B.off[pair], b_end = a.B.off[pair + 1], nb = b_end - b0;
  const int stride = fo_rows_stride(a.B.max_atoms);
  const int n_rows = (int)(blockDim.x / 16);
  float4* sA = reinterpret_cast<float4*>(smem);  // [max_a] x, y, z, alpha
  float4* sB = sA + a.A.max_atoms;               // [max_b] B as given
  float4* sM = sB + a.B.max_atoms;               // [rows][stride] B moved, per start
  float2* tab = reinterpret_cast<float2*>(sM + (size_t)n_rows * stride);  // [max_b][RA16]
  const bool ok = fo_range_ok(a.A, a0, a1) && fo_range_ok(a.B, b0, b_end);
  // one barrier: __syncthreads_or takes several, a tenth of a call of few steps
  const auto any = [&](bool b) {
    const int mine = __any(b) ? 1 : 0;
    if (lane == 0) sBad[wave] = mine;
    __syncthreads();
    int all = sBad[0];
    for (int w = 1; w < n_rows / 4; ++w) all |= sBad[w];
    return all != 0;
  };
  if (!fo_stage(a, ok, sA, a0, na, sB, b0, nb, tid, blockDim.x, any)) {
    if (live && l16 == 0) {
      a.T[item] = __builtin_nanf("");
      if (a.grad)
        for (int c = 0; c < 7; ++c) a.grad[item * 7 + c] = __builtin_nanf("");
      atomicOr(a.flag, 1);
    }
    return;
  }
  for (int e = tid; e < nb * RA16; e += blockDim.x) {
    const int j = e / RA16, i = e % RA16;
    float kk = 0.f, pre = 0.f, f2, lq = -INFINITY;
    if (i < na) {
      const float4 c = sA[i];
      fo_consts(c.w, sB[j].w, kk, pre, f2);
      lq = fmaf(kk, norm2(c.x, c.y, c.z), log2f(pre));
    }
    tab[e] = make_float2(kk, lq);
  }
  __syncthreads();
  const float S = fo_self(sA, na) + fo_self(sB, nb);  // O_AA + O_BB
  float cx[RA], cy[RA], cz[RA];
#pragma unroll
  for (int r = 0; r < RA; ++r) {
    const int i = l16 + 16 * r;
    const float4 c = i < na ? sA[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    cx[r] = c.x;
    cy[r] = c.y;
    cz[r] = c.z;
  }
  float4* mine = sM + (size_t)(wave * 4 + row) * stride;
  const float2* trow = tab + l16;
  // the pose in every lane of the row; its component cA = min(l16, 6) and
  // Adam's moments of it in lane l16 (lanes past 6 repeat component 6)
  float x[7];
  float* ps = a.pose + item * 7;
#pragma unroll
  for (int c = 0; c < 7; ++c) x[c] = ps[c];
  const int cA = l16 < 7 ? l16 : 6;
  float xA = ps[cA], mA = 0.f, vA = 0.f;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  float b1t = 1.f, b2t = 1.f;
  float T = 0.f, g[7];
  for (int it = 0; it <= a.n_steps; ++it) {
    const float n2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
    const float in = rsqrtf(n2);
    const float qw = x[0] * in, qx = x[1] * in, qy = x[2] * in, qz = x[3] * in;
    const float R0 = 1.f - 2.f * (qy * qy + qz * qz), R1 = 2.f * (qx * qy - qw * qz),
                R2 = 2.f * (qx * qz + qw * qy), R3 = 2.f * (qx * qy + qw * qz),
                R4 = 1.f - 2.f * (qx * qx + qz * qz), R5 = 2.f * (qy * qz - qw * qx),
                R6 = 2.f * (qx * qz - qw * qy), R7 = 2.f * (qy * qz + qw * qx),
                R8 = 1.f - 2.f * (qx * qx + qy * qy);
    for (int j = l16; j < nb; j += 16) {
      const float4 c = sB[j];
      const float mx = fmaf(R0, c.x, fmaf(R1, c.y, fmaf(R2, c.z, x[4])));
      const float my = fmaf(R3, c.x, fmaf(R4, c.y, fmaf(R5, c.z, x[5])));
      const float mz = fmaf(R6, c.x, fmaf(R7, c.y, fmaf(R8, c.z, x[6])));
      mine[j] = make_float4(mx, my, mz, norm2(mx, my, mz));
    }
    wave_lds_sync();
    float O[RA], W[RA], Px[RA], Py[RA], Pz[RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) O[r] = W[r] = Px[r] = Py[r] = Pz[r] = 0.f;
    // a few of B's atoms at a time, the next ones read from LDS meanwhile
    const auto load = [&](int j, auto& g) {
#pragma unroll
      for (int u = 0; u < g.V; ++u) {
        g.cj[u] = mine[j + u];
#pragma unroll
        for (int r = 0; r < RA; ++r) g.kp[u * RA + r] = trow[(j + u) * RA16 + 16 * r];
      }
    };
    const auto terms = [&](const auto& g) {
      constexpr int V = std::remove_reference_t<decltype(g)>::V;
      float K[V * RA];
#pragma unroll
      for (int u = 0; u < V; ++u)
#pragma unroll
        for (int r = 0; r < RA; ++r) {
          const float e = fmaf(-2.f * cx[r], g.cj[u].x,
                               fmaf(-2.f * cy[r], g.cj[u].y,
                                    fmaf(-2.f * cz[r], g.cj[u].z, g.cj[u].w)));
          K[u * RA + r] = fmaf(g.kp[u * RA + r].x, e, g.kp[u * RA + r].y);
        }
      trans_group<V * RA>([&](int i) { K[i] = __builtin_amdgcn_exp2f(K[i]); });
#pragma unroll
      for (int u = 0; u < V; ++u)
#pragma unroll
        for (int r = 0; r < RA; ++r) {
          O[r] += K[u * RA + r];
          const float fs = g.kp[u * RA + r].x * K[u * RA + r];
          W[r] += fs;
          Px[r] = fmaf(fs, g.cj[u].x, Px[r]);
          Py[r] = fmaf(fs, g.cj[u].y, Py[r]);
          Pz[r] = fmaf(fs, g.cj[u].z, Pz[r]);
        }
    };
    constexpr int V = fo_term_atoms(RA);
    int j = 0;
    const int whole = nb / V * V;
    if (whole > 0) {
      FoTermGroup<V, RA> g0, g1;
      load(0, g0);
      for (; j + 2 * V <= whole; j += 2 * V) {
        load(j + V, g1);
        terms(g0);
        load(min(j + 2 * V, whole - V), g0);  // the last time read again, unused
        terms(g1);
      }
      if (j < whole) {
        terms(g0);
        j = whole;
      }
    }
    for (; j < nb; ++j) {
      FoTermGroup<1, RA> g;
      load(j, g);
      terms(g);
    }
    wave_lds_sync();  // this start's moved atoms are rewritten next step
    float Fx[RA], Fy[RA], Fz[RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) {
      Fx[r] = fmaf(cx[r], W[r], -Px[r]);
      Fy[r] = fmaf(cy[r], W[r], -Py[r]);
      Fz[r] = fmaf(cz[r], W[r], -Pz[r]);
    }
    float o = O[0], fx = Fx[0], fy = Fy[0], fz = Fz[0];
    float tx = cy[0] * Fz[0] - cz[0] * Fy[0], ty = cz[0] * Fx[0] - cx[0] * Fz[0],
          tz = cx[0] * Fy[0] - cy[0] * Fx[0];
#pragma unroll
    for (int r = 1; r < RA; ++r) {
      o += O[r];
      fx += Fx[r];
      fy += Fy[r];
      fz += Fz[r];
      tx += cy[r] * Fz[r] - cz[r] * Fy[r];
      ty += cz[r] * Fx[r] - cx[r] * Fz[r];
      tz += cx[r] * Fy[r] - cy[r] * Fx[r];
    }
    const float sc = -1.38629436111989061f;  // -2 ln 2
    float r7[7];
    r7[0] = row_sum16(o);
    r7[1] = sc * row_sum16(fx);
    r7[2] = sc * row_sum16(fy);
    r7[3] = sc * row_sum16(fz);
    // torque about B's origin: sum c_i x F_i - t x sum F
    r7[4] = sc * row_sum16(tx) - (x[5] * r7[3] - x[6] * r7[2]);
    r7[5] = sc * row_sum16(ty) - (x[6] * r7[1] - x[4] * r7[3]);
    r7[6] = sc * row_sum16(tz) - (x[4] * r7[2] - x[5] * r7[1]);
    const float D = S - r7[0];
    const float iD = __builtin_amdgcn_rcpf(D);
    const float dTdO = S * iD * iD;
    const float gth[3] = {dTdO * r7[4], dTdO * r7[5], dTdO * r7[6]};
    const float vdg = qx * gth[0] + qy * gth[1] + qz * gth[2];
    g[0] = 2.f * in * (-vdg);
    g[1] = 2.f * in * (qw * gth[0] - (qy * gth[2] - qz * gth[1]));
    g[2] = 2.f * in * (qw * gth[1] - (qz * gth[0] - qx * gth[2]));
    g[3] = 2.f * in * (qw * gth[2] - (qx * gth[1] - qy * gth[0]));
    g[4] = dTdO * r7[1];
    g[5] = dTdO * r7[2];
    g[6] = dTdO * r7[3];
    if (it == a.n_steps) {
      T = r7[0] / D;  // only the final pose's T is returned
      break;
    }
    // Adam on -T, k_fo_align's arithmetic: lane l16 < 7
    // of the row updates component l16, then the row reads the seven new
    // components back from those lanes
    b1t *= b1;
    b2t *= b2;
    const float ic1 = __builtin_amdgcn_rcpf(1.f - b1t), ic2 = __builtin_amdgcn_rcpf(1.f - b2t);
    float gA = g[0];
#pragma unroll
    for (int c = 1; c < 7; ++c) gA = cA == c ? g[c] : gA;
    {
      const float gc = -gA;
      mA = fmaf(b1, mA, (1.f - b1) * gc);
      vA = fmaf(b2, vA, (1.f - b2) * gc * gc);
      const float den = __builtin_amdgcn_sqrtf(vA * ic2) + eps;
      xA = xA - a.lr * (mA * ic1) * __builtin_amdgcn_rcpf(den);
    }
    float xn[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) xn[c] = row_lane(xA, c);
    const float inv = rsqrtf(xn[0] * xn[0] + xn[1] * xn[1] + xn[2] * xn[2] + xn[3] * xn[3]);
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = xn[c] * inv;
#pragma unroll
    for (int c = 4; c < 7; ++c) x[c] = xn[c];
    xA = cA < 4 ? xA * inv : xA;
  }
  if (live && l16 == 0) {
#pragma unroll
    for (int c = 0; c < 7; ++c) ps[c] = x[c];
    a.T[item] = T;
    if (a.grad)
#pragma unroll
      for (int c = 0; c < 7; ++c) a.grad[item * 7 + c] = g[c];
  }
}

// Best start per pair (largest T; lowest index on ties; NaN never wins):
// its pose and T.
__global__ void k_best_pose(const float* __restrict__ T, const float* __restrict__ pose,
                            int n_pairs, int n_starts, float* __restrict__ best_pose,
                            float* __restrict__ best_T) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n_pairs) return;
  int b = 0;
  float bv = -INFINITY;
  for (int s = 0; s < n_starts; ++s) {
    const float t = T[(size_t)p * n_starts + s];
    if (t > bv) {
      bv = t;
      b = s;
    }
  }
  const float* src = pose + ((size_t)p * n_starts + b) * 7;
  for (int c = 0; c < 7; ++c) best_pose[(size_t)p * 7 + c] = src[c];
  if (best_T) best_T[p] = T[(size_t)p * n_starts + b];
}

// Conformer ensembles: the largest T of each group of consecutive entries
// (max over conformers); lowest index on ties, NaN never wins (a group of
// NaN gives NaN and index -1).
__global__ void k_group_max(const float* __restrict__ T, int64_t n_T, const int* __restrict__ goff,
                            int n_groups, float* __restrict__ best_T, int* __restrict__ best_idx,
                            int* __restrict__ flag) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n_groups) return;
  int b = -1;
  float bv = -INFINITY;
  const int e0 = goff[g], e1 = goff[g + 1];
  if (e0 < 0 || e1 > n_T || e1 < e0) {
    // a group outside T (or reversed) reads nothing: NaN, -1, data error
    best_T[g] = __builtin_nanf("");
    if (best_idx) best_idx[g] = -1;
    atomicOr(flag, 1);
    return;
  }
  for (int e = e0; e < e1; ++e) {
    const float t = T[e];
    if (t > bv || (b < 0 && t == bv)) {
      bv = t;
      b = e;
    }
  }
  best_T[g] = b < 0 ? __builtin_nanf("") : bv;
  if (best_idx) best_idx[g] = b;
}

// Moved coordinates xyz_out = R(q/|q|) xyz + t, one wave per molecule.
__global__ __launch_bounds__(64) void k_apply_pose(MolsDev M, const float* __restrict__ pose,
                                                   float* __restrict__ out) {
  const int mol = blockIdx.x;
  if (mol >= M.n_mols) return;
  const float* x = pose + (size_t)mol * 7;
  const float in = rsqrtf(x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3]);
  const float qw = x[0] * in, qx = x[1] * in, qy = x[2] * in, qz = x[3] * in;
  const float R0 = 1.f - 2.f * (qy * qy + qz * qz), R1 = 2.f * (qx * qy - qw * qz),
              R2 = 2.f * (qx * qz + qw * qy), R3 = 2.f * (qx * qy + qw * qz),
              R4 = 1.f - 2.f * (qx * qx + qz * qz), R5 = 2.f * (qy * qz - qw * qx),
              R6 = 2.f * (qx * qz - qw * qy), R7 = 2.f * (qy * qz + qw * qx),
              R8 = 1.f - 2.f * (qx * qx + qy * qy);
  const int a0 = M.off[mol], a1 = M.off[mol + 1];
  for (int i = a0 + (int)threadIdx.x; i < a1; i += kWave) {
    const float cx = M.xyz[3 * i], cy = M.xyz[3 * i + 1], cz = M.xyz[3 * i + 2];
    out[3 * i] = fmaf(R0, cx, fmaf(R1, cy, fmaf(R2, cz, x[4])));
    out[3 * i + 1] = fmaf(R3, cx, fmaf(R4, cy, fmaf(R5, cz, x[5])));
    out[3 * i + 2] = fmaf(R6, cx, fmaf(R7, cy, fmaf(R8, cz, x[6])));
  }
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
template <int kLanes>
static hipError_t launch_fo_starts_t(const MolsDev& A, const MolsDev& B, int n_random, uint2 key,
                                     int* flag, float* pose, hipStream_t st) {
  const int64_t blocks = ((int64_t)B.n_mols * kLanes + kWave - 1) / kWave;
  hipLaunchKernelGGL((k_fo_starts<kLanes>), dim3((unsigned)blocks), dim3(kWave),
                     fo_starts_lds_bytes(kLanes, std::max(A.max_atoms, B.max_atoms)), st, A, B,
                     n_random, key, flag, pose);
  return hipGetLastError();
}

hipError_t launch_fo_starts(const MolsDev& A, const MolsDev& B, int n_random, uint2 key,
                            int* flag, float* pose, int n_cu, hipStream_t st) {
  // eight : two lanes, us, 3 random starts: 10-50 atoms, 10,000 pairs 32 : 45, 20,000 53 :
  // 47, 10^6 1,645 : 1,180; 150-256 atoms (one wave's LDS per compute unit), 2,000 67 :
  // 166, 10,000 329 : 276, 100,000 3,560 : 950
  const bool large = std::max(A.max_atoms, B.max_atoms) > 128;
  if (B.n_mols > (large ? 24 : 48) * n_cu)
    return launch_fo_starts_t<2>(A, B, n_random, key, flag, pose, st);
  return launch_fo_starts_t<8>(A, B, n_random, key, flag, pose, st);
}

// For s starts per wave.
static size_t fo_align_lds_bytes(int max_a, int max_b, int s) {
  return (size_t)(max_a + (1 + s) * max_b) * sizeof(float4);
}
size_t fo_align_lds_bytes(int max_a, int max_b) { return fo_align_lds_bytes(max_a, max_b, 2); }

// Row-layout launch shape: rows (starts) per workgroup and its LDS bytes, or
// 0 when the row kernel does not apply (A over 64 atoms, LDS beyond
// kFoRowsLdsMax, or more start blocks than a grid's y extent) and the
// k_fo_align runs instead.
static int fo_rows_per_block(int n_starts) {
  return n_starts >= kFoRowsStarts ? kFoRowsStarts : ((n_starts + 3) / 4) * 4;
}
static size_t fo_rows_lds_bytes(int max_a, int max_b, int n_starts) {
  const int ra = (max_a + 15) / 16;
  if (ra > 4 || (n_starts + kFoRowsStarts - 1) / kFoRowsStarts > 65535) return 0;
  const size_t bytes = (size_t)(max_a + max_b) * sizeof(float4) +
                       (size_t)fo_rows_per_block(n_starts) * fo_rows_stride(max_b) *
                           sizeof(float4) +
                       (size_t)ra * 16 * max_b * sizeof(float2);
  return bytes <= kFoRowsLdsMax ? bytes : 0;
}

bool fo_align_pair_major(int max_a, int max_b, int n_starts) {
  return fo_rows_lds_bytes(max_a, max_b, n_starts) > 0;
}

template <int RA>
static void launch_fo_rows_t(const FoAlignArgs& a, size_t lds, hipStream_t st) {
  const int rows = fo_rows_per_block(a.n_starts);
  const int blocks_y = (a.n_starts + kFoRowsStarts - 1) / kFoRowsStarts;
  hipLaunchKernelGGL((k_fo_align_rows<RA>), dim3((unsigned)a.B.n_mols, (unsigned)blocks_y),
                     dim3(rows / 4 * kWave), lds, st, a);
}

template <int S, int U>
static void launch_fo_align_t(const FoAlignArgs& a, hipStream_t st) {
  const int64_t blocks = (int64_t)a.B.n_mols * ((a.n_starts + S - 1) / S);
  hipLaunchKernelGGL((k_fo_align<S, U>), dim3((unsigned)blocks), dim3(kWave),
                     fo_align_lds_bytes(a.A.max_atoms, a.B.max_atoms, S), st, a);
}

hipError_t launch_fo_align(const MolsDev& A, const MolsDev& B, int n_starts, int n_steps,
                           float lr, int* flag, float* pose, float* T, float* grad,
                           hipStream_t st, const int* order, int n_cu) {
  FoAlignArgs a{A, B, flag, n_starts, n_steps, lr, pose, T, grad, nullptr};
  const size_t lds = fo_rows_lds_bytes(A.max_atoms, B.max_atoms, n_starts);
  if (lds > 0) {
    a.order = order;
    switch ((A.max_atoms + 15) / 16) {
      case 1: launch_fo_rows_t<1>(a, lds, st); break;
      case 2: launch_fo_rows_t<2>(a, lds, st); break;
      case 3: launch_fo_rows_t<3>(a, lds, st); break;
      default: launch_fo_rows_t<4>(a, lds, st); break;
    }
    return hipGetLastError();
  }
  // Four starts per wave once two would give every SIMD more than one wave,
  // while sixteen waves' LDS fit a compute unit (B up to about 100 atoms); two
  // once one would give three.  20 steps, 75 x 50-100 atoms, 8 starts, one : two
  // : four, ms: 384 pairs 0.47 : 0.48 : 0.65, 512 0.58 : 0.48 : 0.65, 768 0.80 :
  // 0.69 : 0.78, 1,024 1.04 : 0.86 : 0.79, 6,000 5.1 : 4.2 : 3.9; 4,000 of 256 x
  // 200-256 atoms 37.9 : 31.9 : 34.6.
  const int64_t items = (int64_t)B.n_mols * n_starts;
  if (items > 24 * n_cu && fo_align_lds_bytes(A.max_atoms, B.max_atoms, 4) <= 10 * 1024)
    launch_fo_align_t<4, 2>(a, st);
  else if (items > 12 * n_cu)
    launch_fo_align_t<2, 4>(a, st);
  else
    launch_fo_align_t<1, 4>(a, st);
  return hipGetLastError();
}

hipError_t launch_best_pose(const float* T, const float* pose, int n_pairs, int n_starts,
                            float* best_pose, float* best_T, hipStream_t st) {
  hipLaunchKernelGGL(k_best_pose, dim3((n_pairs + 255) / 256), dim3(256), 0, st, T, pose,
                     n_pairs, n_starts, best_pose, best_T);
  return hipGetLastError();
}

hipError_t launch_group_max(const float* T, int64_t n_T, const int* goff, int n_groups,
                            float* best_T, int* best_idx, int* flag, hipStream_t st) {
  hipLaunchKernelGGL(k_group_max, dim3((n_groups + 255) / 256), dim3(256), 0, st, T, n_T, goff,
                     n_groups, best_T, best_idx, flag);
  return hipGetLastError();
}

hipError_t launch_apply_pose(const MolsDev& M, const float* pose, float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_apply_pose, dim3((unsigned)M.n_mols), dim3(kWave), 0, st, M, pose, out);
  return hipGetLastError();
}

}  // namespace shape
