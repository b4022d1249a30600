// Differentiable rigid alignment (section "Differentiable alignment and the
// hybrid pipeline", Eqs. pose and grad): value and pose gradient of the
// aligned Tanimoto under common random numbers, and the Adam update.
//
// B is moved rigidly, c''_j = R(q/|q|) c_j + t; A's first n samples r_k and
// weights w_A(r_k) stay fixed, so
//   O(xi) = Z_A/n sum_k w_A(r_k) u_B(r_k; xi),  T = O / (O_aa + O_bb - O).
// Gradient of u_B at one point: du/dc''_j = beta_j (r - c''_j) with
// beta_j = 2 alpha_j o_j prod_{k != j} (1 - o_k).  With B0 = sum beta_j and
// C = sum beta_j c''_j (both carried through the atom loop by a forward
// recurrence, no division by 1 - o_j):
//   du/dt     = B0 r - C
//   du/dtheta = C x r - t' x (B0 r - C)     (infinitesimal rotation about B's
//                                             origin, t' = B's origin)
// and dT/dq follows from dtheta = 2 (w dv - dw v + v x dv) for q = (w, v).
#include "shape_kernels.hpp"
#include "shape_launch.hpp"

#include <algorithm>
#include <type_traits>

#include <math.h>

namespace shape {

__device__ __forceinline__ void quat_rotation(float qw, float qx, float qy, float qz,
                                              float (&R)[9], float& inv_norm) {
  const float n2 = qw * qw + qx * qx + qy * qy + qz * qz;
  inv_norm = rsqrtf(n2);
  const float w = qw * inv_norm, x = qx * inv_norm, y = qy * inv_norm, z = qz * inv_norm;
  R[0] = 1.f - 2.f * (y * y + z * z); R[1] = 2.f * (x * y - w * z); R[2] = 2.f * (x * z + w * y);
  R[3] = 2.f * (x * y + w * z); R[4] = 1.f - 2.f * (x * x + z * z); R[5] = 2.f * (y * z - w * x);
  R[6] = 2.f * (x * z - w * y); R[7] = 2.f * (y * z + w * x); R[8] = 1.f - 2.f * (x * x + y * y);
}

// A molecule's samples k0 .. k1 - 1 and their weights, drawn by the whole
// workgroup D per thread at a time: put(k, x, y, z, w, u) for each of them, a
// thread's in ascending order.  The molecule's records are in its own frame.
template <int D, class Put>
__device__ __forceinline__ void weigh_samples(const Atom* AF, const AtomSampling* AS,
                                              const AtomRec* AR, const float* Aa, int na,
                                              uint32_t id, int k0, int k1, uint2 key, Put put) {
  for (int i = k0 + threadIdx.x; i < k1; i += D * blockDim.x) {
    uint32_t k[D];
    float rx[D], ry[D], rz[D], r2[D], m[D], u[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      k[d] = min(i + d * (int)blockDim.x, k1 - 1);  // past the end: the last sample again
      m[d] = 0.f;
      u[d] = 0.f;
    }
    int j[D];
    float z[3 * D];
    draws<D>(AS, na, id, k, key, j, z);
    draw_points<D>(AF, AS, j, z, 1.0f, rx, ry, rz);
#pragma unroll
    for (int d = 0; d < D; ++d) r2[d] = norm2(rx[d], ry[d], rz[d]);
    eval_density_u_x<D>(AR, Aa, na, rx, ry, rz, r2, m, u);
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (i + d * (int)blockDim.x < k1)
        put((int)k[d], rx[d], ry[d], rz[d], bounded_weight(u[d], m[d]), u[d]);
  }
}

// Phase 1 (whole workgroup): A's samples in A's frame and their weights.
__device__ void align_samples(const AlignArgs& a, int pair, float4* sSamp, Atom* sAF,
                              AtomSampling* sAS, AtomRec* sAR, float* sAa) {
  const int a0 = a.offA[pair], na = a.offA[pair + 1] - a0;
  const float4 cA = a.A.centre[pair];
  for (int i = threadIdx.x; i < na; i += blockDim.x) {
    const Atom at = a.A.atom[a0 + i];
    Atom f = at;
    f.x = at.x - cA.x;
    f.y = at.y - cA.y;
    f.z = at.z - cA.z;
    sAF[i] = f;
    sAS[i] = a.A.samp[a0 + i];
    make_rec(at, cA.x, cA.y, cA.z, sAR[i], sAa[i]);
  }
  __syncthreads();
  const auto put = [&](int k, float x, float y, float z, float w, float) {
    sSamp[k] = make_float4(x, y, z, w);
  };
  // two per thread would draw the last sample in place of those past the end
  if (a.n_samples > (int)blockDim.x)
    weigh_samples<2>(sAF, sAS, sAR, sAa, na, a.A.id[pair], 0, a.n_samples, a.key, put);
  else
    weigh_samples<1>(sAF, sAS, sAR, sAa, na, a.A.id[pair], 0, a.n_samples, a.key, put);
  __syncthreads();
}

// One Adam (Kingma and Ba) ascent step on T for component c of a pose, with
// moments m, v: bias corrections c1, c2, gradient dT; the caller renormalises
// the quaternion.  Shared by the fused optimisation in the alignment kernels
// and by k_adam_pose, so both take the same roundings.
__device__ __forceinline__ float adam_component(float x, float& m, float& v, float dT, float c1,
                                                float c2, float lr, float b1, float b2,
                                                float eps) {
#pragma clang fp contract(off)
  const float g = -dT;  // minimise -T
  m = fmaf(b1, m, (1.f - b1) * g);
  v = fmaf(b2, v, (1.f - b2) * g * g);
  return x - lr * (m / c1) / (sqrtf(v / c2) + eps);
}
__device__ __forceinline__ float quat_inv_norm(float a, float b, float c, float d) {
#pragma clang fp contract(off)
  return rsqrtf(a * a + b * b + c * c + d * d);
}

// A start's optimisation state, one pose component per lane (lanes past 6
// repeat component 6): the pose is read across lanes where it is needed.
struct LanePose {
  float x, m = 0.f, v = 0.f;
  float c1, c2;  // bias corrections of steps 64 k + 1 + lane, refilled every 64 steps
  static __device__ __forceinline__ float lane_of(float f, int l) {
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_readlane(__builtin_bit_cast(int, f), l));
  }
  __device__ __forceinline__ float get(int c) const { return lane_of(x, c); }
  // ascent step t (from 1) along the gradient g[7]
  __device__ __forceinline__ void step(const float (&g)[7], int t, float lr, float b1, float b2,
                                       float eps) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & (kWave - 1);
    float gl = g[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) gl = lane == c ? g[c] : gl;
    const int i = (t - 1) % kWave;
    if (i == 0) {
      c1 = 1.f - powf(b1, (float)(t + lane));
      c2 = 1.f - powf(b2, (float)(t + lane));
    }
    x = adam_component(x, m, v, gl, lane_of(c1, i), lane_of(c2, i), lr, b1, b2, eps);
    const float inv = quat_inv_norm(get(0), get(1), get(2), get(3));
    if (lane < 4) x *= inv;
  }
};

// B's atoms moved by a pose, as the records the evaluation reads:
// expanded-form records in A's frame, and 2 alpha_j (c''_j, 1).
struct MovedAtoms {
  AtomRec* rec;
  float4* c;
  float* a2;
  // atoms lane, lane + 64, ... by the pose P; tx, ty, tz: B's origin (the
  // rotation centre) in A's frame
  __device__ __forceinline__ void move(const Atom* B, int nb, const float (&R)[9], float tx,
                                       float ty, float tz) const {
    for (int i = threadIdx.x & (kWave - 1); i < nb; i += kWave) {
      const Atom at = B[i];
      Atom moved = at;
      moved.x = fmaf(R[0], at.x, fmaf(R[1], at.y, fmaf(R[2], at.z, tx)));
      moved.y = fmaf(R[3], at.x, fmaf(R[4], at.y, fmaf(R[5], at.z, ty)));
      moved.z = fmaf(R[6], at.x, fmaf(R[7], at.y, fmaf(R[8], at.z, tz)));
      make_rec(moved, 0.f, 0.f, 0.f, rec[i], a2[i]);
      // 2 alpha = 2 a2 ln 2
      const float two_al = 2.0f * 0.693147180559945309f * at.a2;
      c[i] = make_float4(two_al * moved.x, two_al * moved.y, two_al * moved.z, two_al);
    }
  }
};

// A lane's samples of slots t .. t + S - 1 (slot i holds sample lane + 64 i;
// past the last sample: sample 0 with weight 0) against B's moved atoms.
// term(s, w, f): the sample's weight and its seven integrands f = u, du/dt
// (3), torque about B's origin (3).
//
// VALU issue bounds this loop: 13 FP32 instructions and one exponential per
// atom and sample, the exponentials of U atoms grouped (trans_group).
template <int S, int U, class Term>
__device__ __forceinline__ void align_eval(const float4* sSamp, int n_samples, int t,
                                           const MovedAtoms& B, int nb, float tx, float ty,
                                           float tz, Term term) {
  const int lane = threadIdx.x & (kWave - 1);
  float rx[S], ry[S], rz[S], r2[S];
  float P[S], S0[S], Sx[S], Sy[S], Sz[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int k = lane + kWave * (t + s);
    const float4 c = sSamp[k < n_samples ? k : 0];
    rx[s] = c.x; ry[s] = c.y; rz[s] = c.z;
    r2[s] = norm2(c.x, c.y, c.z);
    P[s] = 1.f; S0[s] = 0.f; Sx[s] = 0.f; Sy[s] = 0.f; Sz[s] = 0.f;
  }
  const auto atoms = [&](int j, auto count) {
    constexpr int V = decltype(count)::value;
    float o[V * S];
    float4 cj[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const AtomRec b = B.rec[j + u];
      const float aj = B.a2[j + u];
      cj[u] = B.c[j + u];
#pragma unroll
      for (int s = 0; s < S; ++s) o[u * S + s] = exponent_x(b, aj, rx[s], ry[s], rz[s], r2[s]);
    }
    exp2_group(o);
#pragma unroll
    for (int u = 0; u < V; ++u)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        // S <- S (1 - o) + o P c  written as  S + o (c P - S): two fused
        // operations per component, and P <- P - o P
        const float oj = o[u * S + s];
        S0[s] = fmaf(oj, fmaf(cj[u].w, P[s], -S0[s]), S0[s]);
        Sx[s] = fmaf(oj, fmaf(cj[u].x, P[s], -Sx[s]), Sx[s]);
        Sy[s] = fmaf(oj, fmaf(cj[u].y, P[s], -Sy[s]), Sy[s]);
        Sz[s] = fmaf(oj, fmaf(cj[u].z, P[s], -Sz[s]), Sz[s]);
        P[s] = fmaf(-oj, P[s], P[s]);
      }
  };
  int j = 0;
  for (; j + U <= nb; j += U) atoms(j, std::integral_constant<int, U>{});
  if constexpr (U > 1)
    for (; j < nb; ++j) atoms(j, std::integral_constant<int, 1>{});
#pragma unroll
  for (int s = 0; s < S; ++s) {
    // translation gradient of u at this point and the torque about B's origin
    const float gx = fmaf(S0[s], rx[s], -Sx[s]);
    const float gy = fmaf(S0[s], ry[s], -Sy[s]);
    const float gz = fmaf(S0[s], rz[s], -Sz[s]);
    const float cxr_x = Sy[s] * rz[s] - Sz[s] * ry[s];
    const float cxr_y = Sz[s] * rx[s] - Sx[s] * rz[s];
    const float cxr_z = Sx[s] * ry[s] - Sy[s] * rx[s];
    const float txg_x = ty * gz - tz * gy;
    const float txg_y = tz * gx - tx * gz;
    const float txg_z = tx * gy - ty * gx;
    const int k = lane + kWave * (t + s);
    const float w = k < n_samples ? sSamp[k].w : 0.f;
    const float f[7] = {1.f - P[s],      gx, gy, gz, cxr_x - txg_x, cxr_y - txg_y,
                        cxr_z - txg_z};
    term(s, w, f);
  }
}

// T and its gradient over the pose, where asked for, from the seven weighted
// sums of the integrands (FP64).
__device__ __forceinline__ void align_value(const double (&sum)[7], double Za, double S,
                                            int n_samples, const LanePose& ps, float inv_norm,
                                            bool need_T, bool need_grad, float& T,
                                            float (&g)[7]) {
  const double scale = Za / (double)n_samples;
  const double O = scale * sum[0];
  const double D = S - O;
  if (need_T) T = (float)(O / D);
  if (!need_grad) return;
  const double k = scale * S / (D * D);  // dT/dO * Z_A/n
  const double gth[3] = {k * sum[4], k * sum[5], k * sum[6]};
  // dT/dq = (2/|q|) [ -v.g ; w g - v x g ] with (w, v) = q/|q|
  const double in = (double)inv_norm;
  const double w = ps.get(0) * in, vx = ps.get(1) * in, vy = ps.get(2) * in, vz = ps.get(3) * in;
  const double vdg = vx * gth[0] + vy * gth[1] + vz * gth[2];
  const double vxg_x = vy * gth[2] - vz * gth[1];
  const double vxg_y = vz * gth[0] - vx * gth[2];
  const double vxg_z = vx * gth[1] - vy * gth[0];
  g[0] = (float)(2.0 * in * (-vdg));
  g[1] = (float)(2.0 * in * (w * gth[0] - vxg_x));
  g[2] = (float)(2.0 * in * (w * gth[1] - vxg_y));
  g[3] = (float)(2.0 * in * (w * gth[2] - vxg_z));
  g[4] = (float)(k * sum[1]);
  g[5] = (float)(k * sum[2]);
  g[6] = (float)(k * sum[3]);
}

__device__ __forceinline__ void align_write(const AlignArgs& a, size_t o, const LanePose& ps,
                                            float T, const float (&g)[7]) {
  const int lane = threadIdx.x & (kWave - 1);
  if (lane == 0) {
    a.T[o] = T;
    if (a.grad)
#pragma unroll
      for (int c = 0; c < 7; ++c) a.grad[o * 7 + c] = g[c];
  }
  if (a.n_steps > 0 && lane < 7) a.pose_out[o * 7 + lane] = ps.x;
}

// Whether the pair has invalid molecules; then starts [s0, s1) get NaN.
__device__ __forceinline__ bool align_bad(const AlignArgs& a, int pair, int s0, int s1) {
  if (a.A.bad[pair] == 0 && a.B.bad[pair] == 0) return false;
  for (int i = s0 + (int)threadIdx.x; i < s1; i += blockDim.x) {
    const size_t o = (size_t)pair * a.n_starts + i;
    a.T[o] = __builtin_nanf("");
    if (a.grad)
      for (int c = 0; c < 7; ++c) a.grad[o * 7 + c] = __builtin_nanf("");
  }
  return true;
}

// LDS: the samples, then A's records while they are drawn; afterwards the
// same memory holds B's moved atoms (one set per wave or one for the
// workgroup) and, in the split kernel, the samples' integrands.  16-byte
// arrays first, then 8-byte, then 4-byte: each stays aligned.
__host__ __device__ inline size_t align_a_bytes(int max_a) {
  return (size_t)max_a * (sizeof(AtomRec) + sizeof(Atom) + sizeof(AtomSampling) + sizeof(float));
}
__host__ __device__ inline size_t align_b_bytes(int sets, int max_b) {
  return (size_t)sets * max_b * (sizeof(AtomRec) + sizeof(float4) + sizeof(float));
}
struct AlignStage {
  Atom* AF;
  AtomRec* AR;
  AtomSampling* AS;
  float* Aa;
  __device__ AlignStage(void* mem, int max_a) {
    AR = reinterpret_cast<AtomRec*>(mem);
    AF = reinterpret_cast<Atom*>(AR + max_a);
    AS = reinterpret_cast<AtomSampling*>(AF + max_a);
    Aa = reinterpret_cast<float*>(AS + max_a);
  }
};
__device__ __forceinline__ MovedAtoms moved_atoms(void* mem, int sets, int set, int max_b) {
  AtomRec* rec = reinterpret_cast<AtomRec*>(mem);
  float4* c = reinterpret_cast<float4*>(rec + (size_t)sets * max_b);
  float* a2 = reinterpret_cast<float*>(c + (size_t)sets * max_b);
  return MovedAtoms{rec + (size_t)set * max_b, c + (size_t)set * max_b,
                    a2 + (size_t)set * max_b};
}

constexpr int kAS = 4;  // samples per lane evaluated together

// One workgroup per pair and group of starts_per_block starts; A's samples
// are drawn once, then each wave optimises its starts in turn.  An evaluation
// takes a lane's samples in order, so T and the gradient do not depend on how
// the starts are spread over waves and workgroups.  Four samples per lane and
// one atom at a time take 111 registers, four waves per SIMD, as many as the
// samples' LDS allows: 10,000 pairs x 16 starts, 4 steps 17.2 -> 16.1 ms with
// the exponentials grouped (two samples per lane at eight waves per SIMD
// 17.9 ms: three LDS reads per two terms); 300 pairs x 16 starts, one
// evaluation 321 -> 179 us with eight starts per workgroup (one workgroup per
// pair and four waves left a third of the chip idle in its second round).
__global__ __launch_bounds__(kAlignMaxWaves* kWave) __attribute__((amdgpu_waves_per_eu(4)))
void k_align(AlignArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  float4* sSamp = reinterpret_cast<float4*>(smem);  // [n_samples]
  void* rest = sSamp + a.n_samples;
  const int pair = a.order ? a.order[blockIdx.x] : blockIdx.x;
  const int s0 = blockIdx.y * a.starts_per_block;
  const int s1 = min(a.n_starts, s0 + a.starts_per_block);
  if (align_bad(a, pair, s0, s1)) return;
  const AlignStage A(rest, a.max_a);
  align_samples(a, pair, sSamp, A.AF, A.AS, A.AR, A.Aa);

  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave, waves = blockDim.x / kWave;
  const int b0 = a.offB[pair], nb = a.offB[pair + 1] - b0;
  const float4 cA = a.A.centre[pair];
  const double Za = a.A.Z[pair];
  const double S = (double)a.O_aa[pair] + (double)a.O_bb[pair];
  const MovedAtoms B = moved_atoms(rest, waves, wave, a.max_b);
  const int per_lane = (a.n_samples + kWave - 1) / kWave;
  for (int st = s0 + wave; st < s1; st += waves) {
    const size_t o = (size_t)pair * a.n_starts + st;
    LanePose ps;
    ps.x = a.pose[o * 7 + (lane < 7 ? lane : 6)];
    for (int it = 0;; ++it) {  // it = Adam steps taken
      float inv_norm;
      const float tx = ps.get(4) - cA.x, ty = ps.get(5) - cA.y, tz = ps.get(6) - cA.z;
      {
        float R[9];
        quat_rotation(ps.get(0), ps.get(1), ps.get(2), ps.get(3), R, inv_norm);
        B.move(a.B.atom + b0, nb, R, tx, ty, tz);
      }
      wave_lds_sync();
      float acc[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      for (int t = 0; t < per_lane; t += kAS)
        align_eval<kAS, 1>(sSamp, a.n_samples, t, B, nb, tx, ty, tz,
                        [&](int, float w, const float (&f)[7]) {
#pragma unroll
                          for (int c = 0; c < 7; ++c) acc[c] = fmaf(w, f[c], acc[c]);
                        });
      // butterfly sums: every lane holds the totals, so T and its gradient
      // are wave-uniform
      double sum[7];
#pragma unroll
      for (int c = 0; c < 7; ++c) sum[c] = wave_sum((double)acc[c]);
      const bool last = it >= a.n_steps;
      float T, g[7];
      align_value(sum, Za, S, a.n_samples, ps, inv_norm, last, a.grad || !last, T, g);
      wave_lds_sync();  // this pose's records are read before the next move
      if (last) {
        align_write(a, o, ps, T, g);
        break;
      }
      ps.step(g, it + 1, a.lr, 0.9f, 0.999f, 1e-8f);
    }
  }
}

// The same optimisation with one start per workgroup, its samples spread over
// sixteen waves: for calls with too few starts to fill the chip.  The waves
// write each sample's integrands to LDS, and a wave per sum adds them in the
// order one wave would have taken them, so the sums have k_align's bits.
// Latency bounds it: of about 10 us per step (2,048 samples, 30 atoms) 2.5 us
// are the serial part of one wave (sums, gradient, Adam, moving the atoms).
// 10 pairs x 16 starts, 60 steps: 12.5 -> 0.65 ms (one wave per start, four
// starts in turn, before); eight waves of four samples per lane 0.72 ms.
constexpr int kSplitWaves = 16;
constexpr int kSplitS = 2;
constexpr int kSplitSlots = kSplitWaves * kSplitS;  // slots of 64 samples per pass
struct SplitShared {
  double sum[7];  // the integrands' weighted sums
  float t[3];     // B's origin in A's frame
};

__global__ __launch_bounds__(kSplitWaves* kWave) void k_align_split(AlignArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ SplitShared sh;
  float4* sSamp = reinterpret_cast<float4*>(smem);  // [n_samples]
  void* rest = sSamp + a.n_samples;
  const int pair = blockIdx.x, st = blockIdx.y;
  if (align_bad(a, pair, st, st + 1)) return;
  const AlignStage A(rest, a.max_a);
  align_samples(a, pair, sSamp, A.AF, A.AS, A.AR, A.Aa);

  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int b0 = a.offB[pair], nb = a.offB[pair + 1] - b0;
  const float4 cA = a.A.centre[pair];
  const double Za = a.A.Z[pair];
  const double S = (double)a.O_aa[pair] + (double)a.O_bb[pair];
  const MovedAtoms B = moved_atoms(rest, 1, 0, a.max_b);
  const int per_lane = (a.n_samples + kWave - 1) / kWave;
  // integrand c of slot i (of this pass), lane l: sF[(c slots + i) 64 + l]
  const int slots = min(per_lane, kSplitSlots);
  float* sF = reinterpret_cast<float*>((unsigned char*)rest + align_b_bytes(1, a.max_b));
  const size_t o = (size_t)pair * a.n_starts + st;
  LanePose ps;  // wave 0's
  ps.x = a.pose[o * 7 + (lane < 7 ? lane : 6)];
  for (int it = 0;; ++it) {
    float inv_norm = 0.f;
    if (wave == 0) {
      float R[9];
      quat_rotation(ps.get(0), ps.get(1), ps.get(2), ps.get(3), R, inv_norm);
      const float tx = ps.get(4) - cA.x, ty = ps.get(5) - cA.y, tz = ps.get(6) - cA.z;
      B.move(a.B.atom + b0, nb, R, tx, ty, tz);
      if (lane == 0) {
        sh.t[0] = tx;
        sh.t[1] = ty;
        sh.t[2] = tz;
      }
    }
    __syncthreads();  // the moved atoms
    float acc = 0.f;
    for (int t0 = 0; t0 < per_lane; t0 += kSplitSlots) {
      const int t = t0 + wave * kSplitS;
      if (t < per_lane)
        align_eval<kSplitS, 4>(sSamp, a.n_samples, t, B, nb, sh.t[0], sh.t[1], sh.t[2],
                            [&](int s, float, const float (&f)[7]) {
                              const int i = wave * kSplitS + s;
                              if (i < slots)
#pragma unroll
                                for (int c = 0; c < 7; ++c)
                                  sF[(c * slots + i) * kWave + lane] = f[c];
                            });
      __syncthreads();  // this pass's integrands
      if (wave < 7) {
        const int n = min(slots, per_lane - t0);
        const float* F = sF + (size_t)wave * slots * kWave + lane;
#pragma unroll 8
        for (int i = 0; i < n; ++i) {
          const int k = lane + kWave * (t0 + i);
          acc = fmaf(k < a.n_samples ? sSamp[k].w : 0.f, F[i * kWave], acc);
        }
      }
      if (t0 + kSplitSlots < per_lane) __syncthreads();  // read before the next pass writes
    }
    if (wave < 7) {
      const double s = wave_sum((double)acc);
      if (lane == 0) sh.sum[wave] = s;
    }
    __syncthreads();  // the sums (and every read of the moved atoms)
    const bool last = it >= a.n_steps;
    if (wave == 0) {
      double sum[7];
#pragma unroll
      for (int c = 0; c < 7; ++c) sum[c] = sh.sum[c];
      float T, g[7];
      align_value(sum, Za, S, a.n_samples, ps, inv_norm, last, a.grad || !last, T, g);
      if (last)
        align_write(a, o, ps, T, g);
      else
        ps.step(g, it + 1, a.lr, 0.9f, 0.999f, 1e-8f);
    }
    if (last) break;
  }
}

// Self-overlap of each molecule from its own first n samples,
// O_MM = Z_M / n sum_k w_M u_M (pose invariant); one workgroup per molecule of
// the first set, then of the second (from: the launch's first of them).
// The terms are added by kSelfLanes lanes in a fixed order: lane i takes samples
// i, i + kSelfLanes, ...  A workgroup of kSelfLanes threads draws D samples per
// thread and adds them at once; one of kSelfThreads, for few molecules, draws
// them four times as fast into LDS and adds them from there.  VALU issue bounds
// long calls, latency short ones.  256 : 1,024 threads, us, 10-50 atoms: 2,048
// samples, 512 molecules 36 : 25, 1,500 50 : 45, 3,000 72 : 75, 20,000 350 : 393;
// 512 samples, 512 molecules 19 : 19, 1,500 21 : 32, 20,000 118 : 275.
constexpr int kSelfThreads = 1024;
constexpr int kSelfLanes = 256;
constexpr int kSelfChunk = 2048;  // a multiple of kSelfLanes
template <int kThreads, int D>
__global__ __launch_bounds__(kThreads) void k_self_overlap(SelfSet first, SelfSet second,
                                                           int64_t from, int n_samples,
                                                           uint2 key) {
  constexpr bool kStaged = kThreads != kSelfLanes;
  __shared__ float2 sWU[kStaged ? kSelfChunk : 1];  // weight and occupancy of a chunk's samples
  __shared__ Atom sF[SHAPE_MAX_ATOMS];
  __shared__ AtomSampling sS[SHAPE_MAX_ATOMS];
  __shared__ AtomRec sR[SHAPE_MAX_ATOMS];
  __shared__ float sA[SHAPE_MAX_ATOMS];
  __shared__ double red[kSelfLanes / kWave];
  const int64_t item = from + blockIdx.x;
  const bool in_first = item < first.n;
  const SelfSet& set = in_first ? first : second;
  const int mol = (int)(in_first ? item : item - first.n);
  if (mol >= set.n) return;
  const Prepared& M = set.M;
  const int* __restrict__ off = set.off;
  float* __restrict__ out = set.out;
  if (M.bad[mol] != 0) {
    if (threadIdx.x == 0) out[mol] = __builtin_nanf("");
    return;
  }
  const int a0 = off[mol], na = off[mol + 1] - a0;
  const float4 c = M.centre[mol];
  for (int i = threadIdx.x; i < na; i += blockDim.x) {
    const Atom at = M.atom[a0 + i];
    Atom f = at;
    f.x = at.x - c.x;
    f.y = at.y - c.y;
    f.z = at.z - c.z;
    sF[i] = f;
    sS[i] = M.samp[a0 + i];
    make_rec(at, c.x, c.y, c.z, sR[i], sA[i]);
  }
  __syncthreads();
  float acc = 0.f;
  if constexpr (!kStaged) {
    weigh_samples<D>(sF, sS, sR, sA, na, M.id[mol], 0, n_samples, key,
                     [&](int, float, float, float, float w, float u) { acc = fmaf(w, u, acc); });
  } else {
    for (int k0 = 0; k0 < n_samples; k0 += kSelfChunk) {
      const int k1 = min(n_samples, k0 + kSelfChunk);
      weigh_samples<D>(sF, sS, sR, sA, na, M.id[mol], k0, k1, key,
                       [&](int k, float, float, float, float w, float u) {
                         sWU[k - k0] = make_float2(w, u);
                       });
      __syncthreads();
      if (threadIdx.x < kSelfLanes)
        for (int k = threadIdx.x; k < k1 - k0; k += kSelfLanes) {
          const float2 t = sWU[k];
          acc = fmaf(t.x, t.y, acc);
        }
      __syncthreads();
    }
  }
  if (threadIdx.x < kSelfLanes) {
    const double s = wave_sum((double)acc);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kSelfLanes / kWave; ++w) t += red[w];
    out[mol] = (float)(M.Z[mol] * t / (double)n_samples);
  }
}

// Adam (Kingma and Ba) ascent on T over the seven pose parameters, one thread
// per pose; quaternions are renormalised after the update.  The step counter
// lives in device memory so the same launch can be replayed.
__global__ void k_adam_pose(float* __restrict__ pose, const float* __restrict__ dT,
                            float* __restrict__ m, float* __restrict__ v, int64_t n_poses,
                            int* __restrict__ step, float lr, float b1, float b2, float eps) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int t = *step + 1;
  if (i < n_poses) {
    float x[7], mi[7], vi[7], g[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      x[c] = pose[i * 7 + c];
      mi[c] = m[i * 7 + c];
      vi[c] = v[i * 7 + c];
      g[c] = dT[i * 7 + c];
    }
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
#pragma unroll
    for (int c = 0; c < 7; ++c)
      x[c] = adam_component(x[c], mi[c], vi[c], g[c], c1, c2, lr, b1, b2, eps);
    const float inv = quat_inv_norm(x[0], x[1], x[2], x[3]);
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      pose[i * 7 + c] = c < 4 ? x[c] * inv : x[c];
      m[i * 7 + c] = mi[c];
      v[i * 7 + c] = vi[c];
    }
  }
}

// Advances the device step counter after an Adam update (one thread).
__global__ void k_step_advance(int* step) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *step += 1;
}

// Best start per pair by final T (lowest index on ties; NaN never wins).
__global__ void k_best_start(const float* __restrict__ T, int n_pairs, int n_starts,
                             int* __restrict__ best) {
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
  best[p] = b;
}

// The layout with four waves (what a call must fit, whichever kernel runs it).
size_t align_lds_bytes(int n_samples, int max_a, int max_b) {
  return (size_t)n_samples * sizeof(float4) + align_a_bytes(max_a) + align_b_bytes(kAlignMinWaves, max_b);
}

static size_t align_lds(int n_samples, int max_a, int max_b, int sets, int split_slots) {
  return (size_t)n_samples * sizeof(float4) +
         std::max(align_a_bytes(max_a), align_b_bytes(sets, max_b) +
                                            (size_t)split_slots * 7 * kWave * sizeof(float));
}

static size_t split_lds_bytes(int n_samples, int max_a, int max_b) {
  const int per_lane = (n_samples + kWave - 1) / kWave;
  return align_lds(n_samples, max_a, max_b, 1, std::min(per_lane, kSplitSlots));
}
bool align_splits(int n_pairs, int n_starts, int n_steps, int n_samples, int max_a, int max_b,
                  double mean_b, int n_cu, size_t max_lds) {
  const int per_lane = (n_samples + kWave - 1) / kWave;
  const int busy = std::min(kSplitWaves, (per_lane + kSplitS - 1) / kSplitS);
  const int resident = (int)(max_lds / align_lds(n_samples, max_a, max_b, kAlignMinWaves, 0)) *
                       std::min(n_starts, kAlignMinWaves);
  return align_splits_starts(n_pairs, n_starts, n_steps, busy, resident, mean_b, n_cu) &&
         align_split_fits(split_lds_bytes(n_samples, max_a, max_b), sizeof(SplitShared), max_lds);
}

hipError_t launch_align(const AlignArgs& args, int n_pairs, int n_cu, size_t max_lds,
                        hipStream_t st) {
  AlignArgs a = args;
  if (align_splits(n_pairs, a.n_starts, a.n_steps, a.n_samples, a.max_a, a.max_b, a.mean_b, n_cu,
                   max_lds)) {
    hipLaunchKernelGGL(k_align_split, dim3((unsigned)n_pairs, (unsigned)a.n_starts),
                       dim3(kSplitWaves * kWave), split_lds_bytes(a.n_samples, a.max_a, a.max_b),
                       st, a);
    return hipGetLastError();
  }
  const int waves = align_waves(
      n_pairs, a.n_starts, align_lds(a.n_samples, a.max_a, a.max_b, kAlignMaxWaves, 0) <= max_lds,
      3 * align_lds(a.n_samples, a.max_a, a.max_b, kAlignMinWaves, 0) > max_lds, n_cu);
  a.starts_per_block = align_starts_per_block(n_pairs, a.n_starts, waves, n_cu);
  const unsigned groups = (unsigned)((a.n_starts + a.starts_per_block - 1) / a.starts_per_block);
  hipLaunchKernelGGL(k_align, dim3((unsigned)n_pairs, groups), dim3(waves * kWave),
                     align_lds(a.n_samples, a.max_a, a.max_b, waves, 0), st, a);
  return hipGetLastError();
}

template <int kThreads, int D>
static hipError_t launch_self_overlap_t(const SelfSet& a, const SelfSet& b, int n_samples,
                                        uint2 key, hipStream_t st) {
  const int64_t n = a.n + (int64_t)b.n, most = max_workgroups(kThreads);
  for (int64_t from = 0; from < n; from += most) {
    hipLaunchKernelGGL((k_self_overlap<kThreads, D>), dim3((unsigned)std::min(most, n - from)),
                       dim3(kThreads), 0, st, a, b, from, n_samples, key);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_self_overlap(const SelfSet& a, const SelfSet& b, int n_samples, uint2 key,
                               int n_cu, hipStream_t st) {
  // 1,024 threads while their workgroups, two per compute unit, all start within a
  // few turns; with one sample per thread the smaller ones win earlier
  const int64_t n = a.n + (int64_t)b.n;
  if (n_samples > kSelfThreads && n <= (int64_t)8 * n_cu)
    return launch_self_overlap_t<kSelfThreads, 2>(a, b, n_samples, key, st);
  if (n_samples > kSelfLanes && n <= (int64_t)4 * n_cu)
    return launch_self_overlap_t<kSelfThreads, 1>(a, b, n_samples, key, st);
  if (n_samples > kSelfLanes) return launch_self_overlap_t<kSelfLanes, 2>(a, b, n_samples, key, st);
  return launch_self_overlap_t<kSelfLanes, 1>(a, b, n_samples, key, st);
}

hipError_t launch_adam_pose(float* pose, const float* dT, float* m, float* v, int64_t n_poses,
                            int* step, float lr, float b1, float b2, float eps,
                            hipStream_t st) {
  const int64_t blocks = (n_poses + 255) / 256;
  hipLaunchKernelGGL(k_adam_pose, dim3((unsigned)blocks), dim3(256), 0, st, pose, dT, m, v,
                     n_poses, step, lr, b1, b2, eps);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_step_advance, dim3(1), dim3(1), 0, st, step);
  return hipGetLastError();
}

hipError_t launch_best_start(const float* T, int n_pairs, int n_starts, int* best,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_best_start, dim3((n_pairs + 255) / 256), dim3(256), 0, st, T, n_pairs,
                     n_starts, best);
  return hipGetLastError();
}

}  // namespace shape
