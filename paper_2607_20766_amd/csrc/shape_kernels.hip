// HIP kernels of the IS shape-overlap engine: molecule preparation, the
// single-pair estimator and fixed / adaptive screening.
//
// Data layout in HBM (prepared by k_prepare, one record per atom, CSR order):
//   Atom          16 B  (x, y, z, alpha*log2 e)       hot-loop operand
//   AtomSampling   8 B  (1/sqrt(2 alpha), threshold)  only for sampling
//   Z             FP64 per molecule, stream id per molecule, invalid flag.
#include "shape_kernels.hpp"
#include "shape_launch.hpp"

#include <math.h>

namespace shape {

// ---------------------------------------------------------------------------
// Eq. occ widths: alpha = kappa / (lambda R^2).
// ---------------------------------------------------------------------------
__global__ void k_alpha_from_radius(const float* __restrict__ R, int64_t n, double kappa,
                                    double lambda, float* __restrict__ alpha) {
#pragma clang fp contract(off)
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double r = (double)R[i];
  alpha[i] = (float)(kappa / (lambda * r * r));
}

// ---------------------------------------------------------------------------
// Molecule preparation, one wave per molecule (four per workgroup), FP64:
// mixture weights v_i = (pi/alpha_i)^(3/2) (= t sqrt t, t = pi/alpha_i), one
// atom per lane and chunk of 64; Z = sum v_i and the running sums behind the
// thresholds floor(2^32 cumsum(v)/Z) are the plain sequential sums in atom
// order, bit for bit: the wave adds the weights one lane at a time (read
// across lanes, no LDS round trips) and each lane keeps the running sum that
// ends at its own atom.  Inputs stay in registers between the two phases.
// ---------------------------------------------------------------------------
constexpr int kPrepWaves = 4;
constexpr int kPrepChunks = SHAPE_MAX_ATOMS / kWave;

__device__ __forceinline__ void prepare_molecule(const MolsDev& in, const Prepared& out, int m,
                                                 int* __restrict__ flag,
                                                 int* __restrict__ set_flag) {
  // FP64 without contraction: Z and the thresholds are the values the plain
  // expressions define, bit for bit.
#pragma clang fp contract(off)
  const int lane = threadIdx.x & (kWave - 1);
  const int a0 = in.off[m], a1 = in.off[m + 1];
  const int n = a1 - a0;
  const bool range_bad = !(a0 >= 0 && (int64_t)a1 <= in.n_atoms && n >= 1 && n <= in.max_atoms);
  const int n_ok = range_bad ? 0 : n;  // n_ok <= SHAPE_MAX_ATOMS
  bool bad = range_bad;
  float px[kPrepChunks], py[kPrepChunks], pz[kPrepChunks], pa[kPrepChunks];
  double run[kPrepChunks];  // running sum through this lane's atom of each chunk
  float cx = 0.0f, cy = 0.0f, cz = 0.0f;
  double cum = 0.0;
#pragma unroll
  for (int c = 0; c < kPrepChunks; ++c) {
    px[c] = py[c] = pz[c] = 0.0f;
    pa[c] = 1.0f;
    run[c] = 0.0;
    if (c * kWave >= n_ok) continue;  // uniform
    const int i = c * kWave + lane;
    double v = 0.0;
    if (i < n_ok) {
      const float al = in.alpha[a0 + i];
      const float x = in.xyz[3 * (a0 + i)], y = in.xyz[3 * (a0 + i) + 1],
                  z = in.xyz[3 * (a0 + i) + 2];
      if (!(al > 0.0f) || !isfinite(al) || !isfinite(x) || !isfinite(y) || !isfinite(z))
        bad = true;
      const double t = M_PI / (double)al;
      v = t * sqrt(t);
      px[c] = x;
      py[c] = y;
      pz[c] = z;
      pa[c] = al;
      cx += x;
      cy += y;
      cz += z;
    }
    const int cnt = min(kWave, n_ok - c * kWave);
    for (int j = 0; j < cnt; ++j) {
      cum += readlane_f64(v, j);
      if (lane == j) run[c] = cum;
    }
  }
  bad = __ballot(bad) != 0;
  if (lane == 0) {
    out.id[m] = in.id ? in.id[m] : (uint32_t)m;
    out.bad[m] = bad ? 1 : 0;
  }
  if (bad) {
    if (lane == 0) {
      out.Z[m] = __builtin_nan("");
      out.centre[m] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      atomicOr(flag, 1);
      if (set_flag) atomicOr(set_flag, 1);
    }
    return;
  }
  // the centre is only the origin of the molecule's frame: FP32 sums
  const float scx = wave_sum_dpp(cx), scy = wave_sum_dpp(cy), scz = wave_sum_dpp(cz);
  const double Z = cum;
  if (lane == 0) {
    out.Z[m] = Z;
    const float inv_n = 1.0f / (float)n;
    out.centre[m] = make_float4(scx * inv_n, scy * inv_n, scz * inv_n, 0.0f);
  }
  const double log2e = 1.4426950408889634074;
#pragma unroll
  for (int c = 0; c < kPrepChunks; ++c) {
    const int i = c * kWave + lane;
    if (i >= n) continue;
    const double al = (double)pa[c];
    Atom a;
    a.x = px[c];
    a.y = py[c];
    a.z = pz[c];
    a.a2 = (float)(al * log2e);
    out.atom[a0 + i] = a;
    AtomSampling smp;
    smp.sd = (float)(1.0 / sqrt(2.0 * al));
    if (i + 1 < n) {
      double f = floor(4294967296.0 * (run[c] / Z));
      if (f > 4294967295.0) f = 4294967295.0;
      smp.thr = (uint32_t)f;
    } else {
      smp.thr = 0xFFFFFFFFu;
    }
    out.samp[a0 + i] = smp;
  }
}

__global__ __launch_bounds__(256) void k_prepare(MolsDev in, Prepared out, int* __restrict__ flag,
                                                 int* __restrict__ set_flag,
                                                 const int* __restrict__ which, int n_which) {
  const int idx = blockIdx.x * kPrepWaves + threadIdx.x / kWave;
  if (idx >= n_which) return;
  const int m = which ? which[idx] : idx;  // a listed index may repeat
  if (m < 0 || m >= in.n_mols) return;     // or lie outside: the screen flags it
  prepare_molecule(in, out, m, flag, set_flag);
}

// Both one-molecule sets of a pair in one launch, a wave each.
__global__ __launch_bounds__(2 * kWave) void k_prepare_pair(MolsDev inA, Prepared A, MolsDev inB,
                                                            Prepared B, int* __restrict__ flag) {
  if (threadIdx.x < kWave)
    prepare_molecule(inA, A, 0, flag, nullptr);
  else
    prepare_molecule(inB, B, 0, flag, nullptr);
}

// Re-raises the invalid-data flag for a molecule set reused from an earlier
// preparation that found invalid molecules.
__global__ void k_flag_or(int* __restrict__ flag, const int* __restrict__ set_flag) {
  if (threadIdx.x == 0 && *set_flag) atomicOr(flag, 1);
}

__global__ void k_fill_int(int* __restrict__ p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// Block reduction of K doubles (wave butterflies, then waves in order).
// ---------------------------------------------------------------------------
template <int K>
__device__ void block_sum(double (&v)[K], double* lds /* [4][K] */) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
  for (int j = 0; j < K; ++j) v[j] = wave_sum(v[j]);
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < K; ++j) lds[wave * K + j] = v[j];
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = blockDim.x / kWave;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += lds[w * K + j];
      v[j] = s;
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Single pair: per-block partial sums of the eleven per-sample quantities of
// one side (samples from P, partner Q):
//   f1 = w_P u_Q, f2 = w_P u_P, f3 = w_P, f4 = m_Q, f5 = m_P
// sums: f1, f1^2, f2, f2^2, f3, f3^2, f4, f4^2, f5, f5^2, f1 f2.
// blockIdx.y = side (0: P = A, 1: P = B).  A lane takes S independent terms
// (samples, or antithetic pairs by their means) at a time and `turns` times S
// in all, in FP32; the block's lanes are added in FP64.  Invalid molecules
// (bad flags) are not read: the blocks write nothing.
//
// Few samples are bound by latency: one term per lane over four blocks of
// waves per 1,024 samples instead of eight in turn (4,096 samples per side,
// 20 x 24 atoms: 30 -> 9 us).  Many are bound by VALU issue (7 instructions,
// an exponential and 2 to 3 more per atom): four terms at a time with their
// exponentials grouped (trans_group; 10^6 x 0.8 10^6 samples, 30 x 45 atoms:
// 73 -> 49 us).
// ---------------------------------------------------------------------------
template <int S, bool kAnti>
__global__ __launch_bounds__(256) void k_est_partials(Prepared A, Prepared B, int64_t n_a,
                                                      int64_t n_b, uint2 key, int turns,
                                                      double* __restrict__ partials,
                                                      int nblk, const int* __restrict__ offA,
                                                      const int* __restrict__ offB) {
  __shared__ Atom sP[SHAPE_MAX_ATOMS];
  __shared__ Atom sQ[SHAPE_MAX_ATOMS];
  __shared__ AtomSampling sS[SHAPE_MAX_ATOMS];
  __shared__ double red[4 * kEstSums];
  if (A.bad[0] != 0 || B.bad[0] != 0) return;
  const int side = blockIdx.y;
  const Prepared& P = side ? B : A;
  const Prepared& Q = side ? A : B;
  const int* offP = side ? offB : offA;
  const int* offQ = side ? offA : offB;
  const int64_t n = side ? n_b : n_a;
  const int64_t units = kAnti ? n / 2 : n;  // independent terms: samples or pairs
  const int p0 = offP[0], np = offP[1] - offP[0];
  const int q0 = offQ[0], nq = offQ[1] - offQ[0];
  const uint32_t idp = P.id[0];
  for (int i = threadIdx.x; i < np; i += blockDim.x) {
    sP[i] = P.atom[p0 + i];
    sS[i] = P.samp[p0 + i];
  }
  for (int i = threadIdx.x; i < nq; i += blockDim.x) sQ[i] = Q.atom[q0 + i];
  __syncthreads();
  float acc[kEstSums];
#pragma unroll
  for (int j = 0; j < kEstSums; ++j) acc[j] = 0.0f;
  const int64_t base = (int64_t)blockIdx.x * turns * S * blockDim.x + threadIdx.x;
  for (int turn = 0; turn < turns; ++turn) {
    const int64_t first = base + (int64_t)turn * S * blockDim.x;
    if (first >= units) break;
    uint32_t u[S];  // terms lie below 2^32 (at most 2^31 samples)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int64_t t = first + (int64_t)s * blockDim.x;
      u[s] = (uint32_t)(t < units ? t : first);
    }
    int j[S];
    float z[3 * S], f[S][5];
    draws<S>(sS, np, idp, u, key, j, z);
#pragma unroll
    for (int mbr = 0; mbr < (kAnti ? 2 : 1); ++mbr) {
      float rx[S], ry[S], rz[S], mp[S], qp[S], mq[S], qq[S];
      draw_points<S>(sP, sS, j, z, mbr ? -1.0f : 1.0f, rx, ry, rz);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        mp[s] = mq[s] = 0.0f;
        qp[s] = qq[s] = 1.0f;
      }
      eval_density<S>(sP, np, rx, ry, rz, mp, qp);
      eval_density<S>(sQ, nq, rx, ry, rz, mq, qq);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float uP = 1.0f - qp[s], uQ = 1.0f - qq[s];
        const float w = bounded_weight(uP, mp[s]);
        const float g[5] = {w * uQ, w * uP, w, mq[s], mp[s]};
#pragma unroll
        for (int c = 0; c < 5; ++c) f[s][c] = mbr ? 0.5f * (f[s][c] + g[c]) : g[c];
      }
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (first + (int64_t)s * blockDim.x < units) {
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          acc[2 * c] += f[s][c];
          acc[2 * c + 1] += f[s][c] * f[s][c];
        }
        acc[10] += f[s][0] * f[s][1];
      }
    }
  }
  double v[kEstSums];
#pragma unroll
  for (int j = 0; j < kEstSums; ++j) v[j] = (double)acc[j];
  block_sum<kEstSums>(v, red);
  if (threadIdx.x == 0) {
    double* dst = partials + ((size_t)side * nblk + blockIdx.x) * kEstSums;
#pragma unroll
    for (int j = 0; j < kEstSums; ++j) dst[j] = v[j];
  }
}

// The blocks' sums added in a fixed order, and the result from them: thread
// 32 part + q < 22 adds quantity q of blocks part, part + 32, ..., then thread
// q adds the parts.  Lane 5 side + channel of the first wave forms that
// channel's mean and standard error (ten divisions and roots side by side
// instead of in turn).  A chain of FP64 latencies: 11 -> 4 us (16 blocks).
constexpr int kEstParts = 32;
__global__ __launch_bounds__(kEstParts * 32) void k_est_finalize(
    const double* __restrict__ partials, int nblk, Prepared A, Prepared B, int64_t n_a,
    int64_t n_b, int anti, EstOut* __restrict__ out) {
  __shared__ double part[kEstParts][2 * kEstSums];
  __shared__ double tot[2 * kEstSums];
  __shared__ double mean[10], se[10], cov[2];
  const int badA = A.bad[0], badB = B.bad[0];
  if (badA != 0 || badB != 0) {
    if (threadIdx.x == 0) {
      out->bad[0] = badA;
      out->bad[1] = badB;
    }
    return;
  }
  const int q = threadIdx.x % 32, pt = threadIdx.x / 32;
  if (q < 2 * kEstSums) {
    const double* src = partials + (size_t)(q / kEstSums) * nblk * kEstSums + q % kEstSums;
    double v = 0.0;
#pragma unroll 8
    for (int b = pt; b < nblk; b += kEstParts) v += src[(size_t)b * kEstSums];
    part[pt][q] = v;
  }
  __syncthreads();
  if (threadIdx.x < 2 * kEstSums) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < kEstParts; ++k) v += part[k][threadIdx.x];
    tot[threadIdx.x] = v;
  }
  __syncthreads();
  // independent terms per side: samples, or antithetic pair means
  const int l = threadIdx.x;
  if (l < 12) {
    const int side = l < 10 ? l / 5 : l - 10;
    const double n = (double)(anti ? (side ? n_b : n_a) / 2 : (side ? n_b : n_a));
    const double* s = tot + side * kEstSums;
    if (l < 10) {
      const double Z = side ? B.Z[0] : A.Z[0];
      const double sum = s[2 * (l % 5)], sq = s[2 * (l % 5) + 1];
      const double var = (sq - sum * sum / n) / (n - 1.0);
      mean[l] = Z * (sum / n);
      se[l] = Z * sqrt((var > 0.0 ? var : 0.0) / n);
    } else {
      const double Z = side ? B.Z[0] : A.Z[0];
      cov[side] = 0.5 * Z * Z * ((s[10] - s[0] * s[2] / n) / (n - 1.0)) / n;
    }
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  shape_result r;
  r.O_ab_from_a = mean[0];
  r.O_ab_from_b = mean[5];
  r.O_ab = 0.5 * (r.O_ab_from_a + r.O_ab_from_b);
  r.se_O_ab = 0.5 * sqrt(se[0] * se[0] + se[5] * se[5]);
  r.O_aa = mean[1];
  r.O_bb = mean[6];
  r.se_O_aa = se[1];
  r.se_O_bb = se[6];
  r.V_a = mean[2];
  r.V_b = mean[7];
  r.se_V_a = se[2];
  r.se_V_b = se[7];
  r.Ofo_ab_is = 0.5 * (mean[3] + mean[8]);
  r.Ofo_aa_is = mean[4];
  r.Ofo_bb_is = mean[9];
  const double S = r.O_aa + r.O_bb, D = S - r.O_ab;
  r.T = r.O_ab / D;
  const double iD2 = 1.0 / (D * D);
  const double g_ab = S * iD2, g_s = -r.O_ab * iD2;
  r.se_T = fabs(g_ab) * r.se_O_ab;
  const double var_s = r.se_O_aa * r.se_O_aa + r.se_O_bb * r.se_O_bb;
  const double vt = g_ab * g_ab * r.se_O_ab * r.se_O_ab + g_s * g_s * var_s +
                    2.0 * g_ab * g_s * (cov[0] + cov[1]);
  r.se_T_full = sqrt(vt > 0.0 ? vt : 0.0);
  r.n_a = n_a;
  r.n_b = n_b;
  out->bad[0] = out->bad[1] = 0;
  out->r = r;
}

// ---------------------------------------------------------------------------
// Query-side sample cache for screening: the query's own samples, weights and
// self integrand are the same for every library partner (random numbers are
// keyed by molecule), so they are computed once per call.  Points are kept in
// the query's frame (origin at its centre):
//   qs[k] = (r'_k, w_A(r_k)),  qf2[k] = w_A u_A at r_k.
// The densities use the expanded form with the same records the screening
// kernel builds, so a library copy of the query reproduces them bit for bit.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void query_cache(const Prepared& Qp, const int* __restrict__ offQ,
                                            int64_t n, uint2 key, int anti,
                                            float4* __restrict__ qs, float* __restrict__ qf2) {
  __shared__ Atom sF[SHAPE_MAX_ATOMS];          // frame coordinates for sampling
  __shared__ AtomSampling sS[SHAPE_MAX_ATOMS];
  __shared__ AtomRec sR[SHAPE_MAX_ATOMS];
  __shared__ float sA[SHAPE_MAX_ATOMS];
  // an invalid query is never staged (its atom count is not trusted); the
  // screening kernel then reports every pair as NaN without reading the cache
  if (Qp.bad[0] != 0) return;
  const int q0 = offQ[0], nq = offQ[1] - offQ[0];
  const float4 cq = Qp.centre[0];
  for (int i = threadIdx.x; i < nq; i += blockDim.x) {
    const Atom a = Qp.atom[q0 + i];
    Atom f = a;
    f.x = a.x - cq.x;
    f.y = a.y - cq.y;
    f.z = a.z - cq.z;
    sF[i] = f;
    sS[i] = Qp.samp[q0 + i];
    make_rec(a, cq.x, cq.y, cq.z, sR[i], sA[i]);
  }
  __syncthreads();
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  // sample numbers stay below 2^32 (at most 2^20)
  const uint32_t blk[1] = {(uint32_t)(anti ? k >> 1 : k)};
  int j[1];
  float z[3], rx[1], ry[1], rz[1], r2[1];
  draws<1>(sS, nq, Qp.id[0], blk, key, j, z);
  draw_points<1>(sF, sS, j, z, anti && (k & 1) ? -1.0f : 1.0f, rx, ry, rz);
  r2[0] = norm2(rx[0], ry[0], rz[0]);
  float m[1] = {0.0f}, q[1] = {1.0f};
  eval_density_x<1>(sR, sA, nq, rx, ry, rz, r2, m, q);
  const float u = 1.0f - q[0];
  const float w = bounded_weight(u, m[0]);
  qs[k] = make_float4(rx[0], ry[0], rz[0], w);
  qf2[k] = w * u;
}

// ---------------------------------------------------------------------------
// Screening kernel: one workgroup per (query, library) pair, so the pair index
// comes from blockIdx and is uniform by construction (no cross-lane
// broadcast); the hardware dispatcher balances pairs of uneven size.  The
// workgroup is a single wave, or kRounds waves that each take one of kRounds
// consecutive rounds and then add the rounds' totals, with the stop test after
// each, in turn (screen_shape: where single waves would leave the chip short
// of waves; the same bits).  Pairs are renumbered so that each XCD screens tiles of consecutive
// library molecules (xcd_chunk).  Per round, `round_side` samples on each side:
//   side A (query samples, from the cache): f1 = w_A u_B, f2 = w_A u_A
//   side B (library samples, drawn here):   f1 = w_B u_A, f2 = w_B u_B
// FP32 in-lane sums per round, summed across the wave and added in FP64.
// Adaptive mode takes the stopping decision on SE(T) in FP64 after every
// round; the decision is read from the first lane so the branch is scalar.
// ---------------------------------------------------------------------------
// Work granularity of the screening kernel: kSA (kSB) side-A (side-B) points
// per lane are evaluated together against each atom record read from LDS.
// Every variant assigns the same samples to the same lanes and accumulates
// them in the same order, so all variants give bit-identical results; the
// autotuner picks the fastest for a workload.
const int kScreenVariantShape[kScreenVariants][2] = {
    {4, 2}, {2, 2}, {4, 1}, {4, 4}, {8, 2}, {2, 1}, {8, 4}, {2, 4}};

__device__ __forceinline__ double se_tanimoto(double n, double Za, double Zb, double a1,
                                              double a11, double a2, double b1, double b11,
                                              double b2, double* T_out, double* Oab_out,
                                              double* Oaa_out, double* Obb_out) {
#pragma clang fp contract(off)
  const double xa = Za * a1 / n, xb = Zb * b1 / n;
  double va = (a11 - a1 * a1 / n) / (n - 1.0);
  double vb = (b11 - b1 * b1 / n) / (n - 1.0);
  va = va > 0.0 ? va : 0.0;
  vb = vb > 0.0 ? vb : 0.0;
  const double se_a = Za * sqrt(va / n), se_b = Zb * sqrt(vb / n);
  const double O_ab = 0.5 * (xa + xb);
  const double se_O = 0.5 * sqrt(se_a * se_a + se_b * se_b);
  const double O_aa = Za * a2 / n, O_bb = Zb * b2 / n;
  const double S = O_aa + O_bb, D = S - O_ab;
  if (T_out) *T_out = O_ab / D;
  if (Oab_out) *Oab_out = O_ab;
  if (Oaa_out) *Oaa_out = O_aa;
  if (Obb_out) *Obb_out = O_bb;
  return fabs(S / (D * D)) * se_O;
}

// A pair's six running sums (sum f1, sum f1^2, sum f2 of side A, then of side
// B), FP64: lane j < 6 holds sum j.  add() takes one round's per-lane FP32
// partials, sums each across the wave (DPP) and adds the six totals in one
// FP64 instruction; get(j) reads sum j in every lane.
struct RoundSums {
  double s = 0.0;
  // the totals of one round, total j in lane j
  static __device__ __forceinline__ float totals(const float (&fa)[3], const float (&fb)[3]) {
    const int lane = threadIdx.x & (kWave - 1);
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const float t = wave_sum_dpp(j < 3 ? fa[j] : fb[j - 3]);
      v = lane == j ? t : v;
    }
    return v;
  }
  __device__ __forceinline__ void add(float v) { s += (double)v; }
  __device__ __forceinline__ double get(int j) const { return readlane_f64(s, j); }
};

// Whether a pair stops after n_side samples per side.  Adaptive: at the cap,
// or once its seeded budget is spent and SE(T) <= tau.  That test needs no
// division or root: with n independent terms per side, S' = Za a2 + Zb b2,
// D' = S' - (Za a1 + Zb b1)/2 and V = n a11 - a1^2 (clamped at 0), the
// delta-method SE satisfies
//   SE(T)^2 = S'^2 (Za^2 Va + Zb^2 Vb) / (4 (n-1) D'^4),
// so the test is S'^2 (Za^2 Va + Zb^2 Vb) <= 4 tau^2 (n-1) D'^4 with
// D' != 0 (NaN sums never stop).
__device__ __forceinline__ bool screen_stops(const ScreenArgs& a, const RoundSums& S,
                                             int64_t n_side, int64_t first_check, bool anti,
                                             double Za, double Zb) {
#pragma clang fp contract(off)
  if (a.mode != SHAPE_SCREEN_ADAPTIVE) return n_side >= a.n_fixed;
  if (2 * n_side >= a.cap_pair) return true;
  if (2 * n_side < first_check) return false;  // below the pair's seeded budget: no test yet
  const double tau2x4 = 4.0 * a.tau * a.tau;
  const double n = (double)(anti ? n_side / 2 : n_side);  // independent terms
  const double a1 = S.get(0), a11 = S.get(1), b1 = S.get(3), b11 = S.get(4);
  const double Sp = Za * S.get(2) + Zb * S.get(5);
  const double Dp = Sp - 0.5 * (Za * a1 + Zb * b1);
  const double Va = fmax(n * a11 - a1 * a1, 0.0);
  const double Vb = fmax(n * b11 - b1 * b1, 0.0);
  const double lhs = Sp * Sp * (Za * Za * Va + Zb * Zb * Vb);
  const double D2 = Dp * Dp;
  return Dp != 0.0 && lhs <= tau2x4 * (n - 1.0) * D2 * D2;
}

// Rounds for an adaptive pair's workgroup to draw together next, at most R, after n_side
// samples per side: as many as its budget still asks for, or, past that, as (SE(T)/tau)^2
// does, which falls as 1/n.  What it returns changes no result: rounds past the stop are
// dropped.
__device__ __forceinline__ int screen_rounds_for(int R, float more) {
  return !(more < (float)R) ? R : max(1, (int)ceilf(more));
}
__device__ __forceinline__ int screen_next(const ScreenArgs& a, int R, const RoundSums& S,
                                           int64_t n_side, int64_t first_check, bool anti,
                                           double Za, double Zb) {
  const int64_t budget = first_check - 2 * n_side;
  if (budget > 0) return screen_rounds_for(R, (float)budget / (float)(2 * a.round_side));
  const float r = (float)(se_tanimoto((double)(anti ? n_side / 2 : n_side), Za, Zb, S.get(0),
                                      S.get(1), S.get(2), S.get(3), S.get(4), S.get(5), nullptr,
                                      nullptr, nullptr, nullptr) /
                          a.tau);
  return screen_rounds_for(R, (float)n_side / (float)a.round_side * (r * r - 1.0f));
}

// A pair's outputs from its sums (one lane).
__device__ __forceinline__ void screen_write(const ScreenArgs& a, int p, const RoundSums& S,
                                             int64_t n_side, bool anti, double Za, double Zb) {
  double T, O_ab, O_aa, O_bb;
  const double se = se_tanimoto((double)(anti ? n_side / 2 : n_side), Za, Zb, S.get(0), S.get(1),
                                S.get(2), S.get(3), S.get(4), S.get(5), &T, &O_ab, &O_aa, &O_bb);
  if (threadIdx.x == 0) {
    a.T[p] = (float)T;
    a.se_T[p] = (float)se;
    if (a.O_ab) a.O_ab[p] = (float)O_ab;
    if (a.O_aa) a.O_aa[p] = (float)O_aa;
    if (a.O_bb) a.O_bb[p] = (float)O_bb;
    if (a.n_used) a.n_used[p] = (int)(2 * n_side);
  }
}

__device__ __forceinline__ void screen_write_nan(const ScreenArgs& a, int p) {
  if (threadIdx.x == 0) {
    const float nanv = __builtin_nanf("");
    a.T[p] = nanv;
    a.se_T[p] = nanv;
    if (a.O_ab) a.O_ab[p] = nanv;
    if (a.O_aa) a.O_aa[p] = nanv;
    if (a.O_bb) a.O_bb[p] = nanv;
    if (a.n_used) a.n_used[p] = 0;
  }
}

// Samples per side after which a pair stops at the latest.
__device__ __forceinline__ int screen_limit(const ScreenArgs& a) {
  return (int)(a.mode == SHAPE_SCREEN_ADAPTIVE ? a.cap_pair / 2 : a.n_fixed);
}

// The kernel's arguments, read again from the kernel-argument segment: what
// only the end of a pair needs then takes no scalar registers during its
// rounds (they would be spilled into lanes of vector registers, which the
// kernel has none to spare of).
__device__ __forceinline__ const ScreenArgs& screen_args_again() {
  auto k = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(k));
  return *(const ScreenArgs*)k;
}

// LDS of one pair (n = atoms, n' = rec_pairs(n)):
//   BF    [max_b]  Atom          library atoms in the library frame (sampling)
//   BB    [max_b'] AtomRec2      library atoms, library frame (own density)
//   BA    [max_b'] AtomRec2      library atoms, query frame (side A partner)
//   AB    [max_q'] AtomRec2      query atoms, library frame (side B partner)
//   BS    [max_b]  AtomSampling  the library atoms' sampling records
//   guide [kGuideSize] uint8_t   the library molecule's component guide
// 16-byte records first, then the 8-byte and the 1-byte arrays, so every array
// is aligned to its element size whatever the atom counts.
struct ScreenLds {
  Atom* BF;
  AtomRec2 *BB, *BA, *AB;
  AtomSampling* BS;
  uint8_t* guide;
  __device__ ScreenLds(unsigned char* smem, int max_q, int max_b) {
    BF = reinterpret_cast<Atom*>(smem);
    BB = reinterpret_cast<AtomRec2*>(BF + max_b);
    BA = BB + rec_pairs(max_b);
    AB = BA + rec_pairs(max_b);
    BS = reinterpret_cast<AtomSampling*>(AB + rec_pairs(max_q));
    guide = reinterpret_cast<uint8_t*>(BS + max_b);
  }
  // the records of a pair, staged by the whole workgroup
  __device__ __forceinline__ void stage(const ScreenArgs& a, int m, int q0, int nq, int b0,
                                        int nb) const {
    const float4 cA = a.Q.centre[0];
    const float4 cB = a.L.centre[m];
    for (int i = threadIdx.x; i < nq; i += blockDim.x)
      make_rec2(a.Q.atom[q0 + i], cB.x, cB.y, cB.z, AB, i, nq);
    for (int i = threadIdx.x; i < nb; i += blockDim.x) {
      const Atom at = a.L.atom[b0 + i];
      Atom f = at;
      f.x = at.x - cB.x;
      f.y = at.y - cB.y;
      f.z = at.z - cB.z;
      BF[i] = f;
      BS[i] = a.L.samp[b0 + i];
      make_rec2(at, cB.x, cB.y, cB.z, BB, i, nb);
      make_rec2(at, cA.x, cA.y, cA.z, BA, i, nb);
    }
    __syncthreads();
    build_guide(BS, nb, guide, threadIdx.x, blockDim.x);
    __syncthreads();
  }
};

// Slot i of a lane in a round holds sample n_side + lane + 64 i (i.i.d.), or
// for antithetic sampling member i & 1 of pair n_side/2 + lane + 64 (i >> 1),
// i.e. sample n_side + 2 lane + 128 (i >> 1) + (i & 1); the pair's two
// members sit in consecutive slots of one lane and enter the sums as one
// term, their mean (held in pend1, pend2 from the first member on).
template <bool kAnti>
struct SideSums {
  float f[3] = {0.f, 0.f, 0.f};
  float pend1 = 0.f, pend2 = 0.f;
  // slot i's term: f1, and f2 = f2a f2b (a product, fused into the sum)
  __device__ __forceinline__ void term(int i, float f1, float f2a, float f2b) {
#pragma clang fp contract(off)
    if constexpr (!kAnti) {
      f[0] += f1;
      f[1] = fmaf(f1, f1, f[1]);
      f[2] = fmaf(f2a, f2b, f[2]);
    } else if ((i & 1) == 0) {
      pend1 = f1;
      pend2 = f2a * f2b;
    } else {
      const float g1 = 0.5f * (pend1 + f1), g2 = 0.5f * (pend2 + f2a * f2b);
      f[0] += g1;
      f[1] = fmaf(g1, g1, f[1]);
      f[2] += g2;
    }
  }
};

// A lane's points for slots t .. t + S - 1 of a round that starts at sample
// n_side of the library molecule (a slot past the round's last repeats slot
// t): the points sample_point, or sample_point_anti, draws.  All steps of the
// S points go together; sample numbers stay below 2^32 (at most 2^20 per
// side), so the Philox counter's second word is zero.  Antithetic pairs sit
// in consecutive slots and share one block where S is even.
template <int S, bool kAnti>
__device__ __forceinline__ void screen_draw(const ScreenLds& lds, int nb, uint32_t id,
                                            uint32_t n_side, int t, int per_lane, uint2 key,
                                            float (&rx)[S], float (&ry)[S], float (&rz)[S]) {
  constexpr bool kPairs = kAnti && S % 2 == 0;
  constexpr int D = kPairs ? S / 2 : S;
  const uint32_t lane = threadIdx.x & (kWave - 1);
  uint4 x[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const int s = kPairs ? 2 * d : d;
    const uint32_t i = (t + s) < per_lane ? t + s : t;
    const uint32_t blk = kAnti ? n_side / 2 + lane + kWave * (i >> 1) : n_side + lane + kWave * i;
    x[d] = philox_block(blk, id, key);
  }
  int j[D];
  float z[3 * D];
  draws_of<D>(x, [&](const uint32_t (&w)[D], int (&c)[D]) {
    select_components_guided<D>(lds.BS, lds.guide, nb, w, c);
  }, j, z);
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const Atom c = lds.BF[j[d]];
    const float sd = lds.BS[j[d]].sd;
    if constexpr (kPairs) {
      rx[2 * d] = fmaf(z[3 * d], sd, c.x);
      ry[2 * d] = fmaf(z[3 * d + 1], sd, c.y);
      rz[2 * d] = fmaf(z[3 * d + 2], sd, c.z);
      rx[2 * d + 1] = fmaf(-z[3 * d], sd, c.x);
      ry[2 * d + 1] = fmaf(-z[3 * d + 1], sd, c.y);
      rz[2 * d + 1] = fmaf(-z[3 * d + 2], sd, c.z);
    } else {
      // the odd member of an antithetic pair (a slot's parity is its sample's)
      const int i = (t + d) < per_lane ? t + d : t;
      const float sg = kAnti && (i & 1) ? -1.0f : 1.0f;
      rx[d] = fmaf(sg * z[3 * d], sd, c.x);
      ry[d] = fmaf(sg * z[3 * d + 1], sd, c.y);
      rz[d] = fmaf(sg * z[3 * d + 2], sd, c.z);
    }
  }
}

// VALU issue bounds this kernel (per evaluation 5 or 6 FP32 instructions and
// one exponential, about a sixth more for drawing the library's points).  Its
// registers are held to 64, for eight waves per SIMD: the more waves, the
// more often two of them stand at FP32 instructions that can be issued
// together (trans_group); a density loop alone measured 21.6, 24.3 and 28.2
// cycles per evaluation with eight, six and four waves.  On the 100,000 molecules
// of the performance cases (10-50 atoms, 30-atom query, SE(T) <= 0.005; bench.py's
// library takes 6.14e9 instructions and 7.8 ms): 8.07 ms with the exponentials
// among the other instructions (76 registers), 7.15 ms with them grouped, 7.07
// ms with the drawing steps of a lane's points grouped too, 7.00 ms with two
// atoms per LDS word, no remainder loop and three-way XORs (5.67e9 -> 5.52e9
// instructions); fixed 4,096 per side, 7,003 molecules: 0.60 -> 0.52 ms, and
// 0.49 ms with four rounds of a pair at a time (screen_shape).  Of
// 4-cycle issue slots left by the exponentials, 1.62 of 2 hold an instruction.
template <int kSA, int kSB, bool kAnti, int kRounds>
__global__ __launch_bounds__(kRounds * kWave)
__attribute__((amdgpu_waves_per_eu(kSA >= 8 ? 4 : 8)))
void k_screen(ScreenArgs a) {
  // No implicit multiply-add contraction: the fused operations are written
  // out, so every tile variant rounds identically.
#pragma clang fp contract(off)
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ float sTot[2][kRounds][8];  // the rounds' totals (two sets: one barrier per pass)
  const ScreenLds lds(smem, a.max_q, a.max_b);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = kRounds == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // grid = n_pairs; a launch order, when given, is a permutation of the pairs
  const int p = a.order ? a.order[blockIdx.x] : xcd_chunk(blockIdx.x, gridDim.x);
  if (p < 0 || p >= a.n_pairs) return;
  const int m = a.pairs ? a.pairs[p] : p;
  if (a.Q.bad[0] != 0 || m < 0 || m >= a.n_lib || a.L.bad[m] != 0) {
    screen_write_nan(a, p);
    return;
  }
  const int q0 = a.offQ[0], nq = a.offQ[1] - q0;
  const int b0 = a.offL[m], nb = a.offL[m + 1] - b0;
  lds.stage(a, m, q0, nq, b0, nb);
  const uint32_t idb = a.L.id[m];
  const int rs = a.round_side;
  const int per_lane = rs / kWave;
  const bool ragged = per_lane % kSA != 0 || per_lane % kSB != 0;
  RoundSums S;
  int64_t n_side = 0;
  int buf = 0;
  int take = 1;  // rounds of this pass
  if constexpr (kRounds > 1) {
    take = a.first_rounds;
    if (a.n_start && take < kRounds)
      take = max(take, screen_rounds_for(kRounds, (float)a.n_start[p] / (float)(2 * rs)));
  }
  for (;;) {
    SideSums<kAnti> A, B;
    const int n0 = (int)n_side + wave * rs;  // this wave's round, if the pair has it
    if (kRounds == 1 || (wave < take && n0 < screen_limit(screen_args_again()))) {
      // side A: query samples from the cache (query frame), partner = library
      for (int t = 0; t < per_lane; t += kSA) {
        float rx[kSA], ry[kSA], rz[kSA], r2[kSA], w[kSA], f2[kSA], q[kSA];
#pragma unroll
        for (int s = 0; s < kSA; ++s) {
          const int i = (t + s) < per_lane ? t + s : t;
          const int k = kAnti ? n0 + 2 * lane + 2 * kWave * (i >> 1) + (i & 1)
                              : n0 + lane + kWave * i;
          const float4 c = a.qs[k];
          rx[s] = c.x; ry[s] = c.y; rz[s] = c.z; w[s] = c.w;
          r2[s] = norm2(c.x, c.y, c.z);
          f2[s] = a.qf2[k];
          q[s] = 1.0f;
        }
        eval_union_x2<kSA>(lds.BA, nb, rx, ry, rz, r2, q);
#pragma unroll
        for (int s = 0; s < kSA; ++s) {
          if (ragged && t + s >= per_lane) w[s] = f2[s] = 0.0f;  // a slot past the round's last
          A.term(t + s, w[s] * (1.0f - q[s]), f2[s], 1.0f);
        }
      }
      // side B: library samples drawn here (library frame), partner = query
      for (int t = 0; t < per_lane; t += kSB) {
        float rx[kSB], ry[kSB], rz[kSB], r2[kSB], mb[kSB], qb[kSB], qa[kSB];
        screen_draw<kSB, kAnti>(lds, nb, idb, (uint32_t)n0, t, per_lane, a.key, rx, ry, rz);
#pragma unroll
        for (int s = 0; s < kSB; ++s) {
          r2[s] = norm2(rx[s], ry[s], rz[s]);
          mb[s] = 0.0f; qb[s] = 1.0f; qa[s] = 1.0f;
        }
        eval_density_x2<kSB>(lds.BB, nb, rx, ry, rz, r2, mb, qb);
        eval_union_x2<kSB>(lds.AB, nq, rx, ry, rz, r2, qa);
#pragma unroll
        for (int s = 0; s < kSB; ++s) {
          const float ub = 1.0f - qb[s];
          float w = bounded_weight(ub, mb[s]);
          if (ragged && t + s >= per_lane) w = 0.0f;
          B.term(t + s, w * (1.0f - qa[s]), w, ub);
        }
      }
    }
    const float v = RoundSums::totals(A.f, B.f);
    const ScreenArgs& r = screen_args_again();
    bool stop = false;
    if constexpr (kRounds == 1) {
      S.add(v);
      n_side += rs;
      stop = screen_stops(r, S, n_side, r.n_start ? (int64_t)r.n_start[p] : 0, kAnti, r.Q.Z[0],
                          r.L.Z[m]);
    } else {
      if (lane < 6) sTot[buf][wave][lane] = v;
      __syncthreads();
      const int64_t first_check = r.n_start ? (int64_t)r.n_start[p] : 0;
      for (int k = 0; k < take && !stop; ++k) {
        S.add(sTot[buf][k][lane < 6 ? lane : 5]);
        n_side += rs;
        stop = __builtin_amdgcn_readfirstlane(
            screen_stops(r, S, n_side, first_check, kAnti, r.Q.Z[0], r.L.Z[m]));
      }
      buf ^= 1;
      if (!stop && r.first_rounds < kRounds)
        take = __builtin_amdgcn_readfirstlane(screen_next(r, kRounds, S, n_side, first_check,
                                                          kAnti, r.Q.Z[0], r.L.Z[m]));
    }
    if (__builtin_amdgcn_readfirstlane(stop)) break;
  }
  const ScreenArgs& r = screen_args_again();
  screen_write(r, p, S, n_side, kAnti, r.Q.Z[0], r.L.Z[m]);
}

// The same screen with several waves per pair, for calls with too few pairs to
// fill the chip: two waves take two of a round's four slots each, of both
// sides, and a workgroup of eight works on four rounds at a time.  The waves
// write their slots' terms to LDS, one wave per round adds them in the order
// a single wave would have, and the rounds' totals enter the running sums,
// with the stop test after each, in turn: every output has k_screen's bits
// (rounds drawn past the stop are dropped, 1.5 of about twenty).
// Latency bounds such a screen (a pair's rounds are a chain): 501 molecules,
// SE(T) <= 0.005, 358 -> 112 us; one 277 -> 74 us.  One slot per wave (two
// LDS reads per term) 135 us, four slots 141 us, eight rounds at a time 144 us.
// With a few waves per SIMD the next records are read ahead: 110 -> 105 us (one
// molecule, 16,384 samples per side 129 -> 121).
constexpr int kSplitSlots = 4;  // rounds of 256 samples per side
constexpr int kSplitS = 2;      // slots per wave
constexpr int kSplitRounds = 4;
constexpr int kSplitTerms = 5;  // side A: f1, f2; side B: f1, w, u
constexpr int kSplitThreads = kSplitRounds * (kSplitSlots / kSplitS) * kWave;

template <bool kAnti>
__global__ __launch_bounds__(kSplitThreads) void k_screen_split(ScreenArgs a) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int S = kSplitS, kRoundWaves = kSplitSlots / S;
  __shared__ float sF[kSplitRounds][kSplitTerms][kSplitSlots][kWave];
  __shared__ float sTot[kSplitRounds][8];
  const ScreenLds lds(smem, a.max_q, a.max_b);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = wave / kRoundWaves, t = wave % kRoundWaves * S;  // this wave's round, first slot
  const int p = a.order ? a.order[blockIdx.x] : xcd_chunk(blockIdx.x, gridDim.x);
  if (p < 0 || p >= a.n_pairs) return;
  const int m = a.pairs ? a.pairs[p] : p;
  if (a.Q.bad[0] != 0 || m < 0 || m >= a.n_lib || a.L.bad[m] != 0) {
    screen_write_nan(a, p);
    return;
  }
  const int q0 = a.offQ[0], nq = a.offQ[1] - q0;
  const int b0 = a.offL[m], nb = a.offL[m + 1] - b0;
  lds.stage(a, m, q0, nq, b0, nb);
  const uint32_t idb = a.L.id[m];
  const double Za = a.Q.Z[0], Zb = a.L.Z[m];
  const int rs = kSplitSlots * kWave;
  const int limit = screen_limit(a);
  const int64_t first_check = a.n_start ? (int64_t)a.n_start[p] : 0;
  RoundSums sums;
  int64_t n_side = 0;
  for (bool stop = false; !stop;) {
    const int64_t n0 = n_side + (int64_t)g * rs;
    if (n0 < limit) {  // the last round is never past the samples asked for
      {
        float rx[S], ry[S], rz[S], r2[S], w[S], f2[S], q[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int i = t + s;
          const int k = kAnti ? (int)n0 + 2 * lane + 2 * kWave * (i >> 1) + (i & 1)
                              : (int)n0 + lane + kWave * i;
          const float4 c = a.qs[k];
          rx[s] = c.x; ry[s] = c.y; rz[s] = c.z; w[s] = c.w;
          r2[s] = norm2(c.x, c.y, c.z);
          f2[s] = a.qf2[k];
          q[s] = 1.0f;
        }
        eval_union_x2<S, true>(lds.BA, nb, rx, ry, rz, r2, q);
#pragma unroll
        for (int s = 0; s < S; ++s) {
          sF[g][0][t + s][lane] = w[s] * (1.0f - q[s]);
          sF[g][1][t + s][lane] = f2[s];
        }
      }
      {
        float rx[S], ry[S], rz[S], r2[S], mb[S], qb[S], qa[S];
        screen_draw<S, kAnti>(lds, nb, idb, (uint32_t)n0, t, kSplitSlots, a.key, rx, ry, rz);
#pragma unroll
        for (int s = 0; s < S; ++s) {
          r2[s] = norm2(rx[s], ry[s], rz[s]);
          mb[s] = 0.0f; qb[s] = 1.0f; qa[s] = 1.0f;
        }
        eval_density_x2<S, true>(lds.BB, nb, rx, ry, rz, r2, mb, qb);
        eval_union_x2<S, true>(lds.AB, nq, rx, ry, rz, r2, qa);
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float ub = 1.0f - qb[s];
          const float w = bounded_weight(ub, mb[s]);
          sF[g][2][t + s][lane] = w * (1.0f - qa[s]);
          sF[g][3][t + s][lane] = w;
          sF[g][4][t + s][lane] = ub;
        }
      }
    }
    __syncthreads();  // the rounds' terms
    if (wave < kSplitRounds) {
      SideSums<kAnti> A, B;
#pragma unroll
      for (int i = 0; i < kSplitSlots; ++i) {
        A.term(i, sF[wave][0][i][lane], sF[wave][1][i][lane], 1.0f);
        B.term(i, sF[wave][2][i][lane], sF[wave][3][i][lane], sF[wave][4][i][lane]);
      }
      const float v = RoundSums::totals(A.f, B.f);
      if (lane < 6) sTot[wave][lane] = v;
    }
    __syncthreads();  // the rounds' totals (and every read of their terms)
    for (int r = 0; r < kSplitRounds && !stop; ++r) {
      sums.add(sTot[r][lane < 6 ? lane : 5]);
      n_side += rs;
      stop = __builtin_amdgcn_readfirstlane(
          screen_stops(a, sums, n_side, first_check, kAnti, Za, Zb));
    }
  }
  if (wave == 0) screen_write(a, p, sums, n_side, kAnti, Za, Zb);
}

// ---------------------------------------------------------------------------
// Export of the sampling steps of one prepared molecule (section
// "Importance-sampling estimator": exact draws from the normalised mixture),
// for exact comparison of the integer steps: the molecule's thresholds, and
// for samples k0 .. k0+n-1 the Philox block, the selected component (binary
// lifting, as in the single-pair, query-cache, self-overlap and alignment kernels) and
// the point (its component through the guide table, as in the screening kernels),
// computed by the functions those kernels draw with (draws_of, draw_points), several
// samples per thread together as there.  kExportDraws samples per thread at a stride of
// the workgroup, past the end the last one again; one thread per atom for the
// thresholds; records from HBM.
// ---------------------------------------------------------------------------
constexpr int kExportThreads = 256;
constexpr int kExportDraws = 4;
__global__ __launch_bounds__(kExportThreads) void k_sample_points(
    Prepared P, const int* __restrict__ off, int mol, int64_t k0, int n, uint2 key, int anti,
    uint32_t* __restrict__ thr, uint32_t* __restrict__ words, int* __restrict__ comp,
    float* __restrict__ r) {
  constexpr int D = kExportDraws;
  __shared__ uint8_t guide[kGuideSize];  // the screening kernel's table, one entry per thread
  const int a0 = off[mol], na = off[mol + 1] - a0;
  const Atom* atoms = P.atom + a0;
  const AtomSampling* samp = P.samp + a0;
  const int64_t i0 = (int64_t)blockIdx.x * D * kExportThreads + threadIdx.x;
  if (thr)
    for (int d = 0; d < D; ++d)
      if (i0 + d * kExportThreads < na)
        thr[i0 + d * kExportThreads] = samp[i0 + d * kExportThreads].thr;
  build_guide(samp, na, guide, threadIdx.x, blockDim.x);
  __syncthreads();
  if (i0 >= n) return;
  int64_t i[D];
  uint4 x[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const int64_t at = i0 + d * kExportThreads;
    i[d] = at < n ? at : n - 1;
    const uint64_t k = (uint64_t)(k0 + i[d]);
    x[d] = philox_block(anti ? k >> 1 : k, P.id[mol], key);
  }
  int lifted[D], guided[D];
  float z[3 * D];
  draws_of<D>(x, [&](const uint32_t (&w)[D], int (&c)[D]) {
    select_components<D>(samp, na, w, c);
  }, lifted, z);
  draws_of<D>(x, [&](const uint32_t (&w)[D], int (&c)[D]) {
    select_components_guided<D>(samp, guide, na, w, c);
  }, guided, z);
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (words) reinterpret_cast<uint4*>(words)[i[d]] = x[d];
    if (comp) comp[i[d]] = lifted[d];
    if (r) {
      // another component than comp's would move the point far outside the bound of
      // its floating-point steps
      const int j[1] = {guided[d]};
      const float zd[3] = {z[3 * d], z[3 * d + 1], z[3 * d + 2]};
      const float sign = anti && ((k0 + i[d]) & 1) ? -1.0f : 1.0f;
      float rx[1], ry[1], rz[1];
      draw_points<1>(atoms, samp, j, zd, sign, rx, ry, rz);
      r[3 * i[d]] = rx[0];
      r[3 * i[d] + 1] = ry[0];
      r[3 * i[d] + 2] = rz[0];
    }
  }
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------
hipError_t launch_alpha_from_radius(const float* R, int64_t n, double kappa, double lambda,
                                    float* alpha, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(k_alpha_from_radius, dim3((unsigned)blocks), dim3(256), 0, st, R, n, kappa,
                     lambda, alpha);
  return hipGetLastError();
}

hipError_t launch_prepare(const MolsDev& in, const Prepared& out, int* flag, int* set_flag,
                          hipStream_t st, const int* which, int n_which) {
  const int n = which ? n_which : in.n_mols;
  if (n <= 0) return hipSuccess;
  const int blocks = (n + kPrepWaves - 1) / kPrepWaves;
  hipLaunchKernelGGL(k_prepare, dim3(blocks), dim3(256), 0, st, in, out, flag, set_flag, which,
                     n);
  return hipGetLastError();
}

hipError_t launch_flag_or(int* flag, const int* set_flag, hipStream_t st) {
  hipLaunchKernelGGL(k_flag_or, dim3(1), dim3(64), 0, st, flag, set_flag);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int n, int v, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_int, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

hipError_t launch_prepare_pair(const MolsDev& inA, const Prepared& A, const MolsDev& inB,
                               const Prepared& B, int* flag, hipStream_t st) {
  hipLaunchKernelGGL(k_prepare_pair, dim3(1), dim3(2 * kWave), 0, st, inA, A, inB, B, flag);
  return hipGetLastError();
}

// Terms per lane of the single-pair kernel: one while that still leaves at
// most four workgroups per compute unit and side, then four, then eight in
// two turns (which bounds the partial sums at 2,048 terms per block).
struct EstShape {
  int s, turns;
  int per_block() const { return 256 * s * turns; }
};
static EstShape est_shape(int64_t n_units) {
  if (n_units <= 256 * 1024) return {1, 1};
  if (n_units <= 1024 * 1024) return {4, 1};
  return {4, 2};
}

int est_blocks(int64_t n_units) {
  const int per = est_shape(n_units).per_block();
  return (int)((n_units + per - 1) / per);
}

template <int S>
static void launch_est_partials(const Prepared& A, const Prepared& B, const int* offA,
                                const int* offB, int64_t n_a, int64_t n_b, uint2 key, int anti,
                                int turns, double* partials, int nblk, hipStream_t st) {
  if (anti)
    hipLaunchKernelGGL((k_est_partials<S, true>), dim3(nblk, 2), dim3(256), 0, st, A, B, n_a, n_b,
                       key, turns, partials, nblk, offA, offB);
  else
    hipLaunchKernelGGL((k_est_partials<S, false>), dim3(nblk, 2), dim3(256), 0, st, A, B, n_a,
                       n_b, key, turns, partials, nblk, offA, offB);
}

hipError_t launch_estimate(const Prepared& A, const Prepared& B, const int* offA,
                           const int* offB, int64_t n_a, int64_t n_b, uint2 key, int anti,
                           double* partials, int nblk, EstOut* out, hipStream_t st) {
  const EstShape e = est_shape((n_a > n_b ? n_a : n_b) / (anti ? 2 : 1));
  if (e.s == 1)
    launch_est_partials<1>(A, B, offA, offB, n_a, n_b, key, anti, e.turns, partials, nblk, st);
  else
    launch_est_partials<4>(A, B, offA, offB, n_a, n_b, key, anti, e.turns, partials, nblk, st);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(k_est_finalize, dim3(1), dim3(kEstParts * 32), 0, st, partials, nblk, A, B, n_a, n_b,
                     anti, out);
  return hipGetLastError();
}

hipError_t launch_sample_points(const Prepared& P, const int* off, int mol, int max_atoms,
                               int64_t k0, int n, uint2 key, int anti, uint32_t* thr,
                               uint32_t* words, int* comp, float* r, hipStream_t st) {
  const int64_t items = n > max_atoms ? n : max_atoms;
  constexpr int kPer = kExportThreads * kExportDraws;
  hipLaunchKernelGGL(k_sample_points, dim3((unsigned)((items + kPer - 1) / kPer)),
                     dim3(kExportThreads), 0, st, P, off, mol, k0, n, key,
                     anti, thr, words, comp, r);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Launch order of a grid with one workgroup per pair: largest estimated work
// first.  A pair's result depends on that pair alone, so the order in which
// workgroups take the pairs changes no output; it changes how long the last
// workgroups run on after the others have finished.  The caller states the
// work of a pair in atoms' worth from its atom counts (B's, or their square,
// in a quadratic pass) and seeded budget;
// pairs are bucketed by its logarithm, 8 buckets per octave.  With per_xcd,
// each XCD keeps the pairs xcd_chunk deals it (so its L2 still sees whole
// tiles of consecutive molecules and output lines) and takes them largest
// first: block b = 8 r + x, the r-th block the round-robin dispatch sends to
// XCD x, takes the r-th pair of XCD x's order; otherwise block b takes the
// b-th largest.  A counting sort over (group, bucket) in three launches:
// kOrderBlocks blocks histogram their contiguous share of the pairs in LDS;
// one thread per bucket sums its counts over the blocks (prefix and total);
// the same blocks again, each after an LDS scan of the totals, place their
// pairs with LDS atomics (the order inside a bucket is not fixed).  Every
// slot is written on every call, so no memory needs clearing.
// ---------------------------------------------------------------------------
constexpr int kOrderKeys = 256;                    // work buckets per group
constexpr int kOrderBuckets = kXcds * kOrderKeys;  // (group, bucket) pairs
constexpr int kOrderBlocks = 64;
constexpr int kOrderThreads = 1024;

// XCD of the block that xcd_chunk maps to item p of a grid of G blocks:
// below F = G - G mod (8 kXcdTile) tile p / kXcdTile sits on XCD tile mod 8;
// blocks from F on keep their index, so block p runs on XCD p mod 8.
__device__ __forceinline__ int xcd_of_item(int p, int G) {
  const int F = G - G % (kXcds * kXcdTile);
  return p >= F ? p % kXcds : (p / kXcdTile) % kXcds;
}

__device__ __forceinline__ int atoms_of(const int* off, int m, int max_atoms) {
  const int n = off[m + 1] - off[m];
  return n < 0 ? 0 : (n > max_atoms ? max_atoms : n);
}

__device__ __forceinline__ int order_key(const OrderArgs& o, int p) {
  const int g = o.per_xcd ? xcd_of_item(p, o.n) : 0;
  const int m = o.pairs ? o.pairs[p] : p;
  if (m < 0 || m >= o.nB_mols) return g * kOrderKeys;  // an invalid pair only writes NaN
  const uint64_t nb = (uint64_t)atoms_of(o.offB, m, o.max_b);
  uint64_t cost = (uint64_t)o.wB * (o.quad_b ? nb * nb : nb) + o.w0;
  if (o.offA) {
    const int ma = o.a_single ? 0 : p;
    if (ma < o.nA_mols) cost += (uint64_t)o.wA * (uint64_t)atoms_of(o.offA, ma, o.max_a);
  }
  if (o.n_start) {
    const int64_t s = o.n_start[p];
    const int64_t r = s <= o.round_pair ? 1
                    : (s >= o.cap ? o.cap / o.round_pair
                                  : (s + o.round_pair - 1) / o.round_pair);
    cost *= (uint64_t)r;
  }
  const uint32_t c = cost == 0 ? 1u : (cost > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)cost);
  const int e = 31 - __clz(c);
  const uint32_t mant = e >= 3 ? (c >> (e - 3)) & 7u : (c << (3 - e)) & 7u;
  return g * kOrderKeys + 8 * e + (int)mant;  // 8 e + 7 < kOrderKeys
}

__device__ __forceinline__ void order_share(int n, int& begin, int& end) {
  const int64_t per = ((int64_t)n + kOrderBlocks - 1) / kOrderBlocks;
  begin = (int)min((int64_t)n, (int64_t)blockIdx.x * per);
  end = (int)min((int64_t)n, (int64_t)begin + per);
}

// hist[k][b]: pairs of block b's share with key k (bucket-major, so that
// the scan reads each bucket's counts as 16 consecutive 16-byte words)
template <int N>
__device__ __forceinline__ void order_hist(const OrderArgs& o, int* __restrict__ hist, int* h) {
  for (int k = threadIdx.x; k < kOrderBuckets; k += N) h[k] = 0;
  __syncthreads();
  int begin, end;
  order_share(o.n, begin, end);
  for (int64_t p = begin + (int64_t)threadIdx.x; p < end; p += N)
    atomicAdd(&h[order_key(o, (int)p)], 1);
  __syncthreads();
  for (int k = threadIdx.x; k < kOrderBuckets; k += N) hist[k * kOrderBlocks + blockIdx.x] = h[k];
}
__global__ __launch_bounds__(kOrderThreads) void k_order_hist(OrderArgs o,
                                                              int* __restrict__ hist) {
  __shared__ int h[kOrderBuckets];
  order_hist<kOrderThreads>(o, hist, h);
}

// The whole order of a short grid (per_xcd = 0) by one block of kOrderKeys
// threads, key k at thread k; h [kOrderKeys] in LDS.
__device__ __forceinline__ void order_short(const OrderArgs& o, int* __restrict__ order, int* h) {
  const int t = threadIdx.x;
  h[t] = 0;
  __syncthreads();
  for (int p = t; p < o.n; p += kOrderKeys) atomicAdd(&h[order_key(o, p)], 1);
  __syncthreads();
  const int mine = h[t];
  for (int d = 1; d < kOrderKeys; d <<= 1) {  // h[t] = pairs with keys >= t
    const int add = t + d < kOrderKeys ? h[t + d] : 0;
    __syncthreads();
    h[t] += add;
    __syncthreads();
  }
  h[t] -= mine;
  __syncthreads();
  for (int p = t; p < o.n; p += kOrderKeys) {
    int r = atomicAdd(&h[order_key(o, p)], 1);
    if (o.snake > 0 && (r / o.snake & 1)) {  // odd turns over the compute units backwards
      const int first = r / o.snake * o.snake;
      r = first + min(o.snake, o.n - first) - 1 - (r - first);
    }
    order[r] = p;
  }
}

// One thread per key k: replaces hist[k][b] by the number of pairs with key k
// in blocks before b, and writes the key's total to tot[k].  hist is 16-byte
// aligned.
constexpr int kOrderScanThreads = 64;
__device__ __forceinline__ void order_scan(int k, int* __restrict__ hist, int* __restrict__ tot) {
  constexpr int kVec = kOrderBlocks / 4;
  int4* row = reinterpret_cast<int4*>(hist + k * kOrderBlocks);
  int4 h[kVec];
#pragma unroll
  for (int i = 0; i < kVec; ++i) h[i] = row[i];
  int rank = 0;
#pragma unroll
  for (int i = 0; i < kVec; ++i) {
    int4 r;
    r.x = rank; rank += h[i].x;
    r.y = rank; rank += h[i].y;
    r.z = rank; rank += h[i].z;
    r.w = rank; rank += h[i].w;
    row[i] = r;
  }
  tot[k] = rank;
}
__global__ __launch_bounds__(kOrderScanThreads) void k_order_scan(int* __restrict__ hist,
                                                                 int* __restrict__ tot) {
  order_scan(blockIdx.x * kOrderScanThreads + threadIdx.x, hist, tot);
}

// Block b places its share: pair p with key k goes to rank
// (pairs of its group with larger keys) + (key-k pairs of earlier blocks) +
// (its arrival among block b's key-k pairs) of its group's order.
__global__ __launch_bounds__(kOrderThreads) void k_order_place(OrderArgs o,
                                                               const int* __restrict__ before,
                                                               const int* __restrict__ tot,
                                                               int* __restrict__ order) {
  constexpr int kPer = kOrderBuckets / kOrderThreads;
  __shared__ int cur[kOrderBuckets];
  int t[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int k = threadIdx.x + j * kOrderThreads;
    t[j] = tot[k];
    cur[k] = t[j];
  }
  __syncthreads();
  // suffix sums within each group's segment: cur[k] = its pairs with keys >= k
  for (int d = 1; d < kOrderKeys; d <<= 1) {
    int add[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int k = threadIdx.x + j * kOrderThreads;
      add[j] = (k % kOrderKeys) + d < kOrderKeys ? cur[k + d] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) cur[threadIdx.x + j * kOrderThreads] += add[j];
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int k = threadIdx.x + j * kOrderThreads;
    cur[k] += before[k * kOrderBlocks + blockIdx.x] - t[j];
  }
  __syncthreads();
  int begin, end;
  order_share(o.n, begin, end);
  const int groups = o.per_xcd ? kXcds : 1;
  for (int64_t p = begin + (int64_t)threadIdx.x; p < end; p += kOrderThreads) {
    const int key = order_key(o, (int)p);
    const int r = atomicAdd(&cur[key], 1);
    order[(int64_t)groups * r + key / kOrderKeys] = (int)p;
  }
}

int work_order_ints() { return kOrderBlocks * kOrderBuckets + kOrderBuckets; }

static hipError_t launch_order_place(const OrderArgs& o, int* order, int* work, hipStream_t st) {
  hipLaunchKernelGGL(k_order_place, dim3(kOrderBlocks), dim3(kOrderThreads), 0, st, o,
                     (const int*)work, (const int*)(work + kOrderBlocks * kOrderBuckets), order);
  return hipGetLastError();
}

hipError_t launch_work_order(const OrderArgs& o, int* order, int* work, hipStream_t st) {
  int* tot = work + kOrderBlocks * kOrderBuckets;
  hipLaunchKernelGGL(k_order_hist, dim3(kOrderBlocks), dim3(kOrderThreads), 0, st, o, work);
  hipLaunchKernelGGL(k_order_scan, dim3(kOrderBuckets / kOrderScanThreads),
                     dim3(kOrderScanThreads), 0, st, work, tot);
  return launch_order_place(o, order, work, st);
}

// ---------------------------------------------------------------------------
// The work before a screen or an alignment, in as few launches as its
// dependences allow (each takes 3 to 5 us in a stream, its work often less):
// both sets' preparation and the order's histograms, blocks of 256 threads of
// each in turn; then the query's sample cache and the order's scan.  A screen
// takes three launches before its kernel with an order and two without, instead
// of six and three (screen of 7,003 molecules, fixed: 497 -> 490 us; 300 pose
// gradients of 16 starts 180 -> 171).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_prepare_sets(PrepSet a, PrepSet b, int* __restrict__ flag,
                                                      OrderArgs o, int* __restrict__ hist,
                                                      int* __restrict__ order) {
  __shared__ int h[kOrderBuckets];
  int blk = blockIdx.x;
  if (hist) {  // the order's blocks come first
    if (blk < kOrderBlocks) {
      order_hist<256>(o, hist, h);
      return;
    }
    blk -= kOrderBlocks;
  } else if (order) {
    if (blk == 0) {
      order_short(o, order, h);
      return;
    }
    --blk;
  }
  const int blocks_a = (a.n + kPrepWaves - 1) / kPrepWaves;
  const bool first = blk < blocks_a;
  const PrepSet& s = first ? a : b;
  const int idx = (first ? blk : blk - blocks_a) * kPrepWaves + threadIdx.x / kWave;
  if (idx >= s.n) return;
  const int m = s.which ? s.which[idx] : idx;  // a listed index may repeat
  if (m < 0 || m >= s.in.n_mols) return;       // or lie outside: the screen flags it
  prepare_molecule(s.in, s.out, m, flag, nullptr);
}

__global__ __launch_bounds__(256) void k_query_cache(Prepared Qp, const int* __restrict__ offQ,
                                                     int64_t n, uint2 key, int anti,
                                                     float4* __restrict__ qs,
                                                     float* __restrict__ qf2, int scan_from,
                                                     int* __restrict__ hist,
                                                     int* __restrict__ tot) {
  if ((int)blockIdx.x >= scan_from)
    order_scan((blockIdx.x - scan_from) * 256 + threadIdx.x, hist, tot);
  else
    query_cache(Qp, offQ, n, key, anti, qs, qf2);
}

hipError_t launch_prepare_sets(const PrepSet& a, const PrepSet& b, int* flag, const OrderArgs* o,
                               int* work, int* order, hipStream_t st) {
  const int64_t blocks = ((int64_t)a.n + kPrepWaves - 1) / kPrepWaves +
                         ((int64_t)b.n + kPrepWaves - 1) / kPrepWaves +
                         (!o ? 0 : (work ? kOrderBlocks : 1));
  if (blocks == 0) return hipSuccess;
  if (prepare_apart(blocks, a.n, b.n)) {
    const PrepSet none{};
    const hipError_t e = launch_prepare_sets(a, none, flag, o, work, order, st);
    return e != hipSuccess ? e
                           : launch_prepare_sets(none, b, flag, nullptr, nullptr, nullptr, st);
  }
  hipLaunchKernelGGL(k_prepare_sets, dim3((unsigned)blocks), dim3(256), 0, st, a, b, flag,
                     o ? *o : OrderArgs{}, o ? work : nullptr, o ? order : nullptr);
  return hipGetLastError();
}

hipError_t launch_query_cache(const Prepared& Q, const int* offQ, int64_t n, uint2 key, int anti,
                              float4* qs, float* qf2, const OrderArgs* o, int* order, int* work,
                              hipStream_t st) {
  const int blocks = (int)((n + 255) / 256);
  hipLaunchKernelGGL(k_query_cache, dim3((unsigned)(blocks + (o ? kOrderBuckets / 256 : 0))),
                     dim3(256), 0, st, Q, offQ, n, key, anti, qs, qf2, blocks, work,
                     o ? work + kOrderBlocks * kOrderBuckets : nullptr);
  return o ? launch_order_place(*o, order, work, st) : hipGetLastError();
}

size_t screen_lds_bytes(int max_q, int max_b) {
  return (size_t)max_b * (sizeof(Atom) + sizeof(AtomSampling)) +
         (size_t)(2 * rec_pairs(max_b) + rec_pairs(max_q)) * sizeof(AtomRec2) +
         kGuideSize * sizeof(uint8_t);
}

template <int A, int B, int R = 1>
static void launch_screen_t(const ScreenArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)a.n_pairs), block(R * kWave);
  const size_t lds = screen_lds_bytes(a.max_q, a.max_b);
  if (a.anti)
    hipLaunchKernelGGL((k_screen<A, B, true, R>), grid, block, lds, st, a);
  else
    hipLaunchKernelGGL((k_screen<A, B, false, R>), grid, block, lds, st, a);
}

static hipError_t launch_screen_split(const ScreenArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)a.n_pairs), block(kSplitThreads);
  const size_t lds = screen_lds_bytes(a.max_q, a.max_b);
  if (a.anti)
    hipLaunchKernelGGL((k_screen_split<true>), grid, block, lds, st, a);
  else
    hipLaunchKernelGGL((k_screen_split<false>), grid, block, lds, st, a);
  return hipGetLastError();
}

hipError_t launch_screen(const ScreenArgs& a, int variant, hipStream_t st) {
  switch (variant) {
    case 0: launch_screen_t<4, 2>(a, st); break;
    case 1: launch_screen_t<2, 2>(a, st); break;
    case 2: launch_screen_t<4, 1>(a, st); break;
    case 3: launch_screen_t<4, 4>(a, st); break;
    case 4: launch_screen_t<8, 2>(a, st); break;
    case 5: launch_screen_t<2, 1>(a, st); break;
    case 6: launch_screen_t<8, 4>(a, st); break;
    case 7: launch_screen_t<2, 4>(a, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_screen_auto(const ScreenArgs& a, int variant, int n_cu, hipStream_t st) {
  if (a.round_side == kSplitSlots * kWave && a.n_pairs <= kSplitPairsPerCu * n_cu)
    return launch_screen_split(a, st);
  const bool adaptive = a.mode == SHAPE_SCREEN_ADAPTIVE;
  const int64_t n_rounds = (adaptive ? a.cap_pair / 2 : a.n_fixed) / a.round_side;
  const ScreenShape shape =
      screen_shape(adaptive, a.n_start != nullptr, a.n_pairs, n_rounds, a.expected, a.round_side,
                   (int64_t)screen_lds_bytes(a.max_q, a.max_b), n_cu);
  const int R = shape.rounds;
  ScreenArgs s = a;
  s.first_rounds = shape.first;
  const bool two = screen_points(a.round_side / kWave) == 2;
  if (R == 4)
    two ? launch_screen_t<2, 2, 4>(s, st) : launch_screen_t<4, 4, 4>(s, st);
  else if (R == 2)
    two ? launch_screen_t<2, 2, 2>(s, st) : launch_screen_t<4, 4, 2>(s, st);
  else
    return launch_screen(s, variant, st);
  return hipGetLastError();
}

}  // namespace shape
