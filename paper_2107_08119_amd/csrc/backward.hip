// Parameter gradient of an energy + force objective over a dataset (gfx950).
//
// For G(z) = sum_s gE_s E_s + sum_i gF_i . F_i, Sec. II A gives
// sum_i gF_i . F_i = -sum_a sum_nu dU_a/dq_nu delta q_a,nu with the
// directional derivative of the descriptor along gF,
//   delta q_a = sum_j (dq_a / dr_aj) . (gF_j - gF_a),
// so that, with x = tanh(a_mu), s = 1 - x^2, t_mu = sum_nu w1[mu][nu] delta q_nu
// and g_a = gE of atom a's structure (Eqs. nn1, nn2):
//   dG/dw1[mu][k] = w2_mu sum_a (alpha_a,mu q_a,k - s_a,mu delta q_a,k),
//   dG/db1[mu]    = -w2_mu sum_a alpha_a,mu,
//   dG/dw2[mu]    = sum_a beta_a,mu,
//   dG/db2        = -sum_a g_a,
// with alpha = s (g + 2 x t) and beta = g x - s t.
//
// k_grad_atoms evaluates q and delta q per atom (lanes split the neighbour
// slots, as in the force kernel; delta q uses the same factorised angular
// form) and writes (alpha, s, beta, q, delta q, g) per atom.  k_grad_contract
// sums them over the atoms of each wave in float64 on the matrix cores, and
// k_grad_final adds the blocks in order and applies the factors w2.
#include <algorithm>

#include "nep_terms.h"

namespace nep {
namespace {

inline unsigned blocks_for(size_t work, int block) { return (unsigned)((work + block - 1) / block); }

constexpr int kLanes = 4;
constexpr int kChunk = 16;      // atoms per step of a wave in the contraction
constexpr int kMaxBlocks = 256;  // its blocks: one per compute unit
// rows of the per-atom record: padded so that 16 atoms are read as float4
inline int rec_stride(int n) { return (n + kChunk - 1) / kChunk * kChunk; }

template <int NR, int NA, int LMAX, int NNEU>
struct GradLayout {
  static constexpr int NDES = NR + NA * LMAX;
  static constexpr int ALPHA = 0, S = NNEU, BETA = 2 * NNEU, Q = 3 * NNEU, DQ = 3 * NNEU + NDES,
                       G = 3 * NNEU + 2 * NDES, FIELDS = 3 * NNEU + 2 * NDES + 1;
};

// The derivatives of the 24 harmonics at the unit vector (x, y, z) along
// (tx, ty, tz), and the harmonics: Yhat_lm = Q_lm(z) Re or Im (x + i y)^m.
__device__ __forceinline__ void harmonics_along(float x, float y, float z, float tx, float ty,
                                                float tz, float (&yh)[24], float (&dy)[24]) {
  const float zz = z * z;
  const PlanePowers p = plane_powers(x, y);
  const ZFactors q = z_factors(z, zz);
  harmonics(x, y, z, yh);
  // of Re and Im (x + i y)^m: m (x + i y)^(m-1) (tx + i ty)
  const float a2 = 2.f * (x * tx - y * ty), b2 = 2.f * (x * ty + y * tx);
  const float a3 = 3.f * (p.a2 * tx - p.b2 * ty), b3 = 3.f * (p.a2 * ty + p.b2 * tx);
  const float a4 = 4.f * (p.a3 * tx - p.b3 * ty), b4 = 4.f * (p.a3 * ty + p.b3 * tx);
  dy[0] = tx, dy[1] = ty, dy[2] = tz;
  dy[5] = 3.f * z * tz, dy[11] = (7.5f * zz - 1.5f) * tz;
  dy[19] = z * (17.5f * zz - 7.5f) * tz;
  auto pair = [&](int re, int im, float q0, float dq, float pa, float pb, float da, float db) {
    dy[re] = dq * pa + q0 * da;
    dy[im] = dq * pb + q0 * db;
  };
  pair(6, 4, q.q21, NEP_S3 * tz, p.a1, p.b1, tx, ty);
  pair(12, 10, q.q31, 2.5f * NEP_S6 * z * tz, p.a1, p.b1, tx, ty);
  pair(20, 18, q.q41, (5.25f * NEP_S10 * zz - 0.75f * NEP_S10) * tz, p.a1, p.b1, tx, ty);
  pair(13, 9, q.q32, 0.5f * NEP_S15 * tz, p.a2, p.b2, a2, b2);
  pair(21, 17, q.q42, 3.5f * NEP_S5 * z * tz, p.a2, p.b2, a2, b2);
  pair(22, 16, q.q43, 0.25f * NEP_S70 * tz, p.a3, p.b3, a3, b3);
  dy[7] = q.q22 * a2, dy[3] = q.q22 * b2;
  dy[14] = q.q33 * a3, dy[8] = q.q33 * b3;
  dy[23] = q.q44 * a4, dy[15] = q.q44 * b4;
}

// Per atom: L lanes split the neighbour slots.  The displacements of the first
// kStage slots are formed once, several loads in flight, and kept in LDS for
// both passes.  Bound: the arithmetic of the two passes, latency below 8,000
// atoms.  The angular part of delta q, per pair and (n, l), is
//   2 g_n'(r) (u.D) sum_m c_nlm Yhat_lm + 2 g_n(r) sum_m c_nlm dYhat_lm
// with dYhat_lm the derivative along (D - u (u.D)) / r: 2 multiply-adds per
// (n, l, m) and one set of directional derivatives, where all three gradient
// components per harmonic and 3 per (n, l, m) took 54 us on 36,863 atoms, now 50
// (256 registers and 11 spilled, 48 bytes of scratch per lane: two waves per SIMD,
// the last 64 of 576 blocks after the rest).
// Eight lanes per atom take as long (49 us; 21 against 23 on 7,700 atoms).
constexpr int kStage = 40;
template <int NR, int NA, int LMAX, int NNEU, int L>
__global__ __launch_bounds__(kBlock, 2) void k_grad_atoms(
    int n, const double* __restrict__ pos, const uint32_t* __restrict__ nl,
    const int* __restrict__ cnt_r, const int* __restrict__ cnt_a,
    const double* __restrict__ boxes, const int* __restrict__ struct_of,
    const float* __restrict__ zpar, float rc_r, float rc_a, const double* __restrict__ gE,
    const float* __restrict__ gF, const float* __restrict__ F, double* __restrict__ gpos, int ld,
    float* __restrict__ rec) {
  using Lay = GradLayout<NR, NA, LMAX, NNEU>;
  constexpr int NLM = (LMAX + 1) * (LMAX + 1) - 1;
  constexpr int NDES = Lay::NDES;
  constexpr int NPAR = (NDES + 2) * NNEU + 1;
  __shared__ float sz[NPAR];
  for (int t = threadIdx.x; t < NPAR; t += blockDim.x) sz[t] = zpar[t];
  __syncthreads();
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int i = gid / L;
  const int lane = gid % L;
  const bool active = i < n;
  const int ii = active ? i : 0;
  const int cr = active ? cnt_r[i] : 0;
  const int ca = active ? cnt_a[i] : 0;
  const double xi = pos[ii], yi = pos[n + ii], zi = pos[2 * n + ii];
  const double* H = boxes + 9 * (size_t)struct_of[ii];
  const float rcr_inv = 1.f / rc_r, rca_inv = 1.f / rc_a;

  constexpr int KS = kStage, kBatch = 5;
  __shared__ float4 sd[KS][kBlock / L];  // displacement and, in .w, the neighbour
  const int la = threadIdx.x / L;
  const int staged = min(cr, KS);
  for (int s0 = lane; s0 < staged; s0 += L * kBatch) {
    uint32_t e[kBatch];
    double pj[kBatch][3];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) e[b] = nl[(size_t)min(s0 + b * L, staged - 1) * n + i];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int j = (int)(e[b] & kAtomMask);
      pj[b][0] = pos[j];
      pj[b][1] = pos[n + j];
      pj[b][2] = pos[2 * n + j];
    }
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      if (s0 + b * L >= staged) break;
      float dx, dy, dz;
      image_displacement(e[b], pj[b][0], pj[b][1], pj[b][2], xi, yi, zi, H, dx, dy, dz);
      sd[s0 + b * L][la] = make_float4(dx, dy, dz, __int_as_float((int)(e[b] & kAtomMask)));
    }
  }
  // a lane reads back only the entries it wrote
  auto pair = [&](int s, int& j, float& dx, float& dy, float& dz) {
    if (s < KS) {
      const float4 v = sd[s][la];
      dx = v.x;
      dy = v.y;
      dz = v.z;
      j = __float_as_int(v.w);
    } else {
      displacement(nl[(size_t)s * n + i], pos, n, xi, yi, zi, H, j, dx, dy, dz);
    }
  };

  const float rcr2 = rc_r * rc_r, rca2 = rc_a * rc_a;
  float q[NDES];
  float c[NA][NLM];
#pragma unroll
  for (int v = 0; v < NDES; ++v) q[v] = 0.f;
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int m = 0; m < NLM; ++m) c[a][m] = 0.f;
  for (int s = lane; s < cr; s += L) {
    int j;
    float dx, dy, dz;
    pair(s, j, dx, dy, dz);
    const float r2 = pair_r2(dx, dy, dz);
    pair_descriptor<NR, NA, LMAX>(dx, dy, dz, r2 < rcr2, s < ca && r2 < rca2, rcr_inv, rca_inv, q,
                                  c);
  }
#pragma unroll
  for (int a = 0; a < NR; ++a) q[a] = group_sum<L>(q[a]);
  radial_finish<NR>(q);
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int m = 0; m < NLM; ++m) c[a][m] = group_sum<L>(c[a][m]);
  angular_invariants<NR, NA, LMAX>(c, q);

  // delta q: directional derivative of the descriptor along gF
  float dq[NDES];
#pragma unroll
  for (int v = 0; v < NDES; ++v) dq[v] = 0.f;
  if (gF) {
    const float gxi = gF[ii], gyi = gF[n + ii], gzi = gF[2 * n + ii];
    int j = 0;
    float dx = 1.f, dy = 0.f, dz = 0.f, ax = 0.f, ay = 0.f, az = 0.f;
    auto fetch = [&](int s) {  // pair s and gF of its neighbour, one slot ahead
      pair(s, j, dx, dy, dz);
      ax = gF[j];
      ay = gF[n + j];
      az = gF[2 * n + j];
    };
    if (lane < cr) fetch(lane);
    for (int s = lane; s < cr; s += L) {
      const float r2 = pair_r2(dx, dy, dz);
      const float rinv = __builtin_amdgcn_rsqf(r2);
      const float r = r2 * rinv;
      const float x = dx * rinv, y = dy * rinv, z = dz * rinv;
      const float Dx = ax - gxi, Dy = ay - gyi, Dz = az - gzi;
      if (s + L < cr) fetch(s + L);
      const float uD = x * Dx + y * Dy + z * Dz;
      if (r2 < rcr2) {
        float g[NR], dg[NR];
        radial_basis<NR, true>(r, rcr_inv, g, dg);
#pragma unroll
        for (int a = 0; a < NR; ++a) dq[a] += dg[a] * uD;
      }
      if (s < ca && r2 < rca2) {
        float g[NA], dg[NA], yh[24], dyh[24];
        radial_basis<NA, true>(r, rca_inv, g, dg);
        harmonics_along(x, y, z, (Dx - x * uD) * rinv, (Dy - y * uD) * rinv, (Dz - z * uD) * rinv,
                        yh, dyh);
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          const float gy = 2.f * dg[a] * uD, gd = 2.f * g[a];
#pragma unroll
          for (int l = 1; l <= LMAX; ++l) {
            float sy = 0.f, sd2 = 0.f;
#pragma unroll
            for (int m = l * l - 1; m < (l + 1) * (l + 1) - 1; ++m) {
              sy += c[a][m] * yh[m];
              sd2 += c[a][m] * dyh[m];
            }
            dq[NR + a * LMAX + (l - 1)] += gy * sy + gd * sd2;
          }
        }
      }
    }
#pragma unroll
    for (int v = 0; v < NDES; ++v) dq[v] = group_sum<L>(dq[v]);
  }

  // network quantities per neuron (neurons split over the lanes)
  const float* w1 = sz;
  const float* b1 = sz + NNEU * NDES;
  const float ga = (active && gE) ? (float)gE[struct_of[i]] : 0.f;
  if (gpos && active && lane < 3) {  // energy part of the position gradient, -gE F
    const size_t t = (size_t)lane * n + i;
    gpos[t] = gE ? -gE[struct_of[i]] * (double)F[t] : 0.0;
  }
  if (active) {
    for (int mu = lane; mu < NNEU; mu += L) {
      float act = -b1[mu], t = 0.f;
#pragma unroll
      for (int v = 0; v < NDES; ++v) {
        act += w1[mu * NDES + v] * q[v];
        t += w1[mu * NDES + v] * dq[v];
      }
      const float ea = __expf(-2.f * fabsf(act));
      const float inv = __builtin_amdgcn_rcpf(1.f + ea);
      const float xm = copysignf((1.f - ea) * inv, act);
      const float sm = 4.f * ea * inv * inv;
      rec[(size_t)(Lay::ALPHA + mu) * ld + i] = sm * (ga + 2.f * xm * t);
      rec[(size_t)(Lay::S + mu) * ld + i] = sm;
      rec[(size_t)(Lay::BETA + mu) * ld + i] = ga * xm - sm * t;
    }
    for (int v = lane; v < NDES; v += L) {
      rec[(size_t)(Lay::Q + v) * ld + i] = q[v];
      rec[(size_t)(Lay::DQ + v) * ld + i] = dq[v];
    }
    if (lane == 0) rec[(size_t)Lay::G * ld + i] = ga;
  }
}

// out[block][N_par] = sums over the block's atoms, float64:
//   w1 (mu, k): alpha_mu q_k - s_mu dq_k;  b1: alpha_mu;  w2: beta_mu;  b2: g.
// Bound: the read of the records (596 bytes per atom).  The w1 sums are two
// products of 30 x atoms and atoms x 29 matrices, done by 16x16x4 float64
// MFMA steps: a lane reads four consecutive atoms of its row as one float4
// (the K step e takes atom 4 (l/16) + e), converts them, and keeps 2 x 2 tiles
// for all its atoms; column 29 of the second operand is 1, so that it collects
// the b1 sums.  The grid is at most one block per compute unit, each striding
// over the atoms, so k_grad_final adds 256 partial gradients at most.  With
// one thread per parameter over 64-atom blocks and 576 partial gradients this
// took 59 us, and adding them in one chain per parameter 145 us, on 36,863
// atoms; now 11 and 4 us.
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <int NR, int NA, int LMAX, int NNEU>
__global__ __launch_bounds__(kBlock) void k_grad_contract(int n, int ld,
                                                          const float* __restrict__ rec,
                                                          double* __restrict__ out) {
  using Lay = GradLayout<NR, NA, LMAX, NNEU>;
  constexpr int NDES = Lay::NDES;
  constexpr int NPAR = (NDES + 2) * NNEU + 1;
  static_assert(NNEU <= 32 && NDES < 32, "two 16-wide tiles, one column spare");
  constexpr int kW = kBlock / 64;
  __shared__ double tile[kW][32][33];
  __shared__ double side[kW][33];  // beta sums per neuron, then the g sum
  const int w = threadIdx.x / 64, l = threadIdx.x & 63, col = l & 15, h = l >> 4;
  f64x4 acc[2][2];
  double beta[2] = {0.0, 0.0}, gsum = 0.0;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int u = 0; u < 2; ++u) acc[t][u] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int chunks = (n + kChunk - 1) / kChunk;
  for (int c = blockIdx.x * kW + w; c < chunks; c += gridDim.x * kW) {
    const int a0 = c * kChunk + 4 * h;  // the lane's four atoms
    auto rows = [&](int field, int row, int last) {
      return *reinterpret_cast<const float4*>(rec + (size_t)(field + min(row, last)) * ld + a0);
    };
    float4 v[2][5];
    const float4 g4 = rows(Lay::G, 0, 0);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int r = 16 * t + col;  // neuron row and descriptor column of the lane
      v[t][0] = rows(Lay::ALPHA, r, NNEU - 1);
      v[t][1] = rows(Lay::S, r, NNEU - 1);
      v[t][2] = rows(Lay::BETA, r, NNEU - 1);
      v[t][3] = rows(Lay::Q, r, NDES - 1);
      v[t][4] = rows(Lay::DQ, r, NDES - 1);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = a0 + e < n;  // the padding of the rows is never written
      auto at = [&](const float4& x) {
        const float y = e == 0 ? x.x : (e == 1 ? x.y : (e == 2 ? x.z : x.w));
        return in ? (double)y : 0.0;
      };
      double alpha[2], s[2], q[2], dq[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int k = 16 * t + col;
        alpha[t] = at(v[t][0]);
        s[t] = -at(v[t][1]);
        beta[t] += at(v[t][2]);
        q[t] = k < NDES ? at(v[t][3]) : (k == NDES && in ? 1.0 : 0.0);
        dq[t] = k < NDES ? at(v[t][4]) : 0.0;
      }
      gsum += at(g4);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          acc[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(alpha[t], q[u], acc[t][u], 0, 0, 0);
          acc[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(s[t], dq[u], acc[t][u], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) tile[w][16 * t + 4 * r + h][16 * u + col] = acc[t][u][r];
#pragma unroll
  for (int d = 16; d < 64; d <<= 1) {  // the four atom groups of the wave
    beta[0] += __shfl_xor(beta[0], d, 64);
    beta[1] += __shfl_xor(beta[1], d, 64);
    gsum += __shfl_xor(gsum, d, 64);
  }
  if (h == 0) {
    side[w][col] = beta[0];
    side[w][16 + col] = beta[1];
    if (col == 0) side[w][32] = gsum;
  }
  __syncthreads();
  for (int p = threadIdx.x; p < NPAR; p += kBlock) {
    double s = 0.0;
    for (int u = 0; u < kW; ++u) {
      if (p < NNEU * NDES)
        s += tile[u][p / NDES][p % NDES];
      else if (p < NNEU * (NDES + 1))
        s += tile[u][p - NNEU * NDES][NDES];
      else
        s += p < NPAR - 1 ? side[u][p - NNEU * (NDES + 1)] : side[u][32];
    }
    out[(size_t)blockIdx.x * NPAR + p] = s;
  }
}

// grad[p] = factor_p sum_b part[b][p]: 64 parameters per block, 16 threads per
// parameter over consecutive runs of partial gradients, then the runs in order.
template <int NDES, int NNEU>
__global__ __launch_bounds__(1024) void k_grad_final(int nblocks, const float* __restrict__ zpar,
                                                     const double* __restrict__ part,
                                                     double* __restrict__ grad,
                                                     float* __restrict__ grad32) {
  constexpr int NPAR = (NDES + 2) * NNEU + 1;
  __shared__ double run[16][64];
  const int pl = threadIdx.x & 63, u = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + pl;
  const int len = (nblocks + 15) / 16, b1 = min(nblocks, (u + 1) * len);
  double s = 0.0;
  if (p < NPAR)
#pragma unroll 8
    for (int b = u * len; b < b1; ++b) s += part[(size_t)b * NPAR + p];
  run[u][pl] = s;
  __syncthreads();
  if (u != 0 || p >= NPAR) return;
  for (int t = 1; t < 16; ++t) s += run[t][pl];
  const float* w2 = zpar + NNEU * (NDES + 1);
  if (p < NNEU * NDES)
    s *= (double)w2[p / NDES];
  else if (p < NNEU * (NDES + 1))
    s *= -(double)w2[p - NNEU * NDES];
  else if (p == NPAR - 1)
    s = -s;
  grad[p] = s;
  if (grad32) grad32[p] = (float)s;
}

// gpos[c][i] = -gE F of the atom's structure, 0 without gE.
__global__ __launch_bounds__(kBlock) void k_position_gradient(
    int n, const int* __restrict__ struct_of, const double* __restrict__ gE,
    const float* __restrict__ F, double* __restrict__ gpos) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double g = gE ? -gE[struct_of[i]] : 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c)
    gpos[(size_t)c * n + i] = gE ? g * (double)F[(size_t)c * n + i] : 0.0;
}

}  // namespace

hipError_t launch_position_gradient(nep_ctx ctx, nep_dataset ds, const double* gE, const float* F,
                                    double* gpos) {
  launch_kernel(ctx, true, true, k_position_gradient, dim3(blocks_for(ds->N, kBlock)),
                dim3(kBlock), ds->N, (const int*)ds->struct_of.ptr, gE, F, gpos);
  return hipGetLastError();
}

hipError_t launch_backward(nep_ctx ctx, nep_dataset ds, const float* z, const double* gE,
                           const float* gF, const float* F, double* gpos, double* grad,
                           float* grad32) {
  using Lay = GradLayout<9, 5, 4, 30>;
  const int N = ds->N;
  constexpr int NPAR = (Lay::NDES + 2) * 30 + 1;
  const int ld = rec_stride(N);
  const unsigned nblk =
      std::min((unsigned)kMaxBlocks, blocks_for((size_t)N, kChunk * (kBlock / 64)));
  hipError_t e = ds->grad_rec.ensure((size_t)Lay::FIELDS * ld);
  if (e == hipSuccess) e = ds->grad_part.ensure((size_t)nblk * NPAR);
  if (e != hipSuccess) return e;
  launch_kernel(ctx, true, false, k_grad_atoms<9, 5, 4, 30, kLanes>,
                dim3(blocks_for((size_t)N * kLanes, kBlock)), dim3(kBlock), N,
                (const double*)ds->pos.ptr, (const uint32_t*)ds->nl.ptr, (const int*)ds->cnt_r.ptr,
                (const int*)ds->cnt_a.ptr, (const double*)ds->boxes.ptr,
                (const int*)ds->struct_of.ptr, z, (float)ctx->hyper.rc_radial,
                (float)ctx->hyper.rc_angular, gE, gF, F, gpos, ld, ds->grad_rec.ptr);
  launch_kernel(ctx, false, false, k_grad_contract<9, 5, 4, 30>, dim3(nblk), dim3(kBlock), N, ld,
                (const float*)ds->grad_rec.ptr, ds->grad_part.ptr);
  launch_kernel(ctx, false, true, k_grad_final<Lay::NDES, 30>, dim3(blocks_for(NPAR, 64)),
                dim3(1024), (int)nblk, z, (const double*)ds->grad_part.ptr, grad, grad32);
  return hipGetLastError();
}

}  // namespace nep
