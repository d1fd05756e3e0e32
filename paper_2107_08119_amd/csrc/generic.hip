// Pass 1 for any model size within n_max^R, n_max^A <= 15, l_max <= 4 and
// at most 64 hidden neurons (the paper's models of Sec. III, e.g. 80-50-1):
// blocks of four waves with four atoms per wave, 16 lanes each, or in small
// systems one atom per wave.
//
// The terms are those of nep_terms.h (factorised angular descriptor, network,
// partial force of Sec. II D):
//   * staging: the block reads the list and reverse slots of its atoms, 48
//     (with one atom per wave 64) slots at a time with atoms fastest, classifies
//     the pairs and packs those inside a cutoff per atom in LDS, angular ones
//     first; the pair vectors r_ij go to the atom's own slots for pass 2 (systems
//     of up to kPairVectorMaxAtoms atoms);
//   * radial q_n: each lane adds f_c T_n of its pairs, the atom's lanes are
//     summed in a fixed order, q_n = (R_n + R_0)/2 (g_n = f_c (T_n + 1)/2);
//   * angular moments c_nlm = sum_j g_n(r_ij) Yhat_lm(u_ij): per atom the
//     product (n x pairs)(pairs x lm) as 16x16x4 MFMA steps, the operands
//     passed through LDS; the sums stay in registers;
//   * network: W1 Q^T and W1^T G for the block's atoms on the matrix cores,
//     a wave per 16 neurons and per 16 descriptor components;
//   * partial forces: lane p evaluates pair p of its atom; the sums over n of
//     a_nlm (T_n + 1) and a_nlm T_n' for all lm are two more products per 16
//     pairs, with a_nlm = 2 dU/dq_nl c_nlm formed where c_nlm lies.
// Every sum has a fixed order, so results are reproducible bit for bit.
//
// Bound: the VALU work per pair (geometry, Chebyshev recursions, harmonics
// and their gradients, about 700 instructions for both loops) and, where an
// atom has few angular pairs, the loads and stores of the list slots.  One
// wave per atom, with the contractions on the VALU from LDS, left most lanes
// idle where an atom has fewer than 64 pairs (6 angular ones in PbTe): 63.0
// against 27.4 us for 80-50-1 on 8,000 atoms, 527 against 213 us for PbTe on
// 64,000 atoms.  Two blocks fit a compute unit: 76,160 bytes of LDS and 187
// registers for 80-50-1, 70,848 bytes and 256 registers (4 spilled) for PbTe; the
// runtime-sized float64 kernel with four atoms per wave takes 86,208 bytes, one
// block per unit (34-24-1 with two species on 64,000 atoms 414 us, with one wave
// per atom 1,538 us).
//
// Multicomponent systems take the descriptor and the hidden layer's input in
// float64 (pair geometry, basis, harmonics, the sums q and c_nlm, and the
// pre-activations with tanh and sech^2): the pair weights sqrt(Z_i Z_j) (up to
// 82) scale the descriptor up by about two orders, unscaled input weights then
// put pre-activations in the hundreds, and sech^2 there changes relatively by
// twice any absolute error of the pre-activation, which float32 sums make about
// 1e-5.  The partial forces stay float32.
#include <type_traits>

#include "nep_terms.h"

namespace nep {
namespace {

// Largest sizes of the runtime-sized instantiation.
constexpr int kMaxR = 16, kMaxA = 16, kMaxNeu = 64;
constexpr int kWaves = 4;  // per block
// Sizes of one instantiation: TR > 0 fixes (n_max^R + 1, n_max^A + 1, l_max,
// N_neu) = (TR, TA, TL, TNEU) at compile time (loops unrolled, LDS sized to
// the model); TR == 0 takes them at run time up to the maxima above.
template <int TR, int TA, int TL, int TNEU>
struct Shape {
  static constexpr bool kFixed = TR > 0;
  static constexpr int MR = kFixed ? TR : kMaxR;
  static constexpr int MA = kFixed ? TA : kMaxA;
  static constexpr int ML = kFixed ? TL : 4;
  static constexpr int MNEU = kFixed ? TNEU : kMaxNeu;
  static constexpr int MDES = MR + MA * ML;
  // A lane of lane group h = lane / 16 holds the moments n = RPL h + r, r < RPL.
  static constexpr int RPL = MA > 8 ? 4 : 2;
  static constexpr int KT = (MDES + 15) / 16;  // 16-wide tiles of the descriptor
  static constexpr int QS = 16 * KT + 4;       // LDS row of an atom's descriptor
  static constexpr int NT = (MNEU + 15) / 16;  // 16-wide tiles of the hidden layer
  static constexpr int GS = 16 * NT + 4;       // LDS row of an atom's w2 sech^2
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// One 16x16x4 step: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16].
// Element r of lane l is C[mma_row(l / 16, r)][l % 16].
__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4 mma(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Row i of A goes to element r of lane group h in C: i = 4 h + r in float32,
// 4 r + h in float64.  A supplies in row i whatever lane (h, r) is to hold.
template <class DT>
__device__ __forceinline__ void mma_owner(int i, int& h, int& r) {
  h = sizeof(DT) == 8 ? i & 3 : i >> 2;
  r = sizeof(DT) == 8 ? i >> 2 : i & 3;
}

// Sum over the L lanes of an atom in a fixed order; every lane gets the same
// bits (each step adds two partial sums, which commutes exactly).
template <int L>
__device__ __forceinline__ float atom_sum(float v) {
  v = group_sum<16>(v);
#pragma unroll
  for (int d = 16; d < L; d <<= 1) v += __shfl_xor(v, d, 64);
  return v;
}
template <int L>
__device__ __forceinline__ double atom_sum(double v) {
#pragma unroll
  for (int d = 1; d < L; d <<= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// l of harmonic index lm = l^2 - 1 + (m + l)
__device__ __forceinline__ int l_of(int lm) { return lm < 3 ? 1 : (lm < 8 ? 2 : (lm < 15 ? 3 : 4)); }

// r_ij of list entry e in float64, rounded exactly as the float32
// displacement is before its final rounding (so the two agree to float32).
__device__ __forceinline__ void image_displacement_d(uint32_t e, const double (&pj)[3], double xi,
                                                     double yi, double zi, const double* h,
                                                     double& dx, double& dy, double& dz) {
  int n0, n1, n2;
  unpack_image(e, n0, n1, n2);
  const double a0 = (double)n0, a1 = (double)n1, a2 = (double)n2;
  dx = (pj[0] - xi) + (a0 * h[0] + a1 * h[3] + a2 * h[6]);
  dy = (pj[1] - yi) + (a0 * h[1] + a1 * h[4] + a2 * h[7]);
  dz = (pj[2] - zi) + (a0 * h[2] + a1 * h[5] + a2 * h[8]);
}

constexpr double kPiD = 3.14159265358979323846;

// cos(pi t) for t near [0, 1] as -sin(y), y = pi (t - 1/2), from the Taylor
// series of sin through y^21 (for |y| <= pi/2 the first omitted term is below
// 2e-18, under float64 rounding).
__device__ __forceinline__ double cos_pi_unit(double t) {
  const double y = kPiD * (t - 0.5);
  const double y2 = y * y;
  double p = 1.0 / 51090942171709440000.0;  // 1/21!
  p = p * y2 - 1.0 / 121645100408832000.0;  // 1/19!
  p = p * y2 + 1.0 / 355687428096000.0;     // 1/17!
  p = p * y2 - 1.0 / 1307674368000.0;       // 1/15!
  p = p * y2 + 1.0 / 6227020800.0;          // 1/13!
  p = p * y2 - 1.0 / 39916800.0;            // 1/11!
  p = p * y2 + 1.0 / 362880.0;              // 1/9!
  p = p * y2 - 1.0 / 5040.0;                // 1/7!
  p = p * y2 + 1.0 / 120.0;                 // 1/5!
  p = p * y2 - 1.0 / 6.0;                   // 1/3!
  p = p * y2 + 1.0;
  return -y * p;
}

// f_c(r) = (1 + cos(pi r/r_c))/2 and T_n(x), x = 2 (r/r_c - 1)^2 - 1, n < NB,
// in float64: the factors of g_n = f_c (T_n + 1)/2 (Eq. g_n).
template <int NB>
__device__ __forceinline__ void chebyshev_values_d(double r, double rc_inv, double& fc, double* T) {
  const double t = r * rc_inv;
  fc = 0.5 * (1.0 + cos_pi_unit(t));
  const double tm1 = t - 1.0;
  const double x = 2.0 * tm1 * tm1 - 1.0;
  T[0] = 1.0;
  if constexpr (NB > 1) T[1] = x;
#pragma unroll
  for (int k = 2; k < NB; ++k) T[k] = 2.0 * x * T[k - 1] - T[k - 2];
}

// g_n(r), n < nb (<= MB), zero beyond, in float64.
template <int MB>
__device__ __forceinline__ void radial_basis_d(double r, double rc_inv, int nb, double* g) {
  double fc, T[MB];
  chebyshev_values_d<MB>(r, rc_inv, fc, T);
#pragma unroll
  for (int k = 0; k < MB; ++k) g[k] = k < nb ? 0.5 * (T[k] + 1.0) * fc : 0.0;
}

// The 24 harmonics Yhat_lm (l = 1..4) in float64: the same polynomials, with
// the square roots in their float64 values.
#pragma push_macro("NEP_S3")
#pragma push_macro("NEP_S5")
#pragma push_macro("NEP_S6")
#pragma push_macro("NEP_S10")
#pragma push_macro("NEP_S15")
#pragma push_macro("NEP_S35")
#pragma push_macro("NEP_S70")
#undef NEP_S3
#undef NEP_S5
#undef NEP_S6
#undef NEP_S10
#undef NEP_S15
#undef NEP_S35
#undef NEP_S70
#define NEP_S3 1.7320508075688772935
#define NEP_S5 2.2360679774997896964
#define NEP_S6 2.4494897427831780982
#define NEP_S10 3.1622776601683793320
#define NEP_S15 3.8729833462074168852
#define NEP_S35 5.9160797830996160426
#define NEP_S70 8.3666002653407554798
__device__ __forceinline__ void harmonics_d(double x, double y, double z, double (&out)[24]) {
  const double xx = x * x, yy = y * y, zz = z * z, xy = x * y, xz = x * z, yz = y * z;
  const double xyz = xy * z;
  (void)xyz;
#define NEP_Y(idx, YV, GX, GY, GZ) out[idx] = (YV);
  NEP_YLM_TABLE(NEP_Y)
#undef NEP_Y
}
#pragma pop_macro("NEP_S70")
#pragma pop_macro("NEP_S35")
#pragma pop_macro("NEP_S15")
#pragma pop_macro("NEP_S10")
#pragma pop_macro("NEP_S6")
#pragma pop_macro("NEP_S5")
#pragma pop_macro("NEP_S3")

// Radial basis g_n, n < nb (<= MB), zero beyond.
template <int MB>
__device__ __forceinline__ void radial_basis_n(float r, float rc_inv, int nb, float* g) {
  radial_basis<MB, false>(r, rc_inv, g, nullptr);
#pragma unroll
  for (int n = 0; n < MB; ++n) g[n] = n < nb ? g[n] : 0.f;
}

// F64: the float64 descriptor and hidden-layer input of multicomponent
// systems (wspd = sqrt(Z) in float64 beside wsp).
// AW: atoms per wave, 64 / AW lanes each.
template <int TR, int TA, int TL, int TNEU, bool F64, int AW>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(F64 && TR == 0 && AW > 1 ? 1 : 2))) void k_partials_generic(
    int n, const double* __restrict__ pos, const uint32_t* __restrict__ nl,
    const int* __restrict__ cnt_r, const int* __restrict__ cnt_a, const int* __restrict__ rev,
    Box box, const float* __restrict__ z, int nr_rt, int na_rt, int lmax_rt, int nneu_rt,
    double rc_rd, double rc_ad, const double* __restrict__ wspd, const int* __restrict__ perm,
    Partial3* __restrict__ pin, float* __restrict__ fown, float* __restrict__ U,
    Partial3* __restrict__ geo) {
  using S = Shape<TR, TA, TL, TNEU>;
  using DT = typename std::conditional<F64, double, float>::type;
  using D4 = typename std::conditional<F64, f64x4, f32x4>::type;
  constexpr int MR = S::MR, MA = S::MA, RPL = S::RPL, KT = S::KT, QS = S::QS, NT = S::NT,
                GS = S::GS;
  constexpr int L = 64 / AW;            // lanes per atom
  constexpr int kAtoms = kWaves * AW;   // per block
  // List slots per atom staged at a time: with 16 lanes per atom most lists with
  // a 0.5 A skin fit at once, longer ones (80 slots in PbTe) take further rounds.
  constexpr int W = 64 * kWaves / kAtoms;  // slots staged side by side
  constexpr int T = W >= 48 ? 1 : 48 / W;  // slots per thread
  constexpr int kSlots = W * T;
  constexpr int kRow = kSlots + 1;  // LDS row of an atom's pairs (odd: no bank aliasing)
  static_assert(kSlots <= 64, "slot masks");
  const float rc_r = (float)rc_rd, rc_a = (float)rc_ad;
  const int NR = S::kFixed ? TR : nr_rt;
  const int NA = S::kFixed ? TA : na_rt;
  const int LMAX = S::kFixed ? TL : lmax_rt;
  const int NNEU = S::kFixed ? TNEU : nneu_rt;
  const int NLM = (LMAX + 1) * (LMAX + 1) - 1;
  const int NDES = NR + NA * LMAX;

  // staged pairs of the block's atoms: r_ij and the index of the reverse slot
  __shared__ float4 s_pair[F64 ? 1 : kAtoms][F64 ? 1 : kRow];
  __shared__ double s_d[F64 ? 4 : 1][F64 ? kAtoms : 1][F64 ? kRow : 1];  // x, y, z, sqrt(Z_j)
  __shared__ int s_dst[F64 ? kAtoms : 1][F64 ? kRow : 1];
  __shared__ unsigned long long s_mask[2][kAtoms];  // slots of the two pair classes
  __shared__ int s_count[2][kAtoms];                // staged angular pairs, staged pairs
  // Operands of the per-atom products, one buffer per wave.  HB pairs of each
  // of the wave's atoms at a time (float64: half of them, so that two blocks
  // fit a compute unit).  Descriptor: rows (24 Yhat_lm, g_n); forces: rows
  // (T_n + 1, T_n'), replaced by the products (24 + 24).
  constexpr int HB = F64 ? L / 2 : L;
  constexpr int TB = HB < 16 ? HB : 16;  // rows of one product over n
  constexpr int YS = F64 ? 24 + MA + (MA % 2 == 0 ? 1 : 0) : 44;  // DT per descriptor row
  constexpr int FS = 52;                                          // float per force row
  constexpr int kBuf = AW * HB * YS * (int)sizeof(DT) > AW * HB * FS * 4
                           ? AW * HB * YS * (int)sizeof(DT)
                           : AW * HB * FS * 4;
  static_assert(24 + MA <= YS && 8 * RPL <= FS, "operand rows");
  static_assert(MA * 25 * (int)sizeof(DT) <= kBuf, "moments of one atom");
  __shared__ __align__(16) char s_buf[kWaves][kBuf];
  __shared__ __align__(16) DT s_q[kAtoms][QS];  // descriptor, then dU/dq in float32
  __shared__ __align__(16) float s_g[kAtoms][GS];
  __shared__ DT s_u[kWaves][kAtoms];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int h = lane >> 4, col = lane & 15;
  const int g_own = lane / L, sub = lane % L;
  const int al = AW * wave + g_own;  // the lane's atom within the block
  const int ac = col % kAtoms;       // the atom of column `col` of the network's products
  const int i0 = (int)xcd_block(blockIdx.x, gridDim.x) * kAtoms;
  const float rcr_inv = 1.f / rc_r, rca_inv = 1.f / rc_a;
  const double rcr_inv_d = 1.0 / rc_rd, rca_inv_d = 1.0 / rc_ad;
  const float rcr2 = rc_r * rc_r, rca2 = rc_a * rc_a;
  auto wave_lds_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  // ---- staging: thread (a, w) handles slots w, w + W, ... of atom a
  const int sa = tid % kAtoms, sw = tid / kAtoms;
  const int ia = i0 + sa;
  const int cra = ia < n ? cnt_r[ia] : 0, caa = ia < n ? cnt_a[ia] : 0;
  const double xa = ia < n ? pos[ia] : 0.0, ya = ia < n ? pos[n + ia] : 0.0,
               za = ia < n ? pos[2 * n + ia] : 0.0;
  int most = cra;
#pragma unroll
  for (int d = 1; d < kAtoms; d <<= 1) most = max(most, __shfl_xor(most, d, 64));
  const int chunks = (most + kSlots - 1) / kSlots;  // the same for the whole block
  // slots kSlots c ..; the first time they are seen (write) their pair vectors
  // and the zero partial forces of pairs beyond r_c^R are written
  auto stage = [&](int c, bool write) {
    uint32_t e[T];
    int rv[T];
    double pj[T][3], wj[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int sl = c * kSlots + sw + W * t;
      const size_t idx = sl < cra ? (size_t)sl * n + ia : 0;
      e[t] = nl[idx];
      rv[t] = rev[idx];
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int j = c * kSlots + sw + W * t < cra ? (int)(e[t] & kAtomMask) : 0;
      pj[t][0] = pos[j];
      pj[t][1] = pos[n + j];
      pj[t][2] = pos[2 * n + j];
      if constexpr (F64) wj[t] = wspd[perm[j]];
    }
    if (tid < 2 * kAtoms) s_mask[tid / kAtoms][tid % kAtoms] = 0ull;
    __syncthreads();  // the masks are clear, the previous chunk has been read
    float v[T][3];
    double d[T][3];
    int dst[T];
    unsigned long long ma = 0ull, mr = 0ull;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int sl = c * kSlots + sw + W * t;
      if constexpr (F64) {
        image_displacement_d(e[t], pj[t], xa, ya, za, box.h, d[t][0], d[t][1], d[t][2]);
#pragma unroll
        for (int x = 0; x < 3; ++x) v[t][x] = (float)d[t][x];
      } else {
        image_displacement(e[t], pj[t][0], pj[t][1], pj[t][2], xa, ya, za, box.h, v[t][0], v[t][1],
                           v[t][2]);
      }
      dst[t] = rv[t] * n + (int)(e[t] & kAtomMask);
      if (sl >= cra) continue;
      if (write && geo) geo[(size_t)sl * n + ia] = Partial3{v[t][0], v[t][1], v[t][2]};
      const float r2 = pair_r2(v[t][0], v[t][1], v[t][2]);
      if (sl < caa && r2 < rca2)
        ma |= 1ull << (sw + W * t);
      else if (r2 < rcr2)
        mr |= 1ull << (sw + W * t);
      else if (write)
        pin[(size_t)(unsigned)dst[t]] = Partial3{0.f, 0.f, 0.f};
    }
    if (ma) atomicOr(&s_mask[0][sa], ma);
    if (mr) atomicOr(&s_mask[1][sa], mr);
    __syncthreads();
    const unsigned long long fa = s_mask[0][sa], fr = s_mask[1][sa];
    const int na = __popcll(fa);
    if (sw == 0) {
      s_count[0][sa] = na;
      s_count[1][sa] = na + __popcll(fr);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const unsigned long long bit = 1ull << (sw + W * t);
      if (!((fa | fr) & bit)) continue;
      const int k = (fa & bit) ? __popcll(fa & (bit - 1)) : na + __popcll(fr & (bit - 1));
      if constexpr (F64) {
#pragma unroll
        for (int x = 0; x < 3; ++x) s_d[x][sa][k] = d[t][x];
        s_d[3][sa][k] = wj[t];
        s_dst[sa][k] = dst[t];
      } else {
        s_pair[sa][k] = make_float4(v[t][0], v[t][1], v[t][2], __int_as_float(dst[t]));
      }
    }
    __syncthreads();
  };
  // the wave's atoms: staged angular pairs (uniform) and the largest counts
  int n_ang[AW], max_ang, max_in;
  auto counts = [&] {
    max_ang = 0;
    max_in = 0;
#pragma unroll
    for (int g = 0; g < AW; ++g) {
      n_ang[g] = __builtin_amdgcn_readfirstlane(s_count[0][AW * wave + g]);
      max_ang = max(max_ang, n_ang[g]);
      max_in = max(max_in, __builtin_amdgcn_readfirstlane(s_count[1][AW * wave + g]));
    }
  };

  const double wi = F64 ? (i0 + al < n ? wspd[perm[i0 + al]] : 0.0) : 1.0;

  // ---- descriptor
  DT qr[MR];
  D4 c[AW][2];  // moments of atom g, tile t: n = RPL h + r, lm = 16 t + col
#pragma unroll
  for (int a = 0; a < MR; ++a) qr[a] = 0;
#pragma unroll
  for (int g = 0; g < AW; ++g)
#pragma unroll
    for (int t = 0; t < 2; ++t) c[g][t] = D4{0, 0, 0, 0};
  // row `col` of the moments' first operand holds n = RPL oh + orr
  int oh, orr;
  mma_owner<DT>(col, oh, orr);
  const int arow = orr < RPL && RPL * oh + orr < MA ? RPL * oh + orr : -1;
  DT* const yg = reinterpret_cast<DT*>(s_buf[wave]);
  for (int ch = 0; ch < chunks; ++ch) {
    stage(ch, true);
    counts();
    const int my_ang = s_count[0][al], my_in = s_count[1][al];
    for (int base = 0; base < max_in; base += L) {
      const int k = base + sub;
      const bool rad = k < my_in, ang = k < my_ang;
      DT x = 1, y = 0, zz = 0, w = 1;
      if (rad) {
        if constexpr (F64) {
          x = s_d[0][al][k];
          y = s_d[1][al][k];
          zz = s_d[2][al][k];
          w = wi * s_d[3][al][k];
        } else {
          const float4 v = s_pair[al][k];
          x = v.x;
          y = v.y;
          zz = v.z;
        }
      }
      DT r, rinv;
      if constexpr (F64) {
        r = sqrt(x * x + y * y + zz * zz);
        rinv = 1.0 / r;
      } else {
        const float r2 = pair_r2(x, y, zz);
        rinv = __builtin_amdgcn_rsqf(r2);
        r = r2 * rinv;
      }
      if (rad) {  // entries a >= NR are never read
        DT fc, T[MR];
        if constexpr (F64)
          chebyshev_values_d<MR>(r, rcr_inv_d, fc, T);
        else
          chebyshev_values<MR>(r, rcr_inv, fc, T);
        const DT wf = F64 ? w * fc : fc;
        qr[0] += wf;
#pragma unroll
        for (int a = 1; a < MR; ++a) qr[a] += wf * T[a];
      }
      if (base >= max_ang) continue;  // the wave's angular pairs are done
      DT gn[MA], yh[24];
#pragma unroll
      for (int a = 0; a < MA; ++a) gn[a] = 0;
#pragma unroll
      for (int m = 0; m < 24; ++m) yh[m] = 0;
      if (ang) {
        if constexpr (F64) {
          radial_basis_d<MA>(r, rca_inv_d, NA, gn);
#pragma unroll
          for (int a = 0; a < MA; ++a) gn[a] *= w;
          harmonics_d(x * rinv, y * rinv, zz * rinv, yh);
        } else {
          radial_basis_n<MA>(r, rca_inv, NA, gn);
          harmonics(x * rinv, y * rinv, zz * rinv, yh);
        }
      }
#pragma unroll
      for (int half = 0; half < L / HB; ++half) {
        if (base + HB * half >= max_ang) break;
        if (sub / HB == half) {
          DT* row = yg + (g_own * HB + sub % HB) * YS;
          if constexpr (F64) {
#pragma unroll
            for (int m = 0; m < 24; ++m) row[m] = yh[m];
#pragma unroll
            for (int a = 0; a < MA; ++a) row[24 + a] = gn[a];
          } else {
#pragma unroll
            for (int m = 0; m < 24; m += 4)
              *reinterpret_cast<float4*>(row + m) =
                  make_float4(yh[m], yh[m + 1], yh[m + 2], yh[m + 3]);
#pragma unroll
            for (int a = 0; a < MA; a += 4)
              *reinterpret_cast<float4*>(row + 24 + a) =
                  make_float4(gn[a], a + 1 < MA ? gn[a + 1] : 0.f, a + 2 < MA ? gn[a + 2] : 0.f,
                              a + 3 < MA ? gn[a + 3] : 0.f);
          }
        }
        wave_lds_sync();
#pragma unroll
        for (int g = 0; g < AW; ++g) {
          const int np = n_ang[g] - base - HB * half;  // uniform; pairs past it are zero
#pragma unroll
          for (int st = 0; st < HB / 4; ++st) {
            if (4 * st >= np) break;
            const DT* row = yg + (g * HB + 4 * st + h) * YS;
            const DT av = arow >= 0 ? row[24 + (arow >= 0 ? arow : 0)] : (DT)0;
            c[g][0] = mma(av, row[col], c[g][0]);
            c[g][1] = mma(av, col < 8 ? row[16 + (col & 7)] : (DT)0, c[g][1]);
          }
        }
        wave_lds_sync();
      }
    }
  }
  // radial components q_0 = R_0, q_n = (R_n + R_0)/2
  {
    const DT r0 = atom_sum<L>(qr[0]);
    if (sub == 0) s_q[al][0] = r0;
#pragma unroll
    for (int a = 1; a < MR; ++a) {
      const DT v = atom_sum<L>(qr[a]);
      if (sub == 0 && a < NR) s_q[al][a] = (DT)0.5 * (v + r0);
    }
    for (int v = NDES + sub; v < QS; v += L) s_q[al][v] = 0;  // padding
  }
  // angular components q_nl = sum_m c_nlm^2, one atom of the wave at a time
#pragma unroll
  for (int g = 0; g < AW; ++g) {
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int nn = RPL * h + r;
      if (nn < NA) {
        yg[nn * 25 + col] = c[g][0][r];
        if (col < 8) yg[nn * 25 + 16 + col] = c[g][1][r];
      }
    }
    wave_lds_sync();
    for (int v = lane; v < NA * LMAX; v += 64) {
      const int a = v / LMAX, l = v % LMAX + 1;
      DT s2 = 0;
      for (int m = 0; m < 2 * l + 1; ++m) {
        const DT cm = yg[a * 25 + l * l - 1 + m];
        s2 += cm * cm;
      }
      s_q[AW * wave + g][NR + v] = s2;
    }
    wave_lds_sync();
  }
  __syncthreads();

  // ---- network (Eqs. nn1, nn2): wave w evaluates neurons 16 w .. 16 w + 15
  if (wave < NT) {
    int nh, nrr;
    mma_owner<DT>(col, nh, nrr);
    const int mu_a = 16 * wave + 4 * nh + nrr;  // row `col` of W1
    float wv[KT][4];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = 16 * t + 4 * h + e;
        wv[t][e] = mu_a < NNEU && v < NDES ? z[mu_a * NDES + v] : 0.f;
      }
    float b1[4], w2[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int mu = 16 * wave + 4 * h + r;
      b1[r] = mu < NNEU ? z[NNEU * NDES + mu] : 0.f;
      w2[r] = mu < NNEU ? z[NNEU * (NDES + 1) + mu] : 0.f;
    }
    D4 act = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) act = mma((DT)wv[t][e], s_q[ac][16 * t + 4 * h + e], act);
    DT up = 0;
    float gm[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // tanh and its derivative 1 - tanh^2 from e = exp(-2|a|) (no cancellation)
      const DT x = act[r] - (DT)b1[r];
      if constexpr (F64) {
        const double ea = exp(-2.0 * fabs(x));
        const double inv = 1.0 / (1.0 + ea);
        up += (double)w2[r] * copysign((1.0 - ea) * inv, x);
        gm[r] = (float)((double)w2[r] * (4.0 * ea * inv * inv));
      } else {
        const float ea = __expf(-2.f * fabsf(x));
        const float inv = __builtin_amdgcn_rcpf(1.f + ea);
        up += w2[r] * copysignf((1.f - ea) * inv, x);
        gm[r] = w2[r] * (4.f * ea * inv * inv);
      }
    }
    up += __shfl_xor(up, 16, 64);
    up += __shfl_xor(up, 32, 64);
    if (col < kAtoms) {
      if (h == 0) s_u[wave][col] = up;
      *reinterpret_cast<float4*>(&s_g[col][16 * wave + 4 * h]) =
          make_float4(gm[0], gm[1], gm[2], gm[3]);
    }
  }
  __syncthreads();
  if (tid < kAtoms && i0 + tid < n) {
    DT u = s_u[0][tid];
#pragma unroll
    for (int w = 1; w < NT; ++w) u += s_u[w][tid];
    U[i0 + tid] = (float)(u - (DT)z[NNEU * (NDES + 2)]);
  }
  // dU/dq = W1^T G: wave w forms components 16 d .. 16 d + 15, d = w, w + 4, ...
  float* const dq0 = reinterpret_cast<float*>(&s_q[0][0]);  // [kAtoms][QS]
  for (int d = wave; d < KT; d += kWaves) {
    const int v = 16 * d + col;
    float wv[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int mu = 16 * t + 4 * h + e;
        wv[t][e] = mu < NNEU && v < NDES ? z[mu * NDES + v] : 0.f;
      }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = mma(wv[t][e], s_g[ac][16 * t + 4 * h + e], acc);
    if (col < kAtoms)
      *reinterpret_cast<float4*>(dq0 + col * QS + 16 * d + 4 * h) =
          make_float4(acc[0], acc[1], acc[2], acc[3]);
  }
  __syncthreads();

  // ---- partial forces
  // a_nlm = 2 dU/dq_nl c_nlm, the second operand of the products over n
  float an[AW][2][RPL];
#pragma unroll
  for (int g = 0; g < AW; ++g)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int lm = 16 * t + col, l = l_of(lm);
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        const int nn = RPL * h + r;
        const bool in = nn < NA && lm < NLM;
        const float dq = dq0[(AW * wave + g) * QS + (in ? NR + nn * LMAX + (l - 1) : 0)];
        an[g][t][r] = in ? (float)((DT)2 * (DT)dq * c[g][t][r]) : 0.f;
      }
    }
  const float* const dq = dq0 + al * QS;
  float dqs = 0.f;  // sum_n dU/dq_n over the radial components
  for (int a = 0; a < NR; ++a) dqs += dq[a];
  float* const tb = reinterpret_cast<float*>(s_buf[wave]);
  float fx = 0.f, fy = 0.f, fz = 0.f;
  for (int cc = 0; cc < chunks; ++cc) {
    // last chunk first: it is the one that is staged
    if (cc > 0) {
      stage(chunks - 1 - cc, false);
      counts();
    }
    const int my_ang = s_count[0][al], my_in = s_count[1][al];
    for (int base = 0; base < max_in; base += L) {
      const int k = base + sub;
      const bool rad = k < my_in, ang = k < my_ang;
      float dx = 1.f, dy = 0.f, dz = 0.f, wij = 1.f;
      int dst = 0;
      if (rad) {
        if constexpr (F64) {
          dx = (float)s_d[0][al][k];
          dy = (float)s_d[1][al][k];
          dz = (float)s_d[2][al][k];
          wij = (float)wi * (float)s_d[3][al][k];
          dst = s_dst[al][k];
        } else {
          const float4 v = s_pair[al][k];
          dx = v.x;
          dy = v.y;
          dz = v.z;
          dst = __float_as_int(v.w);
        }
      }
      const float r2 = pair_r2(dx, dy, dz);
      const float rinv = __builtin_amdgcn_rsqf(r2);
      const float r = r2 * rinv;
      const float x = dx * rinv, y = dy * rinv, z = dz * rinv;
      float px = 0.f, py = 0.f, pz = 0.f;
      if (rad) {
        // sum_n dU/dq_n g_n' = f_c' (S_1 + sum_n dU/dq_n)/2 + f_c (dx/dr) S_2/2
        float fc, dfc, dxdr, T[MR], dT[MR];
        chebyshev_terms<MR>(r, rcr_inv, fc, dfc, dxdr, T, dT);
        float s1 = dq[0], s2 = 0.f;
#pragma unroll
        for (int a = 1; a < MR; ++a)
          if (a < NR) {
            s1 += dq[a] * T[a];
            s2 += dq[a] * dT[a];
          }
        const float f = 0.5f * (dfc * (s1 + dqs) + fc * dxdr * s2);
        px += f * x;
        py += f * y;
        pz += f * z;
      }
      if (base < max_ang) {
        float fc, dfc, dxdr;
        float At[24], D[24];
        {
          float T[MA], dT[MA];
          chebyshev_terms<MA>(r, rca_inv, fc, dfc, dxdr, T, dT);
#pragma unroll
          for (int half = 0; half < L / HB; ++half) {
            if (base + HB * half >= max_ang) break;
            float* const row = tb + (g_own * HB + sub % HB) * FS;
            if (sub / HB == half) {
              // T_n + 1 and T_n' for n < 4 RPL (n >= N_A meet a_nlm = 0)
              float t1[4 * RPL], t2[4 * RPL];
#pragma unroll
              for (int a = 0; a < 4 * RPL; ++a) {
                t1[a] = a < MA ? T[a < MA ? a : 0] + 1.f : 0.f;
                t2[a] = a < MA ? dT[a < MA ? a : 0] : 0.f;
              }
#pragma unroll
              for (int a = 0; a < 4 * RPL; a += 4) {
                *reinterpret_cast<float4*>(row + a) =
                    make_float4(t1[a], t1[a + 1], t1[a + 2], t1[a + 3]);
                *reinterpret_cast<float4*>(row + 4 * RPL + a) =
                    make_float4(t2[a], t2[a + 1], t2[a + 2], t2[a + 3]);
              }
            }
            wave_lds_sync();
#pragma unroll
            for (int gt = 0; gt < AW * (HB / TB); ++gt) {
              const int g = gt / (HB / TB), first = TB * (gt % (HB / TB));
              if (base + HB * half + first >= n_ang[g]) continue;  // uniform
              float* const rows = tb + (g * HB + first) * FS;
              const float* const src = rows + (col % TB) * FS;
              float t1[RPL], t2[RPL];
#pragma unroll
              for (int q = 0; q < RPL; ++q) {
                t1[q] = src[RPL * h + q];
                t2[q] = src[4 * RPL + RPL * h + q];
              }
              f32x4 p1[2], p2[2];
#pragma unroll
              for (int t = 0; t < 2; ++t) {
                p1[t] = f32x4{0.f, 0.f, 0.f, 0.f};
                p2[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < RPL; ++q) {
                  p1[t] = mma(t1[q], an[g][t][q], p1[t]);
                  p2[t] = mma(t2[q], an[g][t][q], p2[t]);
                }
              }
              wave_lds_sync();  // every lane has read the atom's rows
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                if (4 * h + q >= TB) break;
                float* const o = rows + (4 * h + q) * FS;
                o[col] = p1[0][q];
                o[24 + col] = p2[0][q];
                if (col < 8) {
                  o[16 + col] = p1[1][q];
                  o[40 + col] = p2[1][q];
                }
              }
            }
            wave_lds_sync();
            if (sub / HB == half) {
#pragma unroll
              for (int m = 0; m < 24; m += 4) {
                const float4 v1 = *reinterpret_cast<const float4*>(row + m);
                const float4 v2 = *reinterpret_cast<const float4*>(row + 24 + m);
                At[m] = v1.x, At[m + 1] = v1.y, At[m + 2] = v1.z, At[m + 3] = v1.w;
                D[m] = v2.x, D[m + 1] = v2.y, D[m + 2] = v2.z, D[m + 3] = v2.w;
              }
            }
            wave_lds_sync();  // the rows are written again in the next round
          }
        }
        if (ang) {
          // A = f_c At/2 multiplies the harmonics' gradients and
          // B = f_c' At/2 + f_c (dx/dr) D/2 the harmonics
          float st, sd, gx, gy, gz;
          harmonic_sums(
              x, y, z, [&](int m) { return At[m]; }, [&](int m) { return D[m]; }, st, sd, gx, gy,
              gz);
          const float hf = 0.5f * fc;
          const float sb = 0.5f * (dfc * st + fc * dxdr * sd);
          gx *= hf;
          gy *= hf;
          gz *= hf;
          const float ug = x * gx + y * gy + z * gz;
          px += sb * x + (gx - x * ug) * rinv;
          py += sb * y + (gy - y * ug) * rinv;
          pz += sb * z + (gz - z * ug) * rinv;
        }
      }
      if (rad) {
        if constexpr (F64) {  // every term of the pair carries its weight once
          px *= wij;
          py *= wij;
          pz *= wij;
        }
        fx += px;
        fy += py;
        fz += pz;
        pin[(size_t)(unsigned)dst] = Partial3{px, py, pz};
      }
    }
  }
  fx = atom_sum<L>(fx);
  fy = atom_sum<L>(fy);
  fz = atom_sum<L>(fz);
  if (sub == 0 && i0 + al < n) {
    fown[i0 + al] = fx;
    fown[n + i0 + al] = fy;
    fown[2 * n + i0 + al] = fz;
  }
}

inline unsigned blocks_for(size_t work, int block) { return (unsigned)((work + block - 1) / block); }

}  // namespace

bool generic_supports(const nep_hyper& h) {
  return h.n_max_radial + 1 <= kMaxR && h.n_max_angular + 1 <= kMaxA && h.l_max >= 1 &&
         h.l_max <= 4 && h.n_neuron <= kMaxNeu;
}

namespace {

template <int TR, int TA, int TL, int TNEU, bool F64, int AW>
void launch_atoms(nep_ctx ctx, const double* pos) {
  const System& s = ctx->sys;
  const nep_hyper& h = ctx->hyper;
  launch_kernel(ctx, true, true, k_partials_generic<TR, TA, TL, TNEU, F64, AW>,
                dim3(blocks_for(s.n, kWaves * AW)), dim3(64 * kWaves), s.n, pos,
                (const uint32_t*)s.nl.ptr, (const int*)s.cnt_r.ptr, (const int*)s.cnt_a.ptr,
                (const int*)s.rev.ptr, s.box, (const float*)ctx->z.ptr, h.n_max_radial + 1,
                h.n_max_angular + 1, h.l_max, h.n_neuron, h.rc_radial, h.rc_angular,
                F64 ? (const double*)ctx->species_wd.ptr : (const double*)nullptr,
                (const int*)s.perm.ptr, ctx->p.ptr, ctx->fown.ptr, ctx->U.ptr,
                s.n <= kPairVectorMaxAtoms ? ctx->geo.ptr : (Partial3*)nullptr);
}

// Atoms per wave: one while two blocks per compute unit hold every atom (256
// units x 2 blocks x 4 waves): the chip is then not full and the shorter chain
// of a wave counts (12.9 against 20.5 us for 80-50-1 on 1,000 atoms, 8.9
// against 13.0 us for 29-30-1, 16.9 against 23.5 us for PbTe), else four (20.7
// against 25.9 us for 80-50-1 on 2,744 atoms, 13.3 against 16.3 us for 29-30-1,
// 24.5 against 32.4 us for PbTe; two per wave lie between).
constexpr int kOneAtomWaves = 2048;

template <int TR, int TA, int TL, int TNEU, bool F64>
void launch_shape(nep_ctx ctx, const double* pos) {
  if (ctx->sys.n <= kOneAtomWaves)
    launch_atoms<TR, TA, TL, TNEU, F64, 1>(ctx, pos);
  else
    launch_atoms<TR, TA, TL, TNEU, F64, 4>(ctx, pos);
}

bool is_shape(const nep_hyper& h, int nr, int na, int lmax, int nneu) {
  return h.n_max_radial + 1 == nr && h.n_max_angular + 1 == na && h.l_max == lmax &&
         h.n_neuron == nneu;
}

}  // namespace

// Compile-time sizes for the models of Table I (general Si, silicene, PbTe)
// and the default model; every other size takes the runtime-sized kernel.
// Multicomponent systems take the float64-descriptor kernels (compiled sizes
// for the PbTe and default models).
hipError_t launch_partials_generic(nep_ctx ctx, const double* pos) {
  if (ctx->sys.n == 0) return hipSuccess;
  const nep_hyper& h = ctx->hyper;
  if (ctx->species_on()) {
    if (is_shape(h, 13, 7, 4, 40))
      launch_shape<13, 7, 4, 40, true>(ctx, pos);
    else if (is_shape(h, 9, 5, 4, 30))
      launch_shape<9, 5, 4, 30, true>(ctx, pos);
    else
      launch_shape<0, 0, 0, 0, true>(ctx, pos);
  } else if (is_shape(h, 16, 16, 4, 50)) {
    launch_shape<16, 16, 4, 50, false>(ctx, pos);
  } else if (is_shape(h, 13, 13, 4, 40)) {
    launch_shape<13, 13, 4, 40, false>(ctx, pos);
  } else if (is_shape(h, 13, 7, 4, 40)) {
    launch_shape<13, 7, 4, 40, false>(ctx, pos);
  } else if (is_shape(h, 9, 5, 4, 30)) {
    launch_shape<9, 5, 4, 30, false>(ctx, pos);
  } else {
    launch_shape<0, 0, 0, 0, false>(ctx, pos);
  }
  return hipGetLastError();
}

}  // namespace nep
