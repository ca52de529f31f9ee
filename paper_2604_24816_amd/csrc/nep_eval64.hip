// FP64 evaluation of energy, forces and virial (the NEP_FP64 precision) and the FP64
// parameter gradient.
//
// Every descriptor, network, force and virial operation runs in FP64, from an FP64
// copy of the model parameters, over the same neighbour lists as the FP32 path. It is the
// check form -- central differences at h = 1e-5 A, agreement with an FP64 reference to
// round-off -- for boxes of hundreds to thousands of atoms, so 16 lanes share a center
// (16 centers to a workgroup): lane l takes list entries l, l + 16, ..., all angular
// channels in one pass (120 FP64 accumulators: one wavefront per SIMD), sums over the lanes
// by cross-lane adds, the network spread over the lanes through LDS, FP64 global atomics
// for the angular reaction forces. A thread per center with the accumulators recomputed
// channel by channel took 352 (descriptors), 1317 (forces) and 2567 us (gradient) for 2,048
// atoms.
//
// Quantities (Section III.B): radial q_n = sum_j g_n(r_ij), angular s_nlm = sum_j
// g_n(r_ij) P_lm(u_ij) with q_nl = sum_m W_lm s_nlm^2, the four-body tr(S_n^3), the
// network U_i and dU_i/dq; forces F_i = sum_j [dU_i/dr_ij + dU_j/dr_ji] (radial, by
// gather) plus the angular pair forces applied to both atoms; W_ab = -sum r_a (dU_i/dr_ij)_b.
#include "nep_fast.h"

namespace nep {
namespace {

using namespace kern;

constexpr double kPi64 = 3.14159265358979323846;
constexpr int kL64 = 16;              // lanes of a center
constexpr int kC64 = kBlock / kL64;   // centers of a workgroup

// Sum over the 16 lanes of a center, in every one of them.
__device__ __forceinline__ double lanes_sum64(double v) { return lanes_sum<kL64>(v); }

// f_k(r) = f_c(r) (T_k(x) + 1) / 2 and df_k/dr for k < K, with x = 2 (r/rc - 1)^2 - 1
// and f_c = (1 + cos(pi r / rc)) / 2.
template <int K>
__device__ __forceinline__ void basis64(double r, double rc, double* f, double* df) {
  const double rr = r / rc;
  double sn, cs;
  sincospi(rr, &sn, &cs);
  const double fc = 0.5 * (1.0 + cs);
  const double dfc = -0.5 * kPi64 / rc * sn;
  const double y = rr - 1.0;
  const double x = 2.0 * y * y - 1.0;
  const double dx = 4.0 * y / rc;
  double Tm1 = 1.0, T = x, dTm1 = 0.0, dT = 1.0;
  f[0] = fc;
  df[0] = dfc;
  f[1] = 0.5 * (x + 1.0) * fc;
  df[1] = 0.5 * dx * fc + 0.5 * (x + 1.0) * dfc;
#pragma unroll
  for (int k = 2; k < K; ++k) {
    const double Tn = 2.0 * x * T - Tm1;
    const double dTn = 2.0 * T + 2.0 * x * dT - dTm1;
    Tm1 = T;
    T = Tn;
    dTm1 = dT;
    dT = dTn;
    f[k] = 0.5 * (Tn + 1.0) * fc;
    df[k] = 0.5 * dTn * dx * fc + 0.5 * (Tn + 1.0) * dfc;
  }
}

// The model's coefficients and W0 where the lanes read them: with two species the
// coefficient blocks of all species pairs in LDS (the block differs from lane to lane), with
// one through the constant address space; W0, its bias, output weights and scaler in LDS.
typedef const __attribute__((address_space(4))) double* cdouble_ptr;
template <class S, bool MULTI>
struct Param64 {
  static constexpr int kR = S::NR * S::KR, kA = S::NA * S::KA;
  double cR[MULTI ? kMaxTypes * kMaxTypes * kR : 1], cA[MULTI ? kMaxTypes * kMaxTypes * kA : 1];
  double W0[S::H * S::D], b0[S::H], w1[S::H], sigma[S::D];
};
template <class S, bool MULTI>
__device__ __forceinline__ void stage64(const ModelDev& m, const Model64& p, Param64<S, MULTI>& t) {
  using P = Param64<S, MULTI>;
  if constexpr (MULTI) {
    for (int e = threadIdx.x; e < m.T * m.T * P::kR; e += kBlock) t.cR[e] = p.cR[e];
    for (int e = threadIdx.x; e < m.T * m.T * P::kA; e += kBlock) t.cA[e] = p.cA[e];
  }
  for (int e = threadIdx.x; e < S::H * S::D; e += kBlock) t.W0[e] = p.W0[e];
  for (int e = threadIdx.x; e < S::H; e += kBlock) {
    t.b0[e] = p.b0[e];
    t.w1[e] = p.w1[e];
  }
  for (int e = threadIdx.x; e < S::D; e += kBlock) t.sigma[e] = p.sigma[e];
  __syncthreads();
}
// Calls f with the radial (ANG: angular) coefficient block of (center, neighbour) species.
template <bool ANG, class S, bool MULTI, class F>
__device__ __forceinline__ void with_coeffs64(const ModelDev& m, const Model64& p, const Param64<S, MULTI>& t, int tc,
                                              int tk, F&& f) {
  using P = Param64<S, MULTI>;
  if constexpr (MULTI) f((ANG ? t.cA : t.cR) + (tc * m.T + tk) * (ANG ? P::kA : P::kR));
  else f((cdouble_ptr)(ANG ? p.cA : p.cR));
}

// g_n and g_n' for n < N from coefficients c[n][K] and the basis.
template <int N, int K, class CP>
__device__ __forceinline__ void channels64(const double* f, const double* df, CP c, double* g, double* dg) {
#pragma unroll
  for (int n = 0; n < N; ++n) {
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      a += c[n * K + k] * f[k];
      b += c[n * K + k] * df[k];
    }
    g[n] = a;
    dg[n] = b;
  }
}

struct Pair64 {
  int32_t j;
  int t;
  double d[3], r, r2;
};

// Visits lane l's pairs of center i inside rcut (FP64 minimum image over the first kmax
// list entries): fn(p, Pair64). The next entry's position loads while one is worked on.
template <bool MULTI, class Fn>
__device__ __forceinline__ void for_pairs64(const EvalBuffers& b, int64_t i, int l, int kmax, double rcut2, Fn&& fn) {
  if (kmax <= 0) return;
  const int64_t N = b.N;
  const double xi = b.x[i], yi = b.x[N + i], zi = b.x[2 * N + i];
  struct Item {
    int32_t j;
    int t;
    double x, y, z;
  };
  auto load = [&](int p) {
    Item e;
    e.j = b.nbr[(int64_t)(p < kmax ? p : kmax - 1) * N + i];
    e.x = b.x[e.j];
    e.y = b.x[N + e.j];
    e.z = b.x[2 * N + e.j];
    e.t = MULTI ? b.type[e.j] : 0;
    return e;
  };
  Item e = load(l);
  for (int p = l; p < kmax; p += kL64) {
    const Item n = load(p + kL64);
    Pair64 q;
    q.j = e.j;
    q.t = e.t;
    q.d[0] = min_image(e.x - xi, b.box[0]);
    q.d[1] = min_image(e.y - yi, b.box[1]);
    q.d[2] = min_image(e.z - zi, b.box[2]);
    q.r2 = q.d[0] * q.d[0] + q.d[1] * q.d[1] + q.d[2] * q.d[2];
    if (q.r2 < rcut2) {
      q.r = sqrt(q.r2);
      fn(p, q);
    }
    e = n;
  }
}

// 3 det S = tr(S^3) of one channel's traceless S, and d tr(S^3) / d s for its five
// l = 2 accumulators (xy, yz, 3z^2 - r^2, xz, x^2 - y^2).
__device__ __forceinline__ void fourbody64(const double* s2, double& q4, double* d5) {
  const double xy = s2[0], yz = s2[1], zz = s2[2] / 3.0, xz = s2[3];
  const double xx = 0.5 * (s2[4] - zz), yy = 0.5 * (-s2[4] - zz);
  q4 = 3.0 * (xx * (yy * zz - yz * yz) - xy * (xy * zz - yz * xz) + xz * (xy * yz - yy * xz));
  const double Qxx = xx * xx + xy * xy + xz * xz, Qyy = xy * xy + yy * yy + yz * yz;
  const double Qzz = xz * xz + yz * yz + zz * zz;
  const double Qxy = xx * xy + xy * yy + xz * yz, Qyz = xy * xz + yy * yz + yz * zz;
  const double Qxz = xx * xz + xy * yz + xz * zz;
  d5[0] = 6.0 * Qxy;
  d5[1] = 6.0 * Qyz;
  d5[2] = Qzz - 0.5 * (Qxx + Qyy);
  d5[3] = 6.0 * Qxz;
  d5[4] = 1.5 * (Qxx - Qyy);
}

// q_nl and four-body descriptors from the accumulators, into q[NR..D).
template <class S>
__device__ __forceinline__ void finish64(const double* s, double* q) {
  constexpr int NR = S::NR, NA = S::NA, NC = S::NC;
#pragma unroll
  for (int n = 0; n < NA; ++n) {
#pragma unroll
    for (int lm = 0; lm < NC; ++lm)
      q[NR + (comp_l(lm) - 1) * NA + n] += (double)kW[lm] * s[n * NC + lm] * s[n * NC + lm];
    if constexpr (S::FB) {
      double q4, d5[5];
      fourbody64(s + n * NC + 3, q4, d5);
      q[NR + S::L3 * NA + n] = q4;
    }
  }
}

// Descriptors, network, U_i (+ ZBL) and dU_i/dq (FP64): U64[i], Fp64[k][i].
template <class S, bool MULTI>
__global__ void __launch_bounds__(kBlock, 1)
k_desc64(ModelDev m, Model64 p, EvalBuffers b, double* __restrict__ U64, double* __restrict__ Fp64) {
  __shared__ double sh[4];
  __shared__ Param64<S, MULTI> par;
  __shared__ double rows[kC64][S::D + S::H];  // sigma q, then w1 (1 - tanh^2), of each center
  constexpr int NR = S::NR, NA = S::NA, NC = S::NC, KR = S::KR, KA = S::KA, D = S::D, H = S::H;
  stage64<S, MULTI>(m, p, par);
  const int64_t N = b.N;
  const int l = threadIdx.x % kL64;
  const int64_t i = (int64_t)blockIdx.x * kC64 + threadIdx.x / kL64;
  double* qs = rows[threadIdx.x / kL64];
  double* a1 = qs + D;
  double U = 0.0;
  if (i < N) {
    const int ti = MULTI ? b.type[i] : 0;
    const int kA = angular_bound(b, i);
    const double rcA2 = m.rcA64 * m.rcA64;
    double q[D], s[NA * NC], uz = 0.0;
#pragma unroll
    for (int k = 0; k < D; ++k) q[k] = 0.0;
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) s[k] = 0.0;
    for_pairs64<MULTI>(b, i, l, radial_bound(b, i), m.rcR64 * m.rcR64, [&](int k, const Pair64& pr) {
      {
        double f[KR], df[KR], g[NR], dg[NR];
        basis64<KR>(pr.r, m.rcR64, f, df);
        with_coeffs64<false>(m, p, par, ti, pr.t, [&](auto c) { channels64<NR, KR>(f, df, c, g, dg); });
#pragma unroll
        for (int n = 0; n < NR; ++n) q[n] += g[n];
      }
      if (pr.r2 < m.zbl_o2) {
        double e, de;
        zbl_pair<MULTI>(m, ti * m.T + pr.t, pr.r, e, de);
        uz += 0.5 * e;
      }
      if (k < kA && pr.r2 < rcA2) {
        double f[KA], df[KA], g[NA], dg[NA];
        basis64<KA>(pr.r, m.rcA64, f, df);
        with_coeffs64<true>(m, p, par, ti, pr.t, [&](auto c) { channels64<NA, KA>(f, df, c, g, dg); });
        const double ir = 1.0 / pr.r;
        for_each_poly<NC>(pr.d[0] * ir, pr.d[1] * ir, pr.d[2] * ir, [&](int lm, double P) {
#pragma unroll
          for (int n = 0; n < NA; ++n) s[n * NC + lm] += g[n] * P;
        });
      }
    });
#pragma unroll
    for (int n = 0; n < NR; ++n) q[n] = lanes_sum64(q[n]);
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) s[k] = lanes_sum64(s[k]);
    uz = lanes_sum64(uz);
    finish64<S>(s, q);
#pragma unroll
    for (int k = 0; k < D; ++k)
      if (k % kL64 == l) qs[k] = par.sigma[k] * q[k];
    wave_lds_sync();
    for (int mu = l; mu < H; mu += kL64) {
      double h = -par.b0[mu];
      for (int k = 0; k < D; ++k) h += par.W0[mu * D + k] * qs[k];
      const double t = tanh(h);
      U += par.w1[mu] * t;
      a1[mu] = par.w1[mu] * (1.0 - t * t);
    }
    U = lanes_sum64(U) - p.b1 + uz;
    wave_lds_sync();
    for (int k = l; k < D; k += kL64) {
      double v = 0.0;
      for (int mu = 0; mu < H; ++mu) v += par.W0[mu * D + k] * a1[mu];
      Fp64[(int64_t)k * N + i] = par.sigma[k] * v;
    }
    if (l == 0) U64[i] = U;
  }
  double e[1] = {l == 0 ? U : 0.0}, sum[1];
  block_sum_n<1>(e, sum, sh);
  if (threadIdx.x == 0) b.ew[(int64_t)blockIdx.x * kPartialStride + P_ENERGY] = sum[0];
}

// Forces (F64 [3][N], zeroed before) and virial partials (FP64).
template <class S, bool MULTI>
__global__ void __launch_bounds__(kBlock, 1)
k_force64(ModelDev m, Model64 p, EvalBuffers b, const double* __restrict__ Fp64, double* __restrict__ F64) {
  __shared__ double sh[4 * 9];
  __shared__ Param64<S, MULTI> par;
  constexpr int NR = S::NR, NA = S::NA, NC = S::NC, KR = S::KR, KA = S::KA;
  stage64<S, MULTI>(m, p, par);
  const int64_t N = b.N;
  const int l = threadIdx.x % kL64;
  const int64_t i = (int64_t)blockIdx.x * kC64 + threadIdx.x / kL64;
  double f[3] = {0.0, 0.0, 0.0}, w[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) w[k] = 0.0;
  auto add_pair = [&](const Pair64& q, const double* fij) {  // dU_i/dr_ij on both atoms + virial
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int c = 0; c < 3; ++c) w[a * 3 + c] -= q.d[a] * fij[c];
    }
  };
  if (i < N) {
    const int ti = MULTI ? b.type[i] : 0;
    const int kA = angular_bound(b, i);
    const double rcA2 = m.rcA64 * m.rcA64;
    // the accumulators, then dU_i/ds_nlm in their place
    double G[NA * NC];
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) G[k] = 0.0;
    for_pairs64<MULTI>(b, i, l, kA, rcA2, [&](int, const Pair64& pr) {
      double fk[KA], df[KA], g[NA], dg[NA];
      basis64<KA>(pr.r, m.rcA64, fk, df);
      with_coeffs64<true>(m, p, par, ti, pr.t, [&](auto c) { channels64<NA, KA>(fk, df, c, g, dg); });
      const double ir = 1.0 / pr.r;
      for_each_poly<NC>(pr.d[0] * ir, pr.d[1] * ir, pr.d[2] * ir, [&](int lm, double P) {
#pragma unroll
        for (int n = 0; n < NA; ++n) G[n * NC + lm] += g[n] * P;
      });
    });
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) G[k] = lanes_sum64(G[k]);
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      double d5[5] = {}, q4;
      if constexpr (S::FB) fourbody64(G + n * NC + 3, q4, d5);
      const double f4 = S::FB ? Fp64[(int64_t)(NR + (S::FB ? S::L3 : 0) * NA + n) * N + i] : 0.0;
      double fl[S::L3];
#pragma unroll
      for (int k = 0; k < S::L3; ++k) fl[k] = Fp64[(int64_t)(NR + k * NA + n) * N + i];
#pragma unroll
      for (int lm = 0; lm < NC; ++lm) {
        double v = fl[comp_l(lm) - 1] * 2.0 * (double)kW[lm] * G[n * NC + lm];
        if (S::FB && comp_l(lm) == 2) v += f4 * d5[lm - 3];
        G[n * NC + lm] = v;
      }
    }
    double fpi[NR];
#pragma unroll
    for (int n = 0; n < NR; ++n) fpi[n] = Fp64[(int64_t)n * N + i];
    for_pairs64<MULTI>(b, i, l, radial_bound(b, i), m.rcR64 * m.rcR64, [&](int k, const Pair64& q) {
      const double ir = 1.0 / q.r;
      {
        // radial (gather): (dU_i/dr + dU_j/dr) along u; ZBL's pair derivative likewise
        double fk[KR], df[KR], g[NR], dgi[NR], dgj[NR];
        basis64<KR>(q.r, m.rcR64, fk, df);
        with_coeffs64<false>(m, p, par, ti, q.t, [&](auto c) { channels64<NR, KR>(fk, df, c, g, dgi); });
        with_coeffs64<false>(m, p, par, q.t, ti, [&](auto c) { channels64<NR, KR>(fk, df, c, g, dgj); });
        double si = 0.0, sj = 0.0;
#pragma unroll
        for (int n = 0; n < NR; ++n) {
          si += fpi[n] * dgi[n];
          sj += Fp64[(int64_t)n * N + q.j] * dgj[n];
        }
        if (q.r2 < m.zbl_o2) {
          double e, de;
          zbl_pair<MULTI>(m, ti * m.T + q.t, q.r, e, de);
          si += 0.5 * de;
          sj += 0.5 * de;
        }
        double fij[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          f[c] += (si + sj) * q.d[c] * ir;
          fij[c] = si * q.d[c] * ir;
        }
        add_pair(q, fij);
      }
      if (k < kA && q.r2 < rcA2) {
        double fk[KA], df[KA], g[NA], dg[NA];
        basis64<KA>(q.r, m.rcA64, fk, df);
        with_coeffs64<true>(m, p, par, ti, q.t, [&](auto c) { channels64<NA, KA>(fk, df, c, g, dg); });
        const double u[3] = {q.d[0] * ir, q.d[1] * ir, q.d[2] * ir};
        double fij[3] = {0.0, 0.0, 0.0}, sA = 0.0;
        // d(g P_lm)/dr_j = g' P u + g (grad P - l P u) / r
        for_each_poly_grad<NC>(u[0], u[1], u[2], [&](int lm, double P, double px, double py, double pz) {
          double A = 0.0, B = 0.0;
#pragma unroll
          for (int n = 0; n < NA; ++n) {
            A += G[n * NC + lm] * dg[n];
            B += G[n * NC + lm] * g[n];
          }
          B *= ir;
          sA += P * (A - (double)comp_l(lm) * B);
          fij[0] += B * px;
          fij[1] += B * py;
          fij[2] += B * pz;
        });
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          fij[c] += sA * u[c];
          f[c] += fij[c];
          unsafeAtomicAdd(&F64[(int64_t)c * N + q.j], -fij[c]);
        }
        add_pair(q, fij);
      }
    });
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      f[c] = lanes_sum64(f[c]);
      if (l == 0) unsafeAtomicAdd(&F64[(int64_t)c * N + i], f[c]);
    }
  }
  double sum[9];
  block_sum_n<9>(w, sum, sh);
  if (threadIdx.x == 0)
#pragma unroll
    for (int k = 0; k < 9; ++k) b.ew[(int64_t)blockIdx.x * kPartialStride + P_VIR + k] = sum[k];
}

// ------------------------------------------------------------ FP64 parameter gradient
// Gradient of L = gE E + sum_i gF_i . F_i with respect to every packed parameter
// [cR | cA | sigma | W0 | b0 | w1 | b1], all in FP64 (the check form of the FP32
// training kernel). As there, F = -dE/dx turns the force term into
// -sum_i dU_i/dq_i . v_i with v_i = sum_j dq_i/dr_ij . (gF_j - gF_i) the descriptor JVP,
// so each center contributes L_i = gE U_i - Fp_i . v_i (Fp = dU_i/dq). With
// q~ = sigma q, v~ = sigma v, h = W0 q~ - b0, t = tanh h, d = 1 - t^2, z = W0 v~:
//   dL_i/dW0 = alpha q~^T - beta v~^T, alpha = gE w1 d + 2 z w1 t d, beta = w1 d,
//   dL_i/db0 = -alpha, dL_i/dw1 = gE t - z d, dL_i/db1 = -gE,
//   dL_i/dsigma_k = q_k (W0^T alpha)_k - v_k (W0^T beta)_k,
// and the coefficients through rho = dL_i/dq = sigma W0^T alpha and dL_i/dv = -Fp:
//   radial c^{t_i t}_{nk}: sum over neighbours of species t of rho_n f_k - Fp_n f_k' (u.w);
//   angular c^{t_i t}_{nk}: with C_nlm = dL_i/ds_nlm and A_nlm = dL_i/dsd_nlm (sd the
//   JVP of s), sum over neighbours of f_k (X_n + Z_n) + f_k' (u.w) Y_n for
//   X_n = sum_lm C_nlm P_lm, Y_n = sum_lm A_nlm P_lm, Z_n = sum_lm A_nlm (grad P_lm . w - l P_lm (u.w)) / r.
// Three passes over the list (s; sd; the angular coefficients), the accumulators kept in LDS
// between them; the workgroup sums its centers' terms from LDS, one thread to a parameter
// in a fixed order, and adds them to the gradient with one FP64 atomic per parameter.

// w_j - w_i for the force weights w [3][N] (zero without a force term).
__device__ __forceinline__ void weight_diff(const double* w, int64_t N, int64_t i, int32_t j, double* o) {
#pragma unroll
  for (int c = 0; c < 3; ++c) o[c] = w ? w[c * N + j] - w[c * N + i] : 0.0;
}

// d5 = d tr(S^3)/ds (fourbody64) and its derivative along sd, h5 = (d d5/ds) sd; d5 is
// quadratic in s, so h5 = (d5(s + sd) - d5(s - sd)) / 2 exactly.
__device__ __forceinline__ void fourbody_dir64(const double* s2, const double* sd2, double* d5, double* h5) {
  double q4, a[5], b[5], sp[5], sm[5];
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    sp[c] = s2[c] + sd2[c];
    sm[c] = s2[c] - sd2[c];
  }
  fourbody64(s2, q4, d5);
  fourbody64(sp, q4, a);
  fourbody64(sm, q4, b);
#pragma unroll
  for (int c = 0; c < 5; ++c) h5[c] = 0.5 * (a[c] - b[c]);
}

// What the lanes of a center share, and what the workgroup sums over its centers.
template <class S, bool MULTI>
struct Center64 {
  static constexpr int TT = MULTI ? kMaxTypes : 1;
  double q[S::D], v[S::D];                  // descriptors and their JVP
  double al[S::H], be[S::H], gw[S::H];      // alpha, beta, gE t - z d
  double sa[S::D], sb[S::D];                // W0^T alpha, W0^T beta
  double F[TT][S::KR], E[TT][S::KR];        // radial basis sums
  union {
    struct {
      double s[S::NA * S::NC], sd[S::NA * S::NC];  // accumulators and JVP, then A and C
    };
    double gc[TT][S::NA * S::KA];           // angular coefficient sums
  };
  int type, valid;
};

template <class S, bool MULTI>
__global__ void __launch_bounds__(kBlock, 1)
k_grad64(ModelDev m, Model64 p, EvalBuffers b, const double* __restrict__ w, double gE, double* __restrict__ grad) {
  constexpr int NR = S::NR, NA = S::NA, NC = S::NC, KR = S::KR, KA = S::KA, D = S::D, H = S::H, L3 = S::L3;
  constexpr int TT = MULTI ? kMaxTypes : 1;
  __shared__ Param64<S, MULTI> par;
  __shared__ Center64<S, MULTI> ctr[kC64];
  stage64<S, MULTI>(m, p, par);
  const int64_t N = b.N;
  const int l = threadIdx.x % kL64;
  const int64_t i = (int64_t)blockIdx.x * kC64 + threadIdx.x / kL64;
  Center64<S, MULTI>& C = ctr[threadIdx.x / kL64];
  const bool valid = i < N;
  const int T = MULTI ? m.T : 1;
  const int ti = (MULTI && valid) ? b.type[i] : 0;
  const int kA = valid ? angular_bound(b, i) : 0, kR = valid ? radial_bound(b, i) : 0;
  const double rcR2 = m.rcR64 * m.rcR64, rcA2 = m.rcA64 * m.rcA64;
  if (l == 0) {
    C.type = ti;
    C.valid = valid ? 1 : 0;
  }
  double vr[NR];  // radial part of the JVP
#pragma unroll
  for (int n = 0; n < NR; ++n) vr[n] = 0.0;
  {
    // radial basis sums and the accumulators
    double q[D], F[TT][KR], E[TT][KR], s[NA * NC];
#pragma unroll
    for (int k = 0; k < D; ++k) q[k] = 0.0;
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int k = 0; k < KR; ++k) F[t][k] = E[t][k] = 0.0;
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) s[k] = 0.0;
    for_pairs64<MULTI>(b, i, l, kR, rcR2, [&](int k0, const Pair64& pr) {
      const double ir = 1.0 / pr.r;
      {
        double f[KR], df[KR], wd[3];
        basis64<KR>(pr.r, m.rcR64, f, df);
        weight_diff(w, N, i, pr.j, wd);
        const double uw = (pr.d[0] * wd[0] + pr.d[1] * wd[1] + pr.d[2] * wd[2]) * ir;
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          const bool on = !MULTI || pr.t == t;
#pragma unroll
          for (int k = 0; k < KR; ++k) {
            F[t][k] += on ? f[k] : 0.0;
            E[t][k] += on ? df[k] * uw : 0.0;
          }
        }
      }
      if (k0 < kA && pr.r2 < rcA2) {
        double f[KA], df[KA], g[NA], dg[NA];
        basis64<KA>(pr.r, m.rcA64, f, df);
        with_coeffs64<true>(m, p, par, ti, pr.t, [&](auto c) { channels64<NA, KA>(f, df, c, g, dg); });
        for_each_poly<NC>(pr.d[0] * ir, pr.d[1] * ir, pr.d[2] * ir, [&](int lm, double P) {
#pragma unroll
          for (int n = 0; n < NA; ++n) s[n * NC + lm] += g[n] * P;
        });
      }
    });
#pragma unroll
    for (int t = 0; t < TT; ++t) {
#pragma unroll
      for (int k = 0; k < KR; ++k) {
        F[t][k] = lanes_sum64(F[t][k]);
        E[t][k] = lanes_sum64(E[t][k]);
        if (k % kL64 == l) {
          C.F[t][k] = F[t][k];
          C.E[t][k] = E[t][k];
        }
      }
      if (MULTI && t >= T) continue;
      with_coeffs64<false>(m, p, par, ti, t, [&](auto c) {
#pragma unroll
        for (int n = 0; n < NR; ++n)
#pragma unroll
          for (int k = 0; k < KR; ++k) {
            q[n] += c[n * KR + k] * F[t][k];
            vr[n] += c[n * KR + k] * E[t][k];
          }
      });
    }
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) {
      s[k] = lanes_sum64(s[k]);
      if (k % kL64 == l) C.s[k] = s[k];
    }
    finish64<S>(s, q);
#pragma unroll
    for (int k = 0; k < D; ++k)
      if (k % kL64 == l) C.q[k] = q[k];
  }
  {
    // JVP of the accumulators: ds/dr . w = g' (u.w) P + g (grad P . w - l P (u.w)) / r
    double sd[NA * NC];
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) sd[k] = 0.0;
    if (w) {
      for_pairs64<MULTI>(b, i, l, kA, rcA2, [&](int, const Pair64& pr) {
        double f[KA], df[KA], g[NA], dg[NA], wd[3];
        basis64<KA>(pr.r, m.rcA64, f, df);
        with_coeffs64<true>(m, p, par, ti, pr.t, [&](auto c) { channels64<NA, KA>(f, df, c, g, dg); });
        weight_diff(w, N, i, pr.j, wd);
        const double ir = 1.0 / pr.r;
        const double u[3] = {pr.d[0] * ir, pr.d[1] * ir, pr.d[2] * ir};
        const double uw = u[0] * wd[0] + u[1] * wd[1] + u[2] * wd[2];
        for_each_poly_grad<NC>(u[0], u[1], u[2], [&](int lm, double P, double px, double py, double pz) {
          const double a = uw * P, bb = (px * wd[0] + py * wd[1] + pz * wd[2] - comp_l(lm) * P * uw) * ir;
#pragma unroll
          for (int n = 0; n < NA; ++n) sd[n * NC + lm] += dg[n] * a + g[n] * bb;
        });
      });
#pragma unroll
      for (int k = 0; k < NA * NC; ++k) sd[k] = lanes_sum64(sd[k]);
    }
#pragma unroll
    for (int k = 0; k < NA * NC; ++k)
      if (k % kL64 == l) C.sd[k] = sd[k];
    wave_lds_sync();
    double v[D];
#pragma unroll
    for (int k = 0; k < D; ++k) v[k] = k < NR ? vr[k < NR ? k : 0] : 0.0;
#pragma unroll
    for (int n = 0; n < NA; ++n) {
#pragma unroll
      for (int lm = 0; lm < NC; ++lm)
        v[NR + (comp_l(lm) - 1) * NA + n] += 2.0 * (double)kW[lm] * C.s[n * NC + lm] * sd[n * NC + lm];
      if constexpr (S::FB) {
        double q4, d5[5], s2[5], v4 = 0.0;
#pragma unroll
        for (int c = 0; c < 5; ++c) s2[c] = C.s[n * NC + 3 + c];
        fourbody64(s2, q4, d5);
#pragma unroll
        for (int c = 0; c < 5; ++c) v4 += d5[c] * sd[n * NC + 3 + c];
        v[NR + L3 * NA + n] = v4;
      }
    }
#pragma unroll
    for (int k = 0; k < D; ++k)
      if (k % kL64 == l) C.v[k] = v[k];
  }
  wave_lds_sync();
  // network
  for (int mu = l; mu < H; mu += kL64) {
    double h = -par.b0[mu], z = 0.0;
    for (int k = 0; k < D; ++k) {
      h += par.W0[mu * D + k] * (par.sigma[k] * C.q[k]);
      z += par.W0[mu * D + k] * (par.sigma[k] * C.v[k]);
    }
    const double t = tanh(h), d = 1.0 - t * t, w1 = par.w1[mu];
    C.be[mu] = valid ? w1 * d : 0.0;
    C.al[mu] = valid ? gE * w1 * d + 2.0 * z * w1 * t * d : 0.0;
    C.gw[mu] = valid ? gE * t - z * d : 0.0;
  }
  wave_lds_sync();
  for (int k = l; k < D; k += kL64) {
    double sa = 0.0, sb = 0.0;
    for (int mu = 0; mu < H; ++mu) {
      sa += par.W0[mu * D + k] * C.al[mu];
      sb += par.W0[mu * D + k] * C.be[mu];
    }
    C.sa[k] = sa;
    C.sb[k] = sb;
  }
  wave_lds_sync();
  // C_nlm and A_nlm in place of sd and s: channel n by lane n
  if (l < NA) {
    const int n = l;
    double d5[5] = {}, h5[5] = {}, s2[5], sd2[5];
    if constexpr (S::FB) {
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        s2[c] = C.s[n * NC + 3 + c];
        sd2[c] = C.sd[n * NC + 3 + c];
      }
      fourbody_dir64(s2, sd2, d5, h5);
    }
    const int k4 = S::FB ? NR + L3 * NA + n : 0;
    const double rho4 = par.sigma[k4] * C.sa[k4], fp4 = par.sigma[k4] * C.sb[k4];
#pragma unroll
    for (int lm = 0; lm < NC; ++lm) {
      const int k = NR + (comp_l(lm) - 1) * NA + n;
      const double rho = par.sigma[k] * C.sa[k], fp = par.sigma[k] * C.sb[k];
      const double s = C.s[n * NC + lm], sd = C.sd[n * NC + lm];
      double c = 2.0 * (double)kW[lm] * (rho * s - fp * sd);
      double a = -2.0 * (double)kW[lm] * fp * s;
      if (S::FB && comp_l(lm) == 2) {
        c += rho4 * d5[lm - 3] - fp4 * h5[lm - 3];
        a -= fp4 * d5[lm - 3];
      }
      C.s[n * NC + lm] = a;
      C.sd[n * NC + lm] = c;
    }
  }
  wave_lds_sync();
  // angular coefficients
  double gc[TT][NA * KA];
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int k = 0; k < NA * KA; ++k) gc[t][k] = 0.0;
  for_pairs64<MULTI>(b, i, l, kA, rcA2, [&](int, const Pair64& pr) {
    double wd[3], X[NA], Y[NA], Z[NA];
    weight_diff(w, N, i, pr.j, wd);
    const double ir = 1.0 / pr.r;
    const double u[3] = {pr.d[0] * ir, pr.d[1] * ir, pr.d[2] * ir};
    const double uw = u[0] * wd[0] + u[1] * wd[1] + u[2] * wd[2];
#pragma unroll
    for (int n = 0; n < NA; ++n) X[n] = Y[n] = Z[n] = 0.0;
    for_each_poly_grad<NC>(u[0], u[1], u[2], [&](int lm, double P, double px, double py, double pz) {
      const double bb = (px * wd[0] + py * wd[1] + pz * wd[2] - comp_l(lm) * P * uw) * ir;
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        const double a = C.s[n * NC + lm];
        X[n] += C.sd[n * NC + lm] * P;
        Y[n] += a * P;
        Z[n] += a * bb;
      }
    });
    double f[KA], df[KA];
    basis64<KA>(pr.r, m.rcA64, f, df);
#pragma unroll
    for (int n = 0; n < NA; ++n)
#pragma unroll
      for (int k = 0; k < KA; ++k) {
        const double t1 = f[k] * (X[n] + Z[n]) + df[k] * uw * Y[n];
#pragma unroll
        for (int t = 0; t < TT; ++t) gc[t][n * KA + k] += !MULTI || pr.t == t ? t1 : 0.0;
      }
  });
  wave_lds_sync();  // A and C are read no more
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int k = 0; k < NA * KA; ++k) {
      const double x = lanes_sum64(gc[t][k]);
      if (k % kL64 == l) C.gc[t][k] = x;
    }
  __syncthreads();
  // sums over the workgroup's centers, one thread to a parameter (centers past the system
  // hold zeros; the coefficients take the centers of their species only)
  const int oA = T * T * NR * KR, oS = oA + T * T * NA * KA, oW = oS + D, oB0 = oW + H * D, oW1 = oB0 + H,
            oB1 = oW1 + H;
  for (int e = threadIdx.x; e <= oB1; e += kBlock) {
    double sum = 0.0;
    for (int c = 0; c < kC64; ++c) {
      const Center64<S, MULTI>& A = ctr[c];
      double x;
      if (e < oA) {
        const int pr = e / (NR * KR), n = e / KR % NR, k = e % KR, t = pr % T;
        x = !MULTI || A.type == pr / T
                ? par.sigma[n] * A.sa[n] * A.F[t][k] - par.sigma[n] * A.sb[n] * A.E[t][k] : 0.0;
      } else if (e < oS) {
        const int u = e - oA, pr = u / (NA * KA);
        x = !MULTI || A.type == pr / T ? A.gc[pr % T][u % (NA * KA)] : 0.0;
      } else if (e < oW) {
        const int k = e - oS;
        x = A.q[k] * A.sa[k] - A.v[k] * A.sb[k];
      } else if (e < oB0) {
        const int mu = (e - oW) / D, k = (e - oW) % D;
        x = A.al[mu] * (par.sigma[k] * A.q[k]) - A.be[mu] * (par.sigma[k] * A.v[k]);
      } else if (e < oW1) {
        x = -A.al[e - oB0];
      } else if (e < oB1) {
        x = A.gw[e - oW1];
      } else {
        x = A.valid ? -gE : 0.0;
      }
      sum += x;
    }
    unsafeAtomicAdd(grad + e, sum);
  }
}

// soa_sorted[c][i] = aos_orig[perm[i]][c]
__global__ void k_gather_vec64(int64_t N, const int32_t* __restrict__ perm, const double* __restrict__ aos_orig,
                               double* __restrict__ soa_sorted) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int64_t o = perm[i];
#pragma unroll
  for (int c = 0; c < 3; ++c) soa_sorted[c * N + i] = aos_orig[3 * o + c];
}

__global__ void k_zero64(int64_t n, double* __restrict__ a) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) a[k] = 0.0;
}

}  // namespace

int eval64_rows(int64_t N) { return grid_blocks(N, kC64); }

namespace {

template <class S>
hipError_t launch64_shape(const ModelDev& m, const Model64& p, const EvalBuffers& b, double* U64, double* Fp64,
                          double* F64, hipStream_t st) {
  const int nb = eval64_rows(b.N);
  hipLaunchKernelGGL(k_zero64, dim3(grid_blocks(3 * b.N)), dim3(kBlock), 0, st, 3 * b.N, F64);
  if (m.T > 1) {
    hipLaunchKernelGGL((k_desc64<S, true>), dim3(nb), dim3(kBlock), 0, st, m, p, b, U64, Fp64);
    hipLaunchKernelGGL((k_force64<S, true>), dim3(nb), dim3(kBlock), 0, st, m, p, b, Fp64, F64);
  } else {
    hipLaunchKernelGGL((k_desc64<S, false>), dim3(nb), dim3(kBlock), 0, st, m, p, b, U64, Fp64);
    hipLaunchKernelGGL((k_force64<S, false>), dim3(nb), dim3(kBlock), 0, st, m, p, b, Fp64, F64);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_eval64(const ModelDev& m, const Model64& p, const EvalBuffers& b, double* U64, double* Fp64,
                         double* F64, hipStream_t st) {
  if (is_shape<FullShape>(m)) return launch64_shape<FullShape>(m, p, b, U64, Fp64, F64, st);
  if (is_shape<SurShape>(m)) return launch64_shape<SurShape>(m, p, b, U64, Fp64, F64, st);
  return hipErrorInvalidValue;
}

template <class S>
hipError_t grad64_shape(const ModelDev& m, const Model64& p, const EvalBuffers& b, const double* w, double gE,
                        double* grad, int64_t n_params, hipStream_t st) {
  hipLaunchKernelGGL(k_zero64, dim3(grid_blocks(n_params)), dim3(kBlock), 0, st, n_params, grad);
  const int nb = eval64_rows(b.N);
  if (m.T > 1)
    hipLaunchKernelGGL((k_grad64<S, true>), dim3(nb), dim3(kBlock), 0, st, m, p, b, w, gE, grad);
  else
    hipLaunchKernelGGL((k_grad64<S, false>), dim3(nb), dim3(kBlock), 0, st, m, p, b, w, gE, grad);
  return hipGetLastError();
}

hipError_t launch_grad64(const ModelDev& m, const Model64& p, const EvalBuffers& b, const double* gF_sorted,
                         double gE, double* grad, int64_t n_params, hipStream_t st) {
  if (is_shape<FullShape>(m)) return grad64_shape<FullShape>(m, p, b, gF_sorted, gE, grad, n_params, st);
  if (is_shape<SurShape>(m)) return grad64_shape<SurShape>(m, p, b, gF_sorted, gE, grad, n_params, st);
  return hipErrorInvalidValue;
}

hipError_t launch_gather_vec64(int64_t N, const int32_t* perm, const double* aos_orig, double* soa_sorted,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_gather_vec64, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, perm, aos_orig, soa_sorted);
  return hipGetLastError();
}

}  // namespace nep
