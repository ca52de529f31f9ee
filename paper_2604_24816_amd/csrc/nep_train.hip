// Differentiation of L = gE * E + sum_i gF_i . F_i with respect to the network
// parameters theta = (W0, b0, w1, b1), with respect to the expansion coefficients
// and the scaler, and the Adam update.
//
// With F = -dE/dx, sum_i gF_i . F_i = -sum_a dU_a/dq_a . v_a where
// v_a = sum_j dq_a/dr_aj . (gF_j - gF_a) is the descriptor JVP along gF.
// Writing q~ = sigma q, v~ = sigma v, h = W0 q~ - b0, t = tanh h, d = 1 - t^2 and
// z = W0 v~, the per-atom contributions are
//   dL/dW0 = alpha q~^T - beta v~^T,  alpha = gE w1 d + 2 z w1 t d,  beta = w1 d
//   dL/db0 = -alpha,  dL/dw1 = gE t - z d,  dL/db1 = -gE.
// With rho = sigma * (W0^T alpha) = dL/dq and -Fp = -sigma * (W0^T beta) = dL/dv
// (Section III.B names the expansion coefficients c trainable):
//  * scaler: dL/dsigma_k = q_k (W0^T alpha)_k - v_k (W0^T beta)_k;
//  * radial: q_n and v_n are linear in c through the basis sums over the neighbours
//    j of each species t, F_k = sum f_k(r_ij) and E_k = sum f'_k(r_ij) (u.w), so
//    dL/dc^{t_i t}_{nk} += rho_n F_k - Fp_n E_k;
//  * angular: with s_nlm, its JVP sd_nlm and the weights W_lm of q_nl,
//      A_nlm = 2 W_lm Fp_nl s_nlm,  C_nlm = 2 W_lm (rho_nl s_nlm - Fp_nl sd_nlm)
//    (plus, for the four-body term, Fp4 dq4/ds in A and rho4 dq4/ds - Fp4 (d^2q4/ds^2) sd
//    in C), and each pair adds f_k (X_n - Z_n) - f'_k (u.w) Y_n to dL/dc_nk, with
//    X_n = sum_lm C_nlm P_lm, Y_n = sum_lm A_nlm P_lm and
//    Z_n = sum_lm A_nlm (grad P_lm . w - l P_lm (u.w)) / r.
#include "nep_fast.h"

namespace nep {
namespace {

using namespace kern;

// A row of gradient sums: [W0 sums (hidden-major) | alpha | gE t - z d | cR | cA | sigma].
// Every workgroup of the gradient kernel stores a row of its own and the rows are summed in
// a fixed order, so that equal inputs give equal bits. The rows lie in the buffers that only
// an evaluation or a list build uses, one after the other: a workgroup has 16 centers or
// more, for which these hold 1,176 doubles and the list scratch 128 for every 16 entries
// of the radial capacity; a row takes 1,350 at most (two species), fewer where the lanes
// would not fit (train_lanes).
constexpr int kGradSegs = 4;
struct GradRows {
  double* base[kGradSegs];
  int end[kGradSegs];  // rows in the segments up to this one
  int len;             // doubles of a row
  __device__ __forceinline__ double* row(int r) const {
    double* p = base[0];
    int first = 0;
#pragma unroll
    for (int k = 1; k < kGradSegs; ++k)
      if (r >= end[k - 1]) {
        p = base[k];
        first = end[k - 1];
      }
    return p + (int64_t)(r - first) * len;
  }
};
GradRows grad_rows(const TrainBuffers& t, int len) {
  const int64_t N = t.e.N;
  double* const base[kGradSegs] = {t.gpart, reinterpret_cast<double*>(t.e.G), reinterpret_cast<double*>(t.e.rec),
                                   reinterpret_cast<double*>(t.e.rec1)};
  const int64_t size[kGradSegs] = {t.gpart_size, 60 * N, 8 * N, t.rec1_size};
  GradRows g;
  g.len = len;
  int rows = 0;
  for (int k = 0; k < kGradSegs; ++k) {
    rows += (int)(size[k] / len);
    g.base[k] = base[k];
    g.end[k] = rows;
  }
  return g;
}

// The force weights in sorted order, [N][3].
__global__ void k_train_prep(int64_t N, const int32_t* __restrict__ perm, const float* __restrict__ gF,
                             float* __restrict__ w) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  const int64_t o = perm[p];
  for (int c = 0; c < 3; ++c) w[3 * p + c] = gF[3 * o + c];
}

// The neighbours of one lane of a center: entries l, l + L, ... below k1, each with its FP64
// position, force weight (FORCE) and species loaded while the entry before is worked on.
template <bool MULTI, bool FORCE, int L, class Body>
__device__ __forceinline__ void for_each_train(const EvalBuffers& b, const float* __restrict__ w, int64_t i, int l,
                                               int k1, Body&& body) {
  if (k1 <= 0) return;
  struct Item {
    double x, y, z;
    float w0, w1, w2;
    int t;
  };
  const int64_t N = b.N;
  auto load = [&](int p) {
    const int32_t j = b.nbr[(uint64_t)(uint32_t)(p < k1 ? p : k1 - 1) * (uint64_t)N + i];
    Item q;
    q.x = b.x[j];
    q.y = b.x[N + j];
    q.z = b.x[2 * N + j];
    q.w0 = FORCE ? w[3 * (int64_t)j] : 0.f;
    q.w1 = FORCE ? w[3 * (int64_t)j + 1] : 0.f;
    q.w2 = FORCE ? w[3 * (int64_t)j + 2] : 0.f;
    q.t = MULTI ? b.type[j] : 0;
    return q;
  };
  Item q = load(l);
  for (int p = l; p < k1; p += L) {
    const Item n = load(p + L);
    body(p, q);
    q = n;
  }
}

// Gradients of the network parameters and, with COEF, of the coefficients and the scaler,
// each workgroup's sum over its centers into its row. Without a force term (FORCE false) there
// is no JVP: v, z, E_k, sd and what they enter are left out (a backward call of 37,044 atoms,
// network: 152 us with them, 76 without). L lanes share a center: one pass over its list gives the
// basis sums, the accumulators s and their JVP sd together (two accumulators per harmonic
// and channel: one wavefront per SIMD); the network runs on MFMA with the wavefront's
// centers as rows, as does the sum of the outer products over them; the angular
// coefficients take a second pass. Sums over a wavefront are FP32, over wavefronts and
// workgroups FP64.
// A thread per center, with the descriptors, the radial and the angular JVP each in a pass
// of their own and the descriptors computed again for the coefficients, took 287 us for
// the network's gradient of 32,000 atoms and 57 + 89 us for both of 4,000 atoms (l <= 2
// shape); with sincospi and coefficient gathers per pair in place of the tables.
template <class S, bool MULTI, bool COEF, bool FORCE, int L>
__global__ void __launch_bounds__(kBlock, 1)
k_train_grad(ModelDev m, EvalBuffers b, const float* __restrict__ w, double gE, GradRows rows) {
  constexpr int NR = S::NR, NA = S::NA, NC = S::NC, D = S::D, H = S::H, KR = S::KR, KA = S::KA;
  constexpr int TT = MULTI ? kMaxTypes : 1;
  constexpr int CW = 64 / L;                      // centers of a wavefront
  constexpr int RT = CW >= 16 ? CW / 16 : 1;      // their 16-row tiles
  constexpr int TILE = 16 * RT * kNetStride;
  constexpr int NCOEF = TT * TT * (NR * KR + NA * KA) + D;
  constexpr int kNet = 32 * 32 + 2 * 32;          // a wavefront's network sums
  static_assert(5 * TILE >= kNet, "the tiles hold a wavefront's network sums");
  __shared__ NetLds net;
  __shared__ PairTab<S, MULTI> tab;
  __shared__ float tiles[kBlock / 64][5 * TILE];  // q~, v~, h (alpha), z (beta), gE t - z d
  __shared__ float red[kBlock / 64][COEF ? NCOEF : 1];
  stage_network<S>(m, net);
  if constexpr (MULTI) stage_pairs<S>(m, tab);
  __syncthreads();
  const int64_t N = b.N;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t i = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * (kBlock / L) + threadIdx.x / L;
  const int l = threadIdx.x % L;
  const bool valid = i < N;
  const CutConst cutR = cut_const(m.rcR), cutA = cut_const(m.rcA);
  const float kDR = -0.5f * kPiF * cutR.rc_inv, kYR = 4.f * cutR.rc_inv;
  const float kDA = -0.5f * kPiF * cutA.rc_inv, kYA = 4.f * cutA.rc_inv;
  const double rcR2 = m.rcR64 * m.rcR64, rcA2 = m.rcA64 * m.rcA64;
  const double Lx = b.box[0], Ly = b.box[1], Lz = b.box[2];
  const double iLx = 1.0 / Lx, iLy = 1.0 / Ly, iLz = 1.0 / Lz;

  float q[D], v[D], s[NA * NC], sd[NA * NC];
  float Fk[TT][KR], Ek[TT][KR];  // this lane's part of the basis sums per neighbour species
#pragma unroll
  for (int k = 0; k < D; ++k) q[k] = v[k] = 0.f;
#pragma unroll
  for (int k = 0; k < NA * NC; ++k) s[k] = sd[k] = 0.f;
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int k = 0; k < KR; ++k) Fk[t][k] = Ek[t][k] = 0.f;
  int ti = 0, kA = 0;
  double xi = 0, yi = 0, zi = 0;
  float wi0 = 0.f, wi1 = 0.f, wi2 = 0.f;
  if (valid) {
    ti = MULTI ? b.type[i] : 0;
    xi = b.x[i];
    yi = b.x[N + i];
    zi = b.x[2 * N + i];
    if constexpr (FORCE) {
      wi0 = w[3 * i];
      wi1 = w[3 * i + 1];
      wi2 = w[3 * i + 2];
    }
    kA = angular_bound(b, i);
    // Fk, Ek hold sum f_c T_k and sum (f_c T_k)' (u.w) (k >= 1) and the k = 0 sums of f_c
    for_each_train<MULTI, FORCE, L>(b, w, i, l, radial_bound(b, i), [&](int p, const auto& e) {
      double ex, ey, ez;
      const double r2 = pair_r2_64(e.x, e.y, e.z, xi, yi, zi, Lx, Ly, Lz, iLx, iLy, iLz, ex, ey, ez);
      if (!(r2 < rcR2)) return;
      const float dx = (float)ex, dy = (float)ey, dz = (float)ez;
      float r, rinv;
      pair_r(dx, dy, dz, r, rinv);
      const float w0 = e.w0 - wi0, w1 = e.w1 - wi1, w2 = e.w2 - wi2;
      const float ux = dx * rinv, uy = dy * rinv, uz = dz * rinv;
      const float uw = ux * w0 + uy * w1 + uz * w2;
      {
        const RadialGeo g = radial_geo<FORCE>(r, cutR);
        const float df = FORCE ? kDR * g.c * uw : 0.f, xf = FORCE ? g.fc * (kYR * g.y) * uw : 0.f;
        float ft[TT], dt[TT], xt[TT];  // the factors for the neighbour's species, 0 for the others
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          const bool on = !MULTI || e.t == t;
          ft[t] = on ? g.fc : 0.f;
          dt[t] = on ? df : 0.f;
          xt[t] = on ? xf : 0.f;
          Fk[t][0] += ft[t];
          if constexpr (FORCE) Ek[t][0] += dt[t];
        }
        const float x2 = g.x + g.x;
        float Tm = 1.f, T = g.x, Um = 0.f, U = 1.f;  // T_{k-1}, T_k, U_{k-2}, U_{k-1}
#pragma unroll
        for (int k = 1; k < KR; ++k) {
          const float kU = (float)k * U;  // T_k'
#pragma unroll
          for (int t = 0; t < TT; ++t) {
            Fk[t][k] = fmaf(ft[t], T, Fk[t][k]);
            if constexpr (FORCE) Ek[t][k] = fmaf(dt[t], T, fmaf(xt[t], kU, Ek[t][k]));
          }
          const float Tn = fmaf(x2, T, -Tm), Un = fmaf(x2, U, -Um);
          Tm = T;
          T = Tn;
          Um = U;
          U = Un;
        }
      }
      if (p < kA && r2 < rcA2) {
        // ds_nlm . w = g_n' (u.w) P_lm + g_n (grad P_lm . w - l P_lm (u.w)) / r
        const RadialGeo g = radial_geo<FORCE>(r, cutA);
        float gn[NA], gu[NA];
        if constexpr (MULTI) radial_cd_tab<S, FORCE>(g.x, ang_tab(tab, ti, e.t), gn, gu);
        else if constexpr (FORCE) radial_cd_fast<NA, KA>(g.x, uniform_coeffs(m.hA), gn, gu);
        else radial_g_fast<NA, KA>(1.f, g.x, uniform_coeffs(m.hA), gn);
        const float df = FORCE ? kDA * g.c * uw : 0.f, xf = FORCE ? g.fc * (kYA * g.y) * uw : 0.f;
#pragma unroll
        for (int n = 0; n < NA; ++n) {
          if constexpr (FORCE) gu[n] = fmaf(df, gn[n], xf * gu[n]);
          gn[n] *= g.fc;
        }
        if constexpr (FORCE) {
          for_each_poly_grad<NC>(ux, uy, uz, [&](int lm, float P, auto px, auto py, auto pz) {
            const float bb = fmac(w0, px, fmac(w1, py, fmac(w2, pz, -(float)comp_l(lm) * P * uw))) * rinv;
#pragma unroll
            for (int n = 0; n < NA; ++n) {
              s[n * NC + lm] = fmaf(gn[n], P, s[n * NC + lm]);
              sd[n * NC + lm] = fmaf(gu[n], P, fmaf(gn[n], bb, sd[n * NC + lm]));
            }
          });
        } else {
          for_each_poly<NC>(ux, uy, uz, [&](int lm, float P) {
#pragma unroll
            for (int n = 0; n < NA; ++n) s[n * NC + lm] = fmaf(gn[n], P, s[n * NC + lm]);
          });
        }
      }
    });
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      // sum f_k = (sum f_c T_k + sum f_c) / 2, and its derivative likewise
#pragma unroll
      for (int k = 1; k < KR; ++k) {
        Fk[t][k] = 0.5f * (Fk[t][k] + Fk[t][0]);
        if constexpr (FORCE) Ek[t][k] = 0.5f * (Ek[t][k] + Ek[t][0]);
      }
      auto add = [&](auto c) {
#pragma unroll
        for (int n = 0; n < NR; ++n)
#pragma unroll
          for (int k = 0; k < KR; ++k) {
            q[n] = fmaf(c[n * KR + k], Fk[t][k], q[n]);
            if constexpr (FORCE) v[n] = fmaf(c[n * KR + k], Ek[t][k], v[n]);
          }
      };
      if constexpr (MULTI) add(tab.rad + (ti * kMaxTypes + t) * (NR * KR));
      else add(uniform_coeffs(m.cR));
    }
#pragma unroll
    for (int n = 0; n < NR; ++n) {
      q[n] = lanes_sum<L>(q[n]);
      if constexpr (FORCE) v[n] = lanes_sum<L>(v[n]);
    }
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) {
      s[k] = lanes_sum<L>(s[k]);
      if constexpr (FORCE) sd[k] = lanes_sum<L>(sd[k]);
    }
    desc_finish<S>(s, q);
    if constexpr (FORCE) {
#pragma unroll
      for (int n = 0; n < NA; ++n)
#pragma unroll
        for (int lm = 0; lm < NC; ++lm) {
          const int k = NR + (comp_l(lm) - 1) * NA + n;
          v[k] = fmaf(2.f * kW[lm] * s[n * NC + lm], sd[n * NC + lm], v[k]);
        }
    }
    if constexpr (FORCE && S::FB) {
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        float d4[5];
        fourbody_ds(s + n * NC, d4);
#pragma unroll
        for (int c = 0; c < 5; ++c) v[NR + S::L3 * NA + n] = fmaf(d4[c], sd[n * NC + 3 + c], v[NR + S::L3 * NA + n]);
      }
    }
  }
  // network: rows of q~ and v~, then h and z, then alpha and beta (zero for the rows of no center)
  float* tq = tiles[wave];
  float* tv = tq + TILE;
  float* ta = tq + 2 * TILE;
  float* tb = tq + 3 * TILE;
  float* tg = tq + 4 * TILE;
  const int row = (lane / L) * kNetStride;
#pragma unroll
  for (int k = 0; k < 32; ++k)
    if ((k & (L - 1)) == l) {
      tq[row + k] = k < D ? q[k < D ? k : 0] * net.sigma[k] : 0.f;
      if constexpr (FORCE) tv[row + k] = k < D ? v[k < D ? k : 0] * net.sigma[k] : 0.f;
    }
  net_product<RT, true>(tq, ta, net);
  if constexpr (FORCE) net_product<RT, true>(tv, tb, net);
  const float gEf = (float)gE;
#pragma unroll
  for (int mu0 = 0; mu0 < 32; mu0 += L) {
    const int mu = mu0 + l;
    const float t = tanhf(ta[row + mu] - net.b0[mu]), z = FORCE ? tb[row + mu] : 0.f, w1 = net.w1[mu];
    const float d = 1.f - t * t, w1d = w1 * d;
    ta[row + mu] = valid ? (FORCE ? fmaf(gEf, w1d, 2.f * z * w1 * t * d) : gEf * w1d) : 0.f;
    if constexpr (FORCE) tb[row + mu] = valid ? w1d : 0.f;
    tg[row + mu] = valid ? (FORCE ? fmaf(gEf, t, -z * d) : gEf * t) : 0.f;
  }
  wave_lds_sync();
  // sum over the wavefront's centers of alpha q~^T - beta v~^T, and of alpha and gE t - z d
  floatx4 acc[2][2];
#pragma unroll
  for (int R = 0; R < 2; ++R)
#pragma unroll
    for (int C = 0; C < 2; ++C) acc[R][C] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int pass = 0; pass < (FORCE ? 2 : 1); ++pass)
#pragma unroll
    for (int kb = 0; kb < CW / 4; ++kb) {
      const int c0 = (4 * kb + lk) * kNetStride;
      float aop[2], bop[2];
#pragma unroll
      for (int R = 0; R < 2; ++R) aop[R] = pass == 0 ? ta[c0 + 16 * R + lr] : -tb[c0 + 16 * R + lr];
#pragma unroll
      for (int C = 0; C < 2; ++C) bop[C] = pass == 0 ? tq[c0 + 16 * C + lr] : tv[c0 + 16 * C + lr];
#pragma unroll
      for (int R = 0; R < 2; ++R)
#pragma unroll
        for (int C = 0; C < 2; ++C)
          acc[R][C] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[R], bop[C], acc[R][C], 0, 0, 0);
    }
  float ca = 0.f, cb = 0.f;
  if (lane < 32)
    for (int c = 0; c < CW; ++c) {
      ca += ta[c * kNetStride + lane];
      cb += tg[c * kNetStride + lane];
    }
  if constexpr (COEF) {
    constexpr int oA = TT * TT * NR * KR, oS = oA + TT * TT * NA * KA;
    float* rw = red[wave];
    // the sum of x over the wavefront's lanes whose center has species tc, to entry e
    auto total = [&](float x, int e) {
      x = wave_sum_last(x);
      if (lane == 63) rw[e] = x;
    };
    auto total_by_type = [&](float x, int e, int stride) {
      if constexpr (MULTI) {
#pragma unroll
        for (int tc = 0; tc < TT; ++tc) total(ti == tc ? x : 0.f, e + tc * stride);
      } else {
        total(x, e);
      }
    };
    net_product<RT, false>(ta, ta, net);
    if constexpr (FORCE) net_product<RT, false>(tb, tb, net);
    // dL/dq and dU/dq of the lane's center (zero where there is none)
    float rho[D], fp[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const float sa = ta[row + k], sb = FORCE ? tb[row + k] : 0.f;
      rho[k] = net.sigma[k] * sa;
      fp[k] = net.sigma[k] * sb;
      total((k & (L - 1)) == l ? (FORCE ? q[k] * sa - v[k] * sb : q[k] * sa) : 0.f, oS + k);
    }
    // radial coefficients [t_i][t][n][k], linear in the lanes' parts of the basis sums
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int n = 0; n < NR; ++n)
#pragma unroll
        for (int k = 0; k < KR; ++k)
          total_by_type(FORCE ? rho[n] * Fk[t][k] - fp[n] * Ek[t][k] : rho[n] * Fk[t][k], (t * NR + n) * KR + k,
                        TT * NR * KR);
    // angular coefficients A (in place of s) and C (in place of sd)
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      float d4[5] = {}, h4[5] = {};
      if constexpr (S::FB) {
        fourbody_ds(s + n * NC, d4);
        if constexpr (FORCE) fourbody_ds_dir(s + n * NC, sd + n * NC, h4);
      }
#pragma unroll
      for (int lm = 0; lm < NC; ++lm) {
        const int k = NR + (comp_l(lm) - 1) * NA + n;
        float a = FORCE ? 2.f * kW[lm] * fp[k] * s[n * NC + lm] : 0.f;
        float c = FORCE ? 2.f * kW[lm] * (rho[k] * s[n * NC + lm] - fp[k] * sd[n * NC + lm])
                        : 2.f * kW[lm] * (rho[k] * s[n * NC + lm]);
        if constexpr (S::FB) {
          if (comp_l(lm) == 2) {
            const int k4 = NR + S::L3 * NA + n;
            if constexpr (FORCE) a = fmaf(fp[k4], d4[lm - 3], a);
            c += FORCE ? rho[k4] * d4[lm - 3] - fp[k4] * h4[lm - 3] : rho[k4] * d4[lm - 3];
          }
        }
        s[n * NC + lm] = a;
        sd[n * NC + lm] = c;
      }
    }
    float gc[TT][NA * KA];
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int k = 0; k < NA * KA; ++k) gc[t][k] = 0.f;
    for_each_train<MULTI, FORCE, L>(b, w, i, l, kA, [&](int, const auto& e) {
      double ex, ey, ez;
      const double r2 = pair_r2_64(e.x, e.y, e.z, xi, yi, zi, Lx, Ly, Lz, iLx, iLy, iLz, ex, ey, ez);
      if (!(r2 < rcA2)) return;
      const float dx = (float)ex, dy = (float)ey, dz = (float)ez;
      float r, rinv;
      pair_r(dx, dy, dz, r, rinv);
      const float w0 = e.w0 - wi0, w1 = e.w1 - wi1, w2 = e.w2 - wi2;
      const float ux = dx * rinv, uy = dy * rinv, uz = dz * rinv;
      const float uw = ux * w0 + uy * w1 + uz * w2;
      float X[NA], Y[NA], Z[NA];
#pragma unroll
      for (int n = 0; n < NA; ++n) X[n] = Y[n] = Z[n] = 0.f;
      if constexpr (FORCE) {
        for_each_poly_grad<NC>(ux, uy, uz, [&](int lm, float P, auto px, auto py, auto pz) {
          const float bb = fmac(w0, px, fmac(w1, py, fmac(w2, pz, -(float)comp_l(lm) * P * uw))) * rinv;
#pragma unroll
          for (int n = 0; n < NA; ++n) {
            X[n] = fmaf(sd[n * NC + lm], P, X[n]);
            Y[n] = fmaf(s[n * NC + lm], P, Y[n]);
            Z[n] = fmaf(s[n * NC + lm], bb, Z[n]);
          }
        });
      } else {
        for_each_poly<NC>(ux, uy, uz, [&](int lm, float P) {
#pragma unroll
          for (int n = 0; n < NA; ++n) X[n] = fmaf(sd[n * NC + lm], P, X[n]);
        });
      }
      const RadialGeo g = radial_geo<FORCE>(r, cutA);
      // f_k and f'_k (u.w), from T_k and T_k' = k U_{k-1}
      const float df = FORCE ? kDA * g.c * uw : 0.f, xf = FORCE ? g.fc * (kYA * g.y) * uw : 0.f;
      const float x2 = g.x + g.x;
      float Tm = 0.f, T = 1.f, Um = 0.f, U = 0.f;
#pragma unroll
      for (int k = 0; k < KA; ++k) {
        const float f = 0.5f * g.fc * (T + 1.f);
        const float fd = FORCE ? 0.5f * fmaf(df, T + 1.f, xf * ((float)k * U)) : 0.f;
#pragma unroll
        for (int n = 0; n < NA; ++n) {
          const float t1 = FORCE ? fmaf(f, X[n] - Z[n], -fd * Y[n]) : f * X[n];
#pragma unroll
          for (int t = 0; t < TT; ++t) gc[t][n * KA + k] += !MULTI || e.t == t ? t1 : 0.f;
        }
        const float Tn = k == 0 ? g.x : fmaf(x2, T, -Tm);
        const float Un = k == 0 ? 1.f : (k == 1 ? x2 : fmaf(x2, U, -Um));
        Tm = T;
        T = Tn;
        Um = U;
        U = Un;
      }
    });
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int n = 0; n < NA; ++n)
#pragma unroll
        for (int k = 0; k < KA; ++k)
          total_by_type(gc[t][n * KA + k], oA + (t * NA + n) * KA + k, TT * NA * KA);
  }
  // the four wavefronts in FP64, then the workgroup's row
  __syncthreads();
#pragma unroll
  for (int R = 0; R < 2; ++R)
#pragma unroll
    for (int C = 0; C < 2; ++C)
#pragma unroll
      for (int r = 0; r < 4; ++r) tq[(16 * R + 4 * lk + r) * 32 + 16 * C + lr] = acc[R][C][r];
  if (lane < 32) {
    tq[32 * 32 + lane] = ca;
    tq[32 * 32 + 32 + lane] = cb;
  }
  __syncthreads();
  double* out = rows.row(blockIdx.x);
  auto put = [&](int e, float a0, float a1, float a2, float a3) {
    out[e] = ((double)a0 + (double)a1) + ((double)a2 + (double)a3);
  };
  for (int e = threadIdx.x; e < H * D + 2 * H; e += kBlock) {
    const int u = e - H * D;
    const int src = u < 0 ? (e / D) * 32 + e % D : (u < H ? 32 * 32 + u : 32 * 32 + 32 + u - H);
    put(e, tiles[0][src], tiles[1][src], tiles[2][src], tiles[3][src]);
  }
  if constexpr (COEF)
    for (int e = threadIdx.x; e < NCOEF; e += kBlock)
      put(H * D + 2 * H + e, red[0][e], red[1][e], red[2][e], red[3][e]);
}

// More than kGradGroups rows are first summed in that many groups of `per` rows, each into
// its first one. Four threads to an entry, each a quarter of the rows in order.
constexpr int kGradGroups = 256;
__global__ void __launch_bounds__(kBlock) k_grad_groups(GradRows rows, int nrows, int per) {
  __shared__ double sh[kBlock];
  constexpr int E = kBlock / 4;
  const int e = blockIdx.x * E + threadIdx.x % E, part = threadIdx.x / E;
  const int first = blockIdx.y * per, end = first + per < nrows ? first + per : nrows;
  double sum = 0.0;
  if (e < rows.len) {
#pragma unroll 4
    for (int r = first + part; r < end; r += 4) sum += rows.row(r)[e];
  }
  sh[threadIdx.x] = sum;
  __syncthreads();
  const int t = threadIdx.x;
  if (part == 0 && e < rows.len && first < end) rows.row(first)[e] = (sh[t] + sh[t + E]) + (sh[t + 2 * E] + sh[t + 3 * E]);
}

// The gradient from rows 0, per, 2 per, ... below nrows, in packed order: [cR | cA | sigma]
// first when ncoef > 0, then [W0 | b0 | w1 | b1]. kFinishParts threads to an entry, each every
// kFinishParts-th row in order (eight loads in flight: the kernel is the latency of rows that
// other dies wrote), then those sums in a fixed order. At most kGradGroups rows.
constexpr int kFinishParts = 32, kFinishEntries = kBlock / kFinishParts;
__global__ void __launch_bounds__(kBlock)
k_grad_finish(GradRows rows, int nrows, int per, int H, int D, int ncoef, double gE, int64_t N,
              float* __restrict__ grad, int accumulate) {
  __shared__ double sh[kBlock / 64][kFinishEntries];
  const int lane_e = threadIdx.x % kFinishEntries, part = threadIdx.x / kFinishEntries;
  const int e = blockIdx.x * kFinishEntries + lane_e;
  const int G = H * D + 2 * H + 1;
  const int u = e - ncoef;  // entry of the network block
  const int src = u < 0 ? G - 1 + e : u;
  const bool on = e < ncoef + G - 1;
  double v[kGradGroups / kFinishParts], sum = 0.0;
#pragma unroll
  for (int k = 0; k < kGradGroups / kFinishParts; ++k) {
    const int r = (part + k * kFinishParts) * per;
    v[k] = on && r < nrows ? rows.row(r)[src] : 0.0;
  }
#pragma unroll
  for (int k = 0; k < kGradGroups / kFinishParts; ++k) sum += v[k];
#pragma unroll
  for (int o = kFinishEntries; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) < kFinishEntries) sh[threadIdx.x >> 6][lane_e] = sum;
  __syncthreads();
  if (threadIdx.x >= kFinishEntries || e >= ncoef + G) return;
  double out = (sh[0][lane_e] + sh[1][lane_e]) + (sh[2][lane_e] + sh[3][lane_e]);
  if (u >= H * D && u < H * D + H) out = -out;  // dL/db0 = -sum alpha
  if (u == G - 1) out = -gE * (double)N;
  grad[e] = accumulate ? (float)((double)grad[e] + out) : (float)out;
}

__global__ void k_adam(float* __restrict__ theta, const float* __restrict__ g, float* __restrict__ m1,
                       float* __restrict__ m2, int64_t n, double c1, double c2, double lr, double b1,
                       double b2, double eps) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const double gk = g[k];
  const double a = b1 * (double)m1[k] + (1.0 - b1) * gk;
  const double b = b2 * (double)m2[k] + (1.0 - b2) * gk * gk;
  m1[k] = (float)a;
  m2[k] = (float)b;
  theta[k] = (float)((double)theta[k] - lr * (a / c1) / (sqrt(b / c2) + eps));
}

// Lanes per center: as many as keep one wavefront (what the full shape's registers allow)
// on each of the chip's 1,024 SIMDs; above that the fewest, since every lane more costs its
// share of the sums over lanes. The l <= 2 shapes fit two wavefronts and stay at four lanes.
// us of a backward call, network and coefficients:
//             full shape, L = 2     4    16    l <= 2, L = 2     4    16
//   4,000                   149    95    53               43    36    30
//   8,788                   142    87   125               43    35    48
//   32,000                  150   168   307               45    43    92
//   256,000                1081  1244  2359              272   231   623
// Sixteen lanes need a row for every 16 centers: where the list scratch of a small radial
// capacity is too short for a model of many coefficients, four lanes, whose rows always fit.
template <class S>
int train_lanes(int64_t N, const GradRows& rows) {
  constexpr int64_t kLanes = 65536;
  if (N * 16 <= kLanes && grid_blocks(N, kBlock / 16) <= rows.end[kGradSegs - 1]) return 16;
  return N * 4 <= kLanes || S::L3 <= 2 ? 4 : 2;
}

template <class S, bool MULTI, bool COEF, bool FORCE>
void launch_grad(const ModelDev& m, const TrainBuffers& t, int L, int nb, const GradRows& rows, hipStream_t st) {
  const dim3 grid(nb), block(kBlock);
  if (L == 16)
    hipLaunchKernelGGL((k_train_grad<S, MULTI, COEF, FORCE, 16>), grid, block, 0, st, m, t.e, t.w, t.gE, rows);
  else if (L == 4)
    hipLaunchKernelGGL((k_train_grad<S, MULTI, COEF, FORCE, 4>), grid, block, 0, st, m, t.e, t.w, t.gE, rows);
  else if constexpr (S::L3 > 2)
    hipLaunchKernelGGL((k_train_grad<S, MULTI, COEF, FORCE, 2>), grid, block, 0, st, m, t.e, t.w, t.gE, rows);
}

template <class S, bool COEF>
hipError_t launch_backward_shape(const ModelDev& m, const TrainBuffers& t, hipStream_t st) {
  const int64_t N = t.e.N;
  const int ncoef = COEF ? m.T * m.T * (m.nR * m.kR + m.nA * m.kA) + m.D : 0;
  const int net = m.H * m.D + 2 * m.H;
  const GradRows rows = grad_rows(t, net + ncoef);
  const int L = train_lanes<S>(N, rows);
  const int nb = grid_blocks(N, kBlock / L);
  if (nb > rows.end[kGradSegs - 1]) return hipErrorInvalidValue;
  if (t.gF) {
    hipLaunchKernelGGL(k_train_prep, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, t.perm, t.gF, t.w);
    if (m.T > 1) launch_grad<S, true, COEF, true>(m, t, L, nb, rows, st);
    else launch_grad<S, false, COEF, true>(m, t, L, nb, rows, st);
  } else {
    if (m.T > 1) launch_grad<S, true, COEF, false>(m, t, L, nb, rows, st);
    else launch_grad<S, false, COEF, false>(m, t, L, nb, rows, st);
  }
  const int per = (nb + kGradGroups - 1) / kGradGroups;
  if (per > 1)
    hipLaunchKernelGGL(k_grad_groups, dim3(grid_blocks(rows.len, kBlock / 4), (nb + per - 1) / per), dim3(kBlock), 0, st,
                       rows, nb, per);
  hipLaunchKernelGGL(k_grad_finish, dim3(grid_blocks(ncoef + net + 1, kFinishEntries)), dim3(kBlock), 0, st, rows, nb, per,
                     m.H, m.D, ncoef, t.gE, N, t.grad, t.accumulate);
  return hipGetLastError();
}

// The model with every parameter read from a packed FP32 vector
// [cR | cA | sigma | W0 | b0 | w1 | b1].
ModelDev with_params(const ModelDev& m, const float* p) {
  ModelDev mp = m;
  mp.cR = p;
  mp.cA = mp.cR + m.T * m.T * m.nR * m.kR;
  mp.sigma = mp.cA + m.T * m.T * m.nA * m.kA;
  mp.W0 = mp.sigma + m.D;
  mp.b0 = mp.W0 + m.H * m.D;
  mp.w1 = mp.b0 + m.H;
  mp.b1 = mp.w1 + m.H;
  return mp;
}

ModelDev with_theta(const ModelDev& m, const float* theta) {
  ModelDev mt = m;
  const int G = m.H * m.D;
  mt.W0 = theta;
  mt.b0 = theta + G;
  mt.w1 = theta + G + m.H;
  mt.b1 = theta + G + 2 * m.H;
  return mt;
}

}  // namespace

hipError_t launch_adam(float* theta, const float* g, float* m1, float* m2, int64_t n, int64_t t, double lr,
                       double b1, double b2, double eps, hipStream_t st) {
  const double c1 = 1.0 - pow(b1, (double)t);
  const double c2 = 1.0 - pow(b2, (double)t);
  hipLaunchKernelGGL(k_adam, dim3(grid_blocks(n)), dim3(kBlock), 0, st, theta, g, m1, m2, n, c1, c2, lr, b1,
                     b2, eps);
  return hipGetLastError();
}

hipError_t launch_train_forward(const ModelDev& m, const float* theta, const EvalBuffers& b, hipStream_t st) {
  return launch_eval(with_theta(m, theta), 0, b, st);
}

// The model with every parameter taken from `params` and its derived radial tables, which the
// kernels read the coefficients through, built from this vector.
static hipError_t params_model(const ModelDev& m, const float* params, ModelDev& mp, hipStream_t st) {
  mp = with_params(m, params);
  mp.hR = m.hscratch;
  mp.hA = m.hscratch + (int64_t)m.T * m.T * m.nR * (2 * m.kR - 1);
  return launch_derive_coeffs(m.T, m.nR, m.kR, m.nA, m.kA, mp.cR, mp.cA, m.hscratch, const_cast<float*>(mp.hA), st);
}

hipError_t launch_train_forward_params(const ModelDev& m, const float* params, const EvalBuffers& b,
                                       hipStream_t st) {
  ModelDev mp;
  const hipError_t e = params_model(m, params, mp, st);
  return e != hipSuccess ? e : launch_eval(mp, 0, b, st);
}

hipError_t launch_train_backward_params(const ModelDev& m, const TrainBuffers& t, hipStream_t st) {
  ModelDev mp;
  const hipError_t e = params_model(m, t.theta, mp, st);
  if (e != hipSuccess) return e;
  if (is_shape<FullShape>(mp)) return launch_backward_shape<FullShape, true>(mp, t, st);
  if (is_shape<SurShape>(mp)) return launch_backward_shape<SurShape, true>(mp, t, st);
  return hipErrorInvalidValue;
}

hipError_t launch_train_backward(const ModelDev& m, const TrainBuffers& t, hipStream_t st) {
  const ModelDev mt = with_theta(m, t.theta);
  if (is_shape<FullShape>(mt)) return launch_backward_shape<FullShape, false>(mt, t, st);
  if (is_shape<SurShape>(mt)) return launch_backward_shape<SurShape, false>(mt, t, st);
  return hipErrorInvalidValue;
}

}  // namespace nep
