// NEP energy/force evaluation on gfx950: two kernels per force evaluation, one thread per
// center, or in small systems L = 2 to 16 lanes per center that take its list entries in
// turn (desc_lanes, force_lanes).
//
//   k_desc_net  (256-thread workgroups)
//     1. radial descriptors q_n = sum_j g_n(r_ij) (Section III.B) and angular
//        accumulators s_nlm = sum_j g_n(r_ij) P_lm(u_ij) for every channel n in one
//        pass over the center's list with skin, each visited entry's FP32 r^2 tested
//        against the true cutoffs (Algorithm 1's geometry reuse with the channel tile
//        equal to all n_max+1 channels); from them q_nl = sum_m W_lm s_nlm^2 and the
//        four-body invariant tr(S_n^3);
//     2. the network U_i = w1 . tanh(W0 q~ - b0) - b1 and its gradient
//        dU/dq~ = W0^T (w1 (1 - tanh^2)) as two 64-row MFMA products per
//        wavefront (Section V.B Optimization 1, Fig. 2c), operands staged
//        through LDS; FP32 MFMA or bfloat16 MFMA with FP32 accumulation;
//     3. per-atom dU/ds_nlm is written for the force kernel, and the atom's whole
//        neighbour record (its position and radial force coefficients).
//     Neighbour positions are gathered from the 16-byte position array.
//   k_force
//     radial pair forces by gather (F_i += sum_j [dU_i/dr_ij - dU_j/dr_ji]
//     with the neighbour's radial coefficients read from its record), angular and
//     four-body pair forces from dU/ds by scatter into the neighbours (Section V.B
//     Optimization 1: no temporary per-pair force buffer; an LDS copy of the tile's
//     halo, or global atomics where it does not fit), and the virial
//     W_ab = -sum r_a dU_i/dr_b; the tile's energy (the U_i the descriptor kernel
//     wrote) and virial are summed per workgroup in FP64.
//   Pair arithmetic in both comes from nep_fast.h.
#include "nep_fast.h"

namespace nep {
namespace {

using namespace kern;

// ------------------------------------------------------------------------ network
// The network's operand tiles are private to a wavefront, so its lanes only have to see
// each other's LDS writes (wave_lds_sync), not a workgroup barrier: the wavefronts of a
// workgroup leave their descriptor loops independently.

// One wavefront evaluates the network for its 64 centers. qs[lane][v] holds the
// scaled descriptor of the lane's center on entry; on exit fp[v] = dU/dq~ and the
// return value is U. lds: this wavefront's 64 x kNetStride float tile.
template <class S, int PREC>
__device__ __forceinline__ float network_wave(const ModelDev& m, const float* qs, float* fp, float* lds,
                                              const float* __restrict__ W0, const float* __restrict__ b0,
                                              const float* __restrict__ w1, float b1) {
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15;   // row / column within a 16-wide tile
  const int lk = lane >> 4;   // k group
  float* row = lds + lane * kNetStride;
#pragma unroll
  for (int v = 0; v < 32; ++v) row[v] = v < S::D ? qs[v] : 0.f;
  wave_lds_sync();
  floatx4 acc[4][2];
#pragma unroll
  for (int R = 0; R < 4; ++R)
#pragma unroll
    for (int C = 0; C < 2; ++C) acc[R][C] = floatx4{0.f, 0.f, 0.f, 0.f};
  if constexpr (PREC == 0) {
    // h[center][hidden] = sum_desc q~[center][desc] W0[hidden][desc], K = 32 in 8 steps of 4.
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
      const int dcol = 4 * kb + lk;
      float bop[2];
#pragma unroll
      for (int C = 0; C < 2; ++C) {
        const int hid = 16 * C + lr;
        bop[C] = (hid < S::H && dcol < S::D) ? W0[hid * S::D + dcol] : 0.f;
      }
#pragma unroll
      for (int R = 0; R < 4; ++R) {
        const float aop = lds[(16 * R + lr) * kNetStride + dcol];
#pragma unroll
        for (int C = 0; C < 2; ++C)
          acc[R][C] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop, bop[C], acc[R][C], 0, 0, 0);
      }
    }
  } else {
    bf16x8 bop[2];
#pragma unroll
    for (int C = 0; C < 2; ++C) {
      const int hid = 16 * C + lr;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int dcol = 8 * lk + e;
        bop[C][e] = bits_to_bf16((hid < S::H && dcol < S::D) ? m.W0bf[hid * S::D + dcol] : (uint16_t)0);
      }
    }
#pragma unroll
    for (int R = 0; R < 4; ++R) {
      bf16x8 aop;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        aop[e] = bits_to_bf16(f32_to_bf16_bits(lds[(16 * R + lr) * kNetStride + 8 * lk + e]));
#pragma unroll
      for (int C = 0; C < 2; ++C)
        acc[R][C] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bop[C], acc[R][C], 0, 0, 0);
    }
  }
  wave_lds_sync();
  // D layout: lane holds rows 4*lk + r of column lr.
#pragma unroll
  for (int R = 0; R < 4; ++R)
#pragma unroll
    for (int C = 0; C < 2; ++C)
#pragma unroll
      for (int r = 0; r < 4; ++r) lds[(16 * R + 4 * lk + r) * kNetStride + 16 * C + lr] = acc[R][C][r];
  wave_lds_sync();
  float U = -b1;
  float a1[32];
#pragma unroll
  for (int mu = 0; mu < 32; ++mu) {
    if (mu < S::H) {
      const float t = tanh_fast(row[mu] - b0[mu]);
      U = fmaf(w1[mu], t, U);
      a1[mu] = w1[mu] * (1.f - t * t);
    } else {
      a1[mu] = 0.f;
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int mu = 0; mu < 32; ++mu) row[mu] = a1[mu];
  wave_lds_sync();
#pragma unroll
  for (int R = 0; R < 4; ++R)
#pragma unroll
    for (int C = 0; C < 2; ++C) acc[R][C] = floatx4{0.f, 0.f, 0.f, 0.f};
  if constexpr (PREC == 0) {
    // Fp[center][desc] = sum_hidden a[center][hidden] W0[hidden][desc].
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
      const int hid = 4 * kb + lk;
      float bop[2];
#pragma unroll
      for (int C = 0; C < 2; ++C) {
        const int dcol = 16 * C + lr;
        bop[C] = (hid < S::H && dcol < S::D) ? W0[hid * S::D + dcol] : 0.f;
      }
#pragma unroll
      for (int R = 0; R < 4; ++R) {
        const float aop = lds[(16 * R + lr) * kNetStride + hid];
#pragma unroll
        for (int C = 0; C < 2; ++C)
          acc[R][C] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop, bop[C], acc[R][C], 0, 0, 0);
      }
    }
  } else {
    bf16x8 bop[2];
#pragma unroll
    for (int C = 0; C < 2; ++C) {
      const int dcol = 16 * C + lr;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int hid = 8 * lk + e;
        bop[C][e] = bits_to_bf16((hid < S::H && dcol < S::D) ? m.W0bf[hid * S::D + dcol] : (uint16_t)0);
      }
    }
#pragma unroll
    for (int R = 0; R < 4; ++R) {
      bf16x8 aop;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        aop[e] = bits_to_bf16(f32_to_bf16_bits(lds[(16 * R + lr) * kNetStride + 8 * lk + e]));
#pragma unroll
      for (int C = 0; C < 2; ++C)
        acc[R][C] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bop[C], acc[R][C], 0, 0, 0);
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int R = 0; R < 4; ++R)
#pragma unroll
    for (int C = 0; C < 2; ++C)
#pragma unroll
      for (int r = 0; r < 4; ++r) lds[(16 * R + 4 * lk + r) * kNetStride + 16 * C + lr] = acc[R][C][r];
  wave_lds_sync();
#pragma unroll
  for (int v = 0; v < S::D; ++v) fp[v] = row[v];
  return U;
}

// ------------------------------------------------------------------------ descriptors
// Radial descriptors q[0..NR) and angular accumulators s[NA][NC] of center i over the
// pairs inside the true cutoffs, all channels in one pass over the list with skin
// (geometry computed once per pair and reused for every n). The radial descriptors are
// linear in the basis sums over the neighbours of each species t, q_n = sum_t sum_k c^t_nk
// sum_j f_k(r_ij), with sum_j f_k = (sum_j f_c T_k + sum_j f_c) / 2, so a pair adds f_c and
// f_c T_k (k >= 1). Returns the pair counts and the number of pairs inside the
// ZBL radius (nz), which the loops only count; a center with any visits its radial list again
// afterwards (zbl_center).
// With L > 1 this lane (l of the L that share the center) visits entries l, l + L, ... and
// the sums over the lanes are formed at the end, in every lane.
template <class S, int PREC, bool MULTI, int L>
__device__ __forceinline__ void desc_pass(const ModelDev& m, const EvalBuffers& b, const PairTab<S, MULTI>& tab,
                                          int64_t i, int l, int ti, QPos qi, float* q, float* s, int& nz, int& nr,
                                          int& na) {
  constexpr int NR = S::NR, NA = S::NA, NC = S::NC, KR = S::KR, KA = S::KA, TT = MULTI ? kMaxTypes : 1;
  // the bfloat16 network with several species: a pair's g_n from its coefficients, added to q_n
  constexpr bool PAIRWISE = PREC == 1 && MULTI;
  const int64_t N = b.N;
  const float rcR_inv = 1.f / m.rcR, rcA_inv = 1.f / m.rcA;
  const CutConst cutR = cut_const(m.rcR), cutA = cut_const(m.rcA);
  const float rcR2 = (float)(m.rcR64 * m.rcR64), rcA2 = (float)(m.rcA64 * m.rcA64), zbl2 = (float)m.zbl_o2;
  const bool zbl_on = m.zbl_o2 > 0.0;
  const double hx = box_quantum(b.box[0]), hy = box_quantum(b.box[1]), hz = box_quantum(b.box[2]);
  nr = 0;
  na = 0;
  const int kR = radial_bound(b, i), kA = angular_bound(b, i);
  float Qf[TT], QT[TT][KR];  // sum_j f_c and sum_j f_c T_k
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    Qf[t] = 0.f;
#pragma unroll
    for (int k = 0; k < KR; ++k) QT[t][k] = 0.f;
  }
  // one entry: the radial term, and for the angular candidates inside rc_angular the angular one
  auto pair_both = [&](int p, int32_t j, const uint4* w) {
    float dx, dy, dz;
    const float r2 = pair_vec_q(w[0], qi, hx, hy, hz, dx, dy, dz);
    if (!(r2 < rcR2)) return;
    float r, rinv;
    r_of_r2(r2, r, rinv);
    const int tj = MULTI ? (int)w[0].w : 0;
    ++nr;
    nz += (zbl_on && r2 < zbl2) ? 1 : 0;
    if constexpr (PAIRWISE) {
      float g[NR];
      radial_g<NR, KR>(r, rcR_inv, tab.rad + (ti * kMaxTypes + tj) * (NR * KR), g);
#pragma unroll
      for (int n = 0; n < NR; ++n) q[n] += g[n];
    } else {
      // T_k by the recurrence T_{k+1} = 2x T_k - T_{k-1}
      const RadialGeo ra = radial_geo<false>(r, cutR);
      float ft[TT];  // f_c for the neighbour's species, 0 for the others
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        ft[t] = !MULTI || tj == t ? ra.fc : 0.f;
        Qf[t] += ft[t];
      }
      const float x2 = ra.x + ra.x;
      float Tm = 1.f, T = ra.x;
#pragma unroll
      for (int k = 1; k < KR; ++k) {
#pragma unroll
        for (int t = 0; t < TT; ++t) QT[t][k] = fmaf(ft[t], T, QT[t][k]);
        const float Tn = fmaf(x2, T, -Tm);
        Tm = T;
        T = Tn;
      }
    }
    if (p < kA && r2 < rcA2) {
      ++na;
      float g[NA];
      const RadialGeo ra = radial_geo<false>(r, cutA);
      if constexpr (PAIRWISE) {
        radial_g<NA, KA>(r, rcA_inv, ang_tab(tab, ti, tj), g);
      } else if constexpr (MULTI) {
        radial_cd_tab<S, false>(ra.x, ang_tab(tab, ti, tj), g, nullptr);
#pragma unroll
        for (int n = 0; n < NA; ++n) g[n] *= ra.fc;
      } else {
        radial_g_fast<NA, KA>(ra.fc, ra.x, uniform_coeffs(m.hA), g);
      }
      for_each_poly<NC>(dx * rinv, dy * rinv, dz * rinv, [&](int lm, float P) {
#pragma unroll
        for (int n = 0; n < NA; ++n) s[n * NC + lm] = fmaf(g[n], P, s[n * NC + lm]);
      });
    }
  };
  // the angular candidates are the list's prefix [0, kA)
  if constexpr (L > 1)
    for_each_rec_lanes<1, 1, L>(b.nbr, b.pos, N, i, l, kR, pair_both);
  else
    for_each_rec_fast<1, S::DESC_AHEAD, 1>(b.nbr, b.pos, N, i, 0, kR, pair_both);
  if constexpr (L > 1) {
    nr = lanes_sum<L>(nr);
    na = lanes_sum<L>(na);
    nz = lanes_sum<L>(nz);
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      Qf[t] = lanes_sum<L>(Qf[t]);
#pragma unroll
      for (int k = 1; k < KR; ++k) QT[t][k] = lanes_sum<L>(QT[t][k]);
    }
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) s[k] = lanes_sum<L>(s[k]);
  }
  if constexpr (PAIRWISE) return;
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    float Qb[KR];
    Qb[0] = Qf[t];
#pragma unroll
    for (int k = 1; k < KR; ++k) Qb[k] = 0.5f * (QT[t][k] + Qf[t]);
    auto add = [&](auto c) {
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < KR; ++k) a = fmaf(c[n * KR + k], Qb[k], a);
        q[n] += a;
      }
    };
    if constexpr (MULTI) add(tab.rad + (ti * kMaxTypes + t) * (NR * KR));
    else add(uniform_coeffs(m.cR));
  }
}

// dU/ds of one atom as a row (the deterministic form's layout): NA * NC values padded
// to a multiple of four, so that a row is read with 16-byte loads.
template <class S>
constexpr int g_row() {
  static_assert(((S::NA * S::NC + 3) & ~3) <= 5 * 24, "a row must fit the system's dU/ds buffer");
  return (S::NA * S::NC + 3) & ~3;
}
template <class S>
__device__ __forceinline__ void load_g_row(const float* row, float* g) {
  const float4* r4 = reinterpret_cast<const float4*>(row);
#pragma unroll
  for (int k = 0; k < g_row<S>() / 4; ++k) {
    const float4 v = r4[k];
    g[4 * k] = v.x;
    if (4 * k + 1 < S::NA * S::NC) g[4 * k + 1] = v.y;
    if (4 * k + 2 < S::NA * S::NC) g[4 * k + 2] = v.z;
    if (4 * k + 3 < S::NA * S::NC) g[4 * k + 3] = v.w;
  }
}

// The part of the descriptor kernel after the pair loop when L lanes share a center: q[0..NR)
// and s hold the center's sums in every lane. lds: this wavefront's operand tile.
template <class S, bool MULTI, int L>
__device__ __forceinline__ void finish_lanes(const ModelDev& m, const EvalBuffers& b, int64_t i, int l, bool valid,
                                             int ti, const float* q, const float* s, int nz, float* lds,
                                             const NetLds& net, const PairTab<S, MULTI>& tab) {
  constexpr int NR = S::NR, NA = S::NA, NC = S::NC, D = S::D, L3 = S::L3;
  constexpr int RT = 64 / L >= 16 ? 64 / L / 16 : 1;
  constexpr int ROUNDS = (NA + L - 1) / L;  // angular channels of a lane
  const int64_t N = b.N;
  float* row = lds + ((threadIdx.x & 63) / L) * kNetStride;
  // scaled descriptors into the row
#pragma unroll
  for (int n = 0; n < NR; ++n)
    if ((n & (L - 1)) == l) row[n] = q[n] * net.sigma[n];
  for (int v = D + l; v < 32; v += L) row[v] = 0.f;
  float sl[ROUNDS][NC];  // accumulators of channel n = l + r L
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    // picked by bit masks: a chain of selects becomes an indexed load of s, in scratch memory
#pragma unroll
    for (int lm = 0; lm < NC; ++lm) {
      uint32_t v = 0;
#pragma unroll
      for (int n = 0; n < NA; ++n)
        if (n / L == r) v |= __float_as_uint(s[n * NC + lm]) & (l == n % L ? 0xffffffffu : 0u);
      sl[r][lm] = __uint_as_float(v);
    }
    const int n = l + r * L;
    if (n < NA) {
      float ql[L3];
#pragma unroll
      for (int k = 0; k < L3; ++k) ql[k] = 0.f;
#pragma unroll
      for (int lm = 0; lm < NC; ++lm)
        ql[comp_l(lm) - 1] = fmaf(kW[lm], sl[r][lm] * sl[r][lm], ql[comp_l(lm) - 1]);
#pragma unroll
      for (int k = 0; k < L3; ++k) row[NR + k * NA + n] = ql[k] * net.sigma[NR + k * NA + n];
      if constexpr (S::FB) row[NR + L3 * NA + n] = fourbody_q(sl[r]) * net.sigma[NR + L3 * NA + n];
    }
  }
  net_product<RT, true>(lds, lds, net);
  float U = 0.f;
#pragma unroll
  for (int mu0 = 0; mu0 < 32; mu0 += L) {
    const int mu = mu0 + l;
    const float t = tanh_fast(row[mu] - net.b0[mu]), w = net.w1[mu];  // w1 = 0 beyond the last hidden unit
    U = fmaf(w, t, U);
    row[mu] = w * (1.f - t * t);
  }
  U = lanes_sum<L>(U) - m.b1[0];
  net_product<RT, false>(lds, lds, net);
  if (!valid) return;
  auto fp = [&](int v) { return row[v] * net.sigma[v]; };  // dU/dq_v
  // the 64-byte records: position (words 0..2), radial coefficients (3..11), species, zeros
#pragma unroll
  for (int t = 0; t < (MULTI ? kMaxTypes : 1); ++t) {
    static_assert(S::KR == 9 && NR <= 5, "the record holds nine radial coefficients");
    constexpr int TR = (9 + L - 1) / L;
    float w[TR], sum = 0.f;
#pragma unroll
    for (int r = 0; r < TR; ++r) {
      const int k = l + r * L;
      w[r] = 0.f;
      if (k < 9) {
#pragma unroll
        for (int n = 0; n < NR; ++n) {
          const float c = MULTI ? tab.rad[(ti * kMaxTypes + t) * (NR * S::KR) + n * S::KR + k] : m.cR[n * S::KR + k];
          w[r] = fmaf(fp(n), c, w[r]);
        }
      }
      sum += w[r];
    }
    sum = lanes_sum<L>(sum);
    if (l == 0) w[0] += sum;
    float* rec = reinterpret_cast<float*>((t == 0 ? b.rec : b.rec1) + 4 * i);
#pragma unroll
    for (int r = 0; r < TR; ++r)
      if (l + r * L < 9) rec[3 + l + r * L] = w[r];
    const uint32_t* own = reinterpret_cast<const uint32_t*>(b.pos + i);
    uint32_t* recu = reinterpret_cast<uint32_t*>(rec);
#pragma unroll
    for (int k0 = 0; k0 < 7; k0 += L) {  // words 0..2, 12 (species) and 13..15
      const int k = k0 + l;
      if (k < 4) recu[k < 3 ? k : 12] = own[k];
      else if (k < 7) recu[9 + k] = 0u;
    }
  }
  // dU/ds_nlm = dU/dq_nl * 2 W_lm s_nlm (+ four-body part for l = 2) of the lane's channels
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int n = l + r * L;
    if (n < NA) {
      float Gd[NC];
#pragma unroll
      for (int lm = 0; lm < NC; ++lm) Gd[lm] = fp(NR + (comp_l(lm) - 1) * NA + n) * 2.f * kW[lm] * sl[r][lm];
      if constexpr (S::FB) {
        float d5[5];
        fourbody_ds(sl[r], d5);
        const float f4 = fp(NR + L3 * NA + n);
#pragma unroll
        for (int k = 0; k < 5; ++k) Gd[3 + k] = fmaf(f4, d5[k], Gd[3 + k]);
      }
      if (b.deterministic) {
        static_assert(NC % 4 == 0, "a channel of a row is written in 16-byte words");
        float4* g4 = reinterpret_cast<float4*>(b.G + i * g_row<S>() + n * NC);
#pragma unroll
        for (int k = 0; k < NC / 4; ++k) g4[k] = make_float4(Gd[4 * k], Gd[4 * k + 1], Gd[4 * k + 2], Gd[4 * k + 3]);
      } else {
        float* g = b.G + (int64_t)n * NC * N + i;
#pragma unroll
        for (int lm = 0; lm < NC; ++lm) g[lm * N] = Gd[lm];
      }
    }
  }
  for (int c = l; c < 3; c += L) b.F[c * N + i] = 0.f;
  if (nz) {  // ZBL energy (half of each close pair)
    float uz = 0.f;
    zbl_center<MULTI>(m, b, i, ti, b.x[i], b.x[N + i], b.x[2 * N + i], &uz, nullptr, nullptr, l, L);
    U += lanes_sum<L>(uz);
  }
  if (l == 0) b.U[i] = U;
}

// ------------------------------------------------------------------------ descriptor + network
template <class S, int PREC, bool MULTI, int L>
__global__ void __launch_bounds__(kBlock, 2) k_desc_net(ModelDev m, EvalBuffers b) {
  __shared__ float lds[kBlock / 64][(64 / L >= 16 ? 64 / L : 16) * kNetStride];
  constexpr int NR = S::NR, NA = S::NA, NC = S::NC, D = S::D;
  const int64_t N = b.N;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t i = (int64_t)tile * (kBlock / L) + threadIdx.x / L;
  const int l = threadIdx.x % L;
  const bool valid = i < N;
  __shared__ PairTab<S, MULTI> tab;
  if constexpr (MULTI) {
    stage_pairs<S, PREC == 1>(m, tab);
    __syncthreads();
  }
  if constexpr (L > 1) {
    __shared__ NetLds net;
    stage_network<S>(m, net);
    float q[NR], s[NA * NC];
#pragma unroll
    for (int n = 0; n < NR; ++n) q[n] = 0.f;
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) s[k] = 0.f;
    const int ti = valid ? (MULTI ? b.type[i] : 0) : 0;
    int nz = 0;
    if (valid) {
      const uint4 w0 = b.pos[i];
      int nr = 0, na = 0;
      desc_pass<S, PREC, MULTI, L>(m, b, tab, i, l, ti, QPos{w0.x, w0.y, w0.z}, q, s, nz, nr, na);
      if (l == 0) {
        b.nactR[i] = nr;
        b.nactA[i] = na;
      }
    }
    __syncthreads();  // the staged weights
    finish_lanes<S, MULTI, L>(m, b, i, l, valid, ti, q, s, nz, lds[threadIdx.x >> 6], net, tab);
    return;
  }

  float q[D];
#pragma unroll
  for (int v = 0; v < D; ++v) q[v] = 0.f;
  float s[NA * NC];
#pragma unroll
  for (int k = 0; k < NA * NC; ++k) s[k] = 0.f;
  const int ti = valid ? (MULTI ? b.type[i] : 0) : 0;
  int nz = 0;  // pairs inside the ZBL radius

  if (valid) {
    const uint4 w0 = b.pos[i];
    int nr = 0, na = 0;
    desc_pass<S, PREC, MULTI, 1>(m, b, tab, i, 0, ti, QPos{w0.x, w0.y, w0.z}, q, s, nz, nr, na);
    b.nactR[i] = nr;
    b.nactA[i] = na;
    desc_finish<S>(s, q);
  }
  // 3. network (whole wavefronts take part; inactive lanes carry zeros)
  float qs[D], fp[D];
#pragma unroll
  for (int v = 0; v < D; ++v) qs[v] = q[v] * m.sigma[v];
  float U = network_wave<S, PREC>(m, qs, fp, lds[threadIdx.x >> 6], m.W0, m.b0, m.w1, m.b1[0]);
#pragma unroll
  for (int v = 0; v < D; ++v) fp[v] *= m.sigma[v];  // dU/dq = sigma * dU/dq~

  if (valid) {
    // the whole 64-byte record of each plane: position, v = w_0 + sum_k w_k and w_1..w_8 with
    // w_k = sum_n (dU/dq_n) c_nk (the radial force of a pair is then a Chebyshev series in
    // w_i + w_j), species
    const uint4 own = b.pos[i];
#pragma unroll
    for (int t = 0; t < (MULTI ? kMaxTypes : 1); ++t) {
      static_assert(S::KR == 9, "the record holds nine radial coefficients");
      float w[9], sum = 0.f;
      auto form = [&](auto c) {
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          float a = 0.f;
#pragma unroll
          for (int n = 0; n < NR; ++n) a = fmaf(fp[n], c[n * S::KR + k], a);
          w[k] = a;
          sum += a;
        }
      };
      if constexpr (MULTI) form(tab.rad + (ti * kMaxTypes + t) * (NR * S::KR));
      else form(uniform_coeffs(m.cR));
      w[0] += sum;
      uint4* r = (t == 0 ? b.rec : b.rec1) + 4 * i;
      r[0] = make_uint4(own.x, own.y, own.z, __float_as_uint(w[0]));
      reinterpret_cast<float4*>(r + 1)[0] = make_float4(w[1], w[2], w[3], w[4]);
      reinterpret_cast<float4*>(r + 2)[0] = make_float4(w[5], w[6], w[7], w[8]);
      r[3] = make_uint4(own.w, 0u, 0u, 0u);
    }
    // 4. dU/ds_nlm = dU/dq_nl * 2 W_lm s_nlm (+ four-body part for l = 2)
    float Gd[NA * NC];
#pragma unroll
    for (int n = 0; n < NA; ++n)
#pragma unroll
      for (int lm = 0; lm < NC; ++lm) {
        const int l = comp_l(lm);
        Gd[n * NC + lm] = fp[NR + (l - 1) * NA + n] * 2.f * kW[lm] * s[n * NC + lm];
      }
    if constexpr (S::FB) {
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        float d5[5];
        fourbody_ds(s + n * NC, d5);
        const float f4 = fp[NR + S::L3 * NA + n];
#pragma unroll
        for (int k = 0; k < 5; ++k) Gd[n * NC + 3 + k] = fmaf(f4, d5[k], Gd[n * NC + 3 + k]);
      }
    }
    if (b.deterministic) {
      // atom-major rows for the force kernel's gathers of the neighbours' dU/ds
      float4* g4 = reinterpret_cast<float4*>(b.G + i * g_row<S>());
#pragma unroll
      for (int k = 0; k < g_row<S>() / 4; ++k)
        g4[k] = make_float4(Gd[4 * k], 4 * k + 1 < NA * NC ? Gd[4 * k + 1] : 0.f,
                            4 * k + 2 < NA * NC ? Gd[4 * k + 2] : 0.f, 4 * k + 3 < NA * NC ? Gd[4 * k + 3] : 0.f);
    } else {
#pragma unroll
      for (int k = 0; k < NA * NC; ++k) b.G[(int64_t)k * N + i] = Gd[k];
    }
    b.F[i] = 0.f;
    b.F[N + i] = 0.f;
    b.F[2 * N + i] = 0.f;
    // ZBL energy (half of each close pair), after the descriptors are no longer live
    if (nz) zbl_center<MULTI>(m, b, i, ti, b.x[i], b.x[N + i], b.x[2 * N + i], &U, nullptr, nullptr);
    b.U[i] = U;
  }
}

// ------------------------------------------------------------------------ force halo in LDS
// The angular force kernel scatters -dU_i/dr_ij into every neighbour j. A workgroup's
// 256 cell-sorted atoms only reach atoms of the cells next to theirs (the tile's halo,
// tabulated at list build), so the scatter goes into an LDS copy of the halo's forces
// and one coalesced global atomic per halo atom and component flushes it at the end
// (scattered global atomics resolve at the memory side one cache line each).
struct HaloLds {
  alignas(16) float F[3][kHaloMax];
  int start[kHaloCellsMax];
  int off[kHaloCellsMax + 1];
};

// Loads the tile's halo table of nc cells and clears the LDS forces of its na atoms (as
// 16-byte words: the rows of F are padded to whole ones). A barrier must follow.
__device__ __forceinline__ void load_halo(const EvalBuffers& b, int tile, int nc, int na, HaloLds& h) {
  for (int k = threadIdx.x; k < nc; k += kBlock) h.start[k] = b.hstart[(int64_t)tile * kHaloCellsMax + k];
  for (int k = threadIdx.x; k <= nc; k += kBlock) h.off[k] = b.hoff[(int64_t)tile * (kHaloCellsMax + 1) + k];
  static_assert(kHaloMax % 4 == 0, "whole words");
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int t = threadIdx.x; 4 * t < na; t += kBlock) {
    reinterpret_cast<float4*>(h.F[0])[t] = zero;
    reinterpret_cast<float4*>(h.F[1])[t] = zero;
    reinterpret_cast<float4*>(h.F[2])[t] = zero;
  }
}

// Adds the halo forces to F with one global atomic per halo atom and component that
// received a force: 16 lanes to a halo cell, whose atoms are contiguous both in the halo
// and in F.
__device__ void flush_halo(const HaloLds& h, int nc, float* __restrict__ F, int64_t N) {
  const int q = threadIdx.x >> 4, u = threadIdx.x & 15;
  for (int c = q; c < nc; c += kBlock / 16) {
    const int o = h.off[c], n = h.off[c + 1] - o;
    const int64_t g0 = h.start[c];
    for (int t = u; t < n; t += 16) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float v = h.F[k][o + t];
        if (v != 0.f) unsafeAtomicAdd(&F[k * N + g0 + t], v);
      }
    }
  }
}

// ------------------------------------------------------------------------ forces
// Waves per SIMD the force kernel is compiled for: the l <= 2 shapes fit three in
// registers and in LDS (the halo takes a third of a CU's LDS); four would spill.
template <class S>
constexpr int force_waves() { return S::L3 <= 2 ? 3 : 2; }

// Constants of the angular pair force (uniform over a launch).
struct AngConst {
  CutConst cutA;
  float kDA;  // f_c' = kDA c (angular cutoff)
  float kYA;  // x' = kYA y
};
__device__ __forceinline__ AngConst ang_const(const ModelDev& m) {
  AngConst a;
  a.cutA = cut_const(m.rcA);
  a.kDA = -0.5f * kPiF * a.cutA.rc_inv;
  a.kYA = 4.f * a.cutA.rc_inv;
  return a;
}

// Angular and four-body force of center c on a neighbour k inside rc_angular, n = -dU_c/dr_ck,
// for the unit vector u from c to k at distance r, from the center's dU/ds (Gc(q) returns
// component q < NA * NC, channel-major) and the pair's types (center tc, neighbour tk):
// F_ck = sum_lm [ A_lm P_lm u + B_lm (grad P_lm - l P_lm u) / r ] with A_lm = sum_n G_nlm g'_n
// and B_lm = sum_n G_nlm g_n; the l P B terms are summed per l and scaled once.
template <class S, bool MULTI, class GF>
__device__ __forceinline__ void angular_pair_force(const ModelDev& m, const AngConst& ac, const PairTab<S, MULTI>& tab,
                                                   GF&& Gc, int tc, int tk, float ux, float uy, float uz, float r,
                                                   float rinv, float& n0, float& n1, float& n2) {
  constexpr int NA = S::NA, NC = S::NC, KA = S::KA;
  float vx = 0.f, vy = 0.f, vz = 0.f;
  // With g_n = f_c C_n and g'_n = f_c' C_n + f_c x' D_n: B_lm = f_c E_lm and
  // A_lm = f_c' E_lm + f_c x' H_lm for E_lm = sum_n G_nlm C_n, H_lm = sum_n G_nlm D_n,
  // so f_c, f_c' and f_c x' are applied once to the sums over lm.
  const RadialGeo rb = radial_geo<true>(r, ac.cutA);
  float Cn[NA], Dn[NA];
  if constexpr (MULTI)
    radial_cd_tab<S, true>(rb.x, ang_tab(tab, tc, tk), Cn, Dn);
  else
    radial_cd_fast<NA, KA>(rb.x, uniform_coeffs(m.hA), Cn, Dn);
  float sH = 0.f;
  float sE[4] = {0.f, 0.f, 0.f, 0.f};
  for_each_poly_grad<NC>(ux, uy, uz, [&](int lm, float P, auto px, auto py, auto pz) {
    float E = Gc(lm) * Cn[0], H = Gc(lm) * Dn[0];
#pragma unroll
    for (int n = 1; n < NA; ++n) {
      E = fmaf(Gc(n * NC + lm), Cn[n], E);
      H = fmaf(Gc(n * NC + lm), Dn[n], H);
    }
    sH = fmaf(P, H, sH);
    sE[comp_l(lm) - 1] = fmaf(P, E, sE[comp_l(lm) - 1]);
    vx = fmac(E, px, vx);
    vy = fmac(E, py, vy);
    vz = fmac(E, pz, vz);
  });
  const float sPE = (sE[0] + sE[1]) + (sE[2] + sE[3]);
  const float lPE = fmaf(4.f, sE[3], fmaf(3.f, sE[2], fmaf(2.f, sE[1], sE[0])));
  const float sA = fmaf(ac.kDA * rb.c, sPE, (rb.fc * (ac.kYA * rb.y)) * sH);
  const float vscale = rb.fc * rinv;
  const float sc = fmaf(-vscale, lPE, sA);
  // n = -dU_c/dr_ck (sign folded into the operands)
  n0 = fmaf(-ux, sc, -(vx * vscale));
  n1 = fmaf(-uy, sc, -(vy * vscale));
  n2 = fmaf(-uz, sc, -(vz * vscale));
}

// Whether the ZBL forces are added after all others, by a launch of their own. Every atomic
// addition to an atom's force rounds to the force's size, and a ZBL force may be many
// times the others'; with L > 4 some twenty workgroups add to each atom. Error of the forces
// against FP64 (norm, relative) for FCC boxes of 4,000 atoms with neighbours inside the ZBL
// radius: one thread per center 6.9e-8, 4 lanes 6.5e-8, 16 lanes 7.8e-8 and with this launch
// 3.5e-8 (9.5e-8 with the ZBL force of each lane summed in FP32). It costs 2 to 4 us; four
// lanes in place of sixteen would cost 16 to 22 of the 150 us of such a box's evaluation.
template <bool DET, int L>
constexpr bool late_zbl() { return !DET && L > 4; }
__global__ void k_add_late(int64_t n, const double* __restrict__ late, float* __restrict__ F) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) F[k] = (float)((double)F[k] + late[k]);
}

// DET: the deterministic form. Nothing is scattered: each atom adds, after its own pair
// terms, the angular forces of the centers that have it as an angular neighbour, each
// recomputed from that center's dU/ds (atom-major rows), and stores its force. With L lanes
// each takes every L-th list entry and the lanes' sums are added in a fixed order, so the
// order follows the list and the lane count, that is the system's size and the model's
// shape. The sets agree: a pair inside rc_angular lies in both atoms' angular prefixes, and
// the box-fraction pair vector of (j, i) is the exact negation of that of (i, j), so both
// sides see the same r^2. The terms are bitwise those the scattering form adds, in a fixed
// order.
template <class S, bool MULTI, bool DET, int L>
__global__ void __launch_bounds__(kBlock, force_waves<S>()) k_force(ModelDev m, EvalBuffers b) {
  __shared__ double red[4 * 10];
  __shared__ HaloLds halo;
  __shared__ PairTab<S, MULTI> tab;
  // two species, full shape: the thread's own coefficients towards each species in LDS, 18
  // registers that its pair loop does not have (864,000 atoms: 1,429 us with them spilled,
  // 1,327 in LDS); the l <= 2 shapes have them, and their third workgroup needs the LDS
  constexpr bool OWN = MULTI && S::L3 > 2;
  __shared__ float own[OWN ? kMaxTypes : 1][OWN ? S::KR : 1][OWN ? kBlock : 1];
  constexpr int NA = S::NA, NC = S::NC;
  const int64_t N = b.N;
  const int sub = xcd_tile(blockIdx.x, gridDim.x);  // L workgroups to a 256-atom tile
  const int64_t i = (int64_t)sub * (kBlock / L) + threadIdx.x / L;
  const int l = threadIdx.x % L;
  const bool valid = i < N;
  // the center's own loads first (clamped for the lanes past the system), so that they are
  // in flight with the halo's
  const int64_t ic = valid ? i : N - 1;
  const int kR = radial_bound(b, ic), kA = angular_bound(b, ic);
  const uint4* ri = b.rec + 4 * ic;
  const uint4 r0 = ri[0], r1 = ri[1], r2w = ri[2];
  const int ti = MULTI ? (int)ri[3].x : 0;
  constexpr int KR = S::KR;
  float G[NA * NC];
  if constexpr (DET) {
    load_g_row<S>(b.G + ic * g_row<S>(), G);
  } else {
#pragma unroll
    for (int k = 0; k < NA * NC; ++k) G[k] = b.G[(int64_t)k * N + ic];
  }
  const int tile = sub / L;
  const int hcells = DET ? 0 : b.hinfo[4 * tile], hatoms = DET ? 0 : b.hinfo[4 * tile + 1];
  const bool lds = !DET && b.hinfo[4 * tile + 2] != 0;
  if constexpr (MULTI) stage_pairs<S>(m, tab);
  if (lds) load_halo(b, tile, hcells, hatoms, halo);
  if (MULTI || lds) __syncthreads();
  const double hx = box_quantum(b.box[0]), hy = box_quantum(b.box[1]), hz = box_quantum(b.box[2]);
  const CutConst cutR = cut_const(m.rcR);
  const float kXR = -0.25f * kPiF * cutR.rc_inv;  // X = kXR Z for the radial series
  const AngConst ac = ang_const(m);
  const bool zbl_on = m.zbl_o2 > 0.0;
  float fx = 0.f, fy = 0.f, fz = 0.f;
  float w[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) w[k] = 0.f;
  if (valid) {
    const QPos qi{r0.x, r0.y, r0.z};
    const uint4* plane = MULTI && ti ? b.rec1 : b.rec;  // the neighbours' coefficients towards this species
    // own radial coefficients (v = w_0 + sum_k w_k and w_1..w_8) towards each species
    const float wi[9] = {__uint_as_float(r0.w),  __uint_as_float(r1.x),  __uint_as_float(r1.y),
                         __uint_as_float(r1.z),  __uint_as_float(r1.w),  __uint_as_float(r2w.x),
                         __uint_as_float(r2w.y), __uint_as_float(r2w.z), __uint_as_float(r2w.w)};
    float wi1[9];
    if constexpr (MULTI) {
      const float* rf = reinterpret_cast<const float*>(b.rec1 + 4 * i) + 3;
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        if constexpr (OWN) {
          own[0][k][threadIdx.x] = wi[k];
          own[1][k][threadIdx.x] = rf[k];
        } else {
          wi1[k] = rf[k];
        }
      }
    }
    const float rcR2 = (float)(m.rcR64 * m.rcR64), rcA2 = (float)(m.rcA64 * m.rcA64), zbl2 = (float)m.zbl_o2;
    int nz = 0;  // pairs inside the ZBL radius
    // One entry: the radial term by gather, F_i += (dU_i/dr_ij + dU_j/dr_ji) along u, with
    // the neighbour's radial coefficients read from its record, the virial taking half of
    // that pair term (the lists are symmetric, so the pair's other half comes from j); and
    // for the angular candidates (the list prefix [0, kA)) inside rc_angular the angular
    // and four-body term dU_i/dr_ij, added to this atom and scattered, negated, into the
    // neighbour.
    auto pair_both = [&](int p, int32_t j, const uint4* rw) {
      float dx, dy, dz;
      const float r2 = pair_vec_q(rw[0], qi, hx, hy, hz, dx, dy, dz);
      if (!(r2 < rcR2)) return;
      const bool ang = p < kA && r2 < rcA2;
      const int lj = (!DET && ang && lds) ? (int)b.nbrl[(int64_t)p * N + i] : 0;
      float r, rinv;
      r_of_r2(r2, r, rinv);
      const int tj = MULTI ? (int)rw[3].x : 0;
      const float wj[9] = {__uint_as_float(rw[0].w), __uint_as_float(rw[1].x), __uint_as_float(rw[1].y),
                           __uint_as_float(rw[1].z), __uint_as_float(rw[1].w), __uint_as_float(rw[2].x),
                           __uint_as_float(rw[2].y), __uint_as_float(rw[2].z), __uint_as_float(rw[2].w)};
      // (dU_i/dr_ij + dU_j/dr_ji) / r, the radial parts: sum_k (w_ik + w_jk) f_k'(r) / r; the
      // pair force is sr (x_j - x_i)
      const RadialGeo ra = radial_geo<true>(r, cutR);
      float W[KR];
#pragma unroll
      for (int k = 0; k < KR; ++k) {
        if constexpr (OWN) W[k] = own[tj][k][threadIdx.x] + wj[k];
        else W[k] = (MULTI && tj ? wi1[k] : wi[k]) + wj[k];
      }
      const float sr = radial_series_z<KR>(ra, W, W[0]) * (kXR * rinv);
      nz += (zbl_on && r2 < zbl2) ? 1 : 0;
      fx = fmaf(sr, dx, fx);
      fy = fmaf(sr, dy, fy);
      fz = fmaf(sr, dz, fz);
      {
        // W_ac -= d_a (sr d_c) / 2
        const float vs = -0.5f * sr;
        const float d[3] = {dx, dy, dz};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const float vd = vs * d[a];
#pragma unroll
          for (int c = 0; c < 3; ++c) w[a * 3 + c] = fmaf(vd, d[c], w[a * 3 + c]);
        }
      }
      if (!ang) return;
      const float ux = dx * rinv, uy = dy * rinv, uz = dz * rinv;
      float n0, n1, n2;  // -dU_i/dr_ij, the force on the neighbour
      angular_pair_force<S, MULTI>(m, ac, tab, [&](int q) { return G[q]; }, ti, tj, ux, uy, uz, r, rinv, n0, n1, n2);
      fx -= n0;
      fy -= n1;
      fz -= n2;
      if constexpr (!DET) {
        if (lds) {
          atomicAdd(&halo.F[0][lj], n0);
          atomicAdd(&halo.F[1][lj], n1);
          atomicAdd(&halo.F[2][lj], n2);
        } else {
          unsafeAtomicAdd(&b.F[j], n0);
          unsafeAtomicAdd(&b.F[N + j], n1);
          unsafeAtomicAdd(&b.F[2 * N + j], n2);
        }
      }
      const float d[3] = {dx, dy, dz};
      const float nf[3] = {n0, n1, n2};
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) w[a * 3 + c] = fmaf(d[a], nf[c], w[a * 3 + c]);
    };
    constexpr int W = MULTI ? 4 : 3;  // words of a record: with several species also the species
    if constexpr (L > 1)
      for_each_rec_lanes<W, 4, L>(b.nbr, plane, N, i, l, kR, pair_both);
    else
      for_each_rec_fast<W, 1, 4>(b.nbr, plane, N, i, 0, kR, pair_both);
    nz = lanes_sum<L>(nz);
    if constexpr (DET) {
      // the neighbours' angular terms on this atom, the lane's entries in list order
      const uint64_t n64 = (uint64_t)N;
      for (int p = l; p < kA; p += L) {
        const int32_t j = b.nbr[(uint64_t)(uint32_t)p * n64 + i];
        float dx, dy, dz;
        const uint4 pj = b.pos[j];
        const float r2 = pair_vec_q(pj, qi, hx, hy, hz, dx, dy, dz);
        if (!(r2 < rcR2 && r2 < rcA2)) continue;
        float r, rinv;
        r_of_r2(r2, r, rinv);
        const int tj = MULTI ? (int)pj.w : 0;
        float Gj[NA * NC];
        load_g_row<S>(b.G + (int64_t)j * g_row<S>(), Gj);
        float n0, n1, n2;  // -dU_j/dr_ji, the force of center j's angular term on this atom
        angular_pair_force<S, MULTI>(m, ac, tab, [&](int q) { return Gj[q]; }, tj, ti, -(dx * rinv), -(dy * rinv),
                                     -(dz * rinv), r, rinv, n0, n1, n2);
        fx += n0;
        fy += n1;
        fz += n2;
      }
    }
    // the center's own force: the sum over its lanes, stored by the first
    fx = lanes_sum<L>(fx);
    fy = lanes_sum<L>(fy);
    fz = lanes_sum<L>(fz);
    // the ZBL force, rounded once with the sum of the others or left to k_add_late
    double f[3] = {0.0, 0.0, 0.0};
    if (nz) {
      zbl_center<MULTI>(m, b, i, ti, b.x[i], b.x[N + i], b.x[2 * N + i], nullptr, f, w, l, L);
#pragma unroll
      for (int c = 0; c < 3; ++c) f[c] = lanes_sum<L>(f[c]);
    }
    if (late_zbl<DET, L>() && zbl_on) {
      if (l == 0)
#pragma unroll
        for (int c = 0; c < 3; ++c) b.late[c * N + i] = f[c];
    } else if (nz) {
      fx = (float)((double)fx + f[0]);
      fy = (float)((double)fy + f[1]);
      fz = (float)((double)fz + f[2]);
    }
    if (l == 0) {
      if constexpr (DET) {
        b.F[i] = fx;
        b.F[N + i] = fy;
        b.F[2 * N + i] = fz;
      } else if (lds) {
        const int li = b.selfl[i];
        atomicAdd(&halo.F[0][li], fx);
        atomicAdd(&halo.F[1][li], fy);
        atomicAdd(&halo.F[2][li], fz);
      } else {
        unsafeAtomicAdd(&b.F[i], fx);
        unsafeAtomicAdd(&b.F[N + i], fy);
        unsafeAtomicAdd(&b.F[2 * N + i], fz);
      }
    }
  }
  if constexpr (!DET) {
    if (lds) {
      __syncthreads();
      flush_halo(halo, hcells, b.F, N);
    }
  }
  // the tile's energy (the descriptor kernel's U_i, ZBL included) and virial in FP64
  double wd[10], ws[10];
  wd[0] = valid && l == 0 ? (double)b.U[i] : 0.0;
#pragma unroll
  for (int k = 0; k < 9; ++k) wd[1 + k] = (double)w[k];
  block_sum_n<10>(wd, ws, red);
  if (threadIdx.x == 0) {
    b.ew[(int64_t)sub * kPartialStride + P_ENERGY] = ws[0];
#pragma unroll
    for (int k = 0; k < 9; ++k) b.ew[(int64_t)sub * kPartialStride + P_VIR + k] = ws[1 + k];
  }
}

template <class S, int PREC, bool MULTI, int L>
void launch_desc(const ModelDev& m, const EvalBuffers& b, hipStream_t st) {
  hipLaunchKernelGGL((k_desc_net<S, PREC, MULTI, L>), dim3(grid_blocks(b.N, kBlock / L)), dim3(kBlock), 0, st, m, b);
}
template <class S, bool MULTI, int L>
void launch_force(const ModelDev& m, const EvalBuffers& b, hipStream_t st) {
  const dim3 nb(grid_blocks(b.N, kBlock / L));
  if (b.deterministic) {
    hipLaunchKernelGGL((k_force<S, MULTI, true, L>), nb, dim3(kBlock), 0, st, m, b);
    return;
  }
  hipLaunchKernelGGL((k_force<S, MULTI, false, L>), nb, dim3(kBlock), 0, st, m, b);
  if (late_zbl<false, L>() && m.zbl_o2 > 0)
    hipLaunchKernelGGL(k_add_late, dim3(grid_blocks(3 * b.N)), dim3(kBlock), 0, st, 3 * b.N, b.late, b.F);
}

// One thread per center fills the chip (1,024 SIMDs, two wavefronts each) from about 131,072
// atoms on; below, a wavefront's own latency is the kernel's time (k_force 102 us from 256
// to 32,000 atoms), so L lanes share a center, as many as keep N L <= 131072. On both sides
// of that line, us of k_desc_net + k_force, one species:
//   N         L = 1    2    4    8   16
//   256         140   89   56   39   32
//   4,000       150   92   59   44   38
//   13,500      160   97   62   58   78
//   32,000      154  104   84  107  146
//   62,500      166  134  150  192  263
//   108,000     217  242  251  307  432
// More lanes cost per wavefront (the sums over lanes, a halo to clear and flush per 256 / L
// centers), fewer leave SIMDs idle.
// The bfloat16 network keeps one lane and its own pair sums (desc_pass): it rounds the
// descriptors to eight bits, so that a sum in another order moves about one in a thousand of
// them by a whole step (outputs then differ by 1e-4 of their norm, with the same error).
constexpr int64_t kFillLanes = 131072;
constexpr int kMaxLanes = 16;
int desc_lanes(int64_t N) {
  int L = kMaxLanes;
  while (L > 1 && N * L > kFillLanes) L /= 2;
  return L;
}
// The force kernel of the full shape also takes four lanes where that makes two or three
// short rounds of workgroups in place of one that leaves a quarter to a half of the chip
// idle: up to 3/4 of 65,536 and of 131,072 atoms. us, one species / two / two deterministic:
//   N         L = 1         2              4
//   46,000      111 133 220   90 105 166    87 109 134
//   62,500      115 135 220   92 106 169   100 115 161
//   80,000      155 192 341  146 198 250   146 166 205
//   120,000     154 192 354  167 197 312   185 215 298
// Two species share the LDS pipe between tables and force sums, so that two lanes cost as much
// per center as one, and the deterministic form gains at every size. They are taken where a
// round of 65,536 centers in place of one of 131,072 ends the launch earlier, and from five
// such rounds on; with one species only just above 131,072 centers. l <= 2: with two species,
// within its first round of 196,608 centers. us, default / deterministic:
//   N, full            L = 1       2        N, l <= 2, default    L = 1    2
//   one      135,036   226 512   209 394    two        95,760     55    45
//            186,624   223 539   225 461               149,355    76    71
//   two      177,293   360 522   283 439               243,200   104   103
//            243,200   369  -    376  -     one        100,800    45    58
//            411,316   744 1197  659 982
//            820,800  1292 2290 1230 1959
// Both modes take the same lanes, since the virial's partial sums follow them.
int force_lanes(const ModelDev& m, int64_t N) {
  const int64_t half = (N + 65535) / 65536;  // rounds of 65,536 centers
  if (m.L3 <= 2) return m.T > 1 && N > 65536 && N <= 196608 ? 2 : desc_lanes(N);
  if ((N > 32768 && N <= 49152) || (N > 65536 && N <= 98304)) return 4;
  if (N > 131072 && (m.T > 1 ? half % 2 == 1 || half > 4 : N <= 163840)) return 2;
  return desc_lanes(N);
}

// ev (nullable): three events recorded before the descriptor kernel, between the two
// kernels and after the force kernel.
template <class S, int PREC, bool MULTI>
hipError_t launch_pair(const ModelDev& m, const EvalBuffers& b, hipStream_t st, hipEvent_t* ev) {
  if (ev) (void)hipEventRecord(ev[0], st);
  if constexpr (PREC == 1) {
    launch_desc<S, 1, MULTI, 1>(m, b, st);
  } else {
    switch (desc_lanes(b.N)) {
      case 16: launch_desc<S, 0, MULTI, 16>(m, b, st); break;
      case 8: launch_desc<S, 0, MULTI, 8>(m, b, st); break;
      case 4: launch_desc<S, 0, MULTI, 4>(m, b, st); break;
      case 2: launch_desc<S, 0, MULTI, 2>(m, b, st); break;
      default: launch_desc<S, 0, MULTI, 1>(m, b, st); break;
    }
  }
  if (ev) (void)hipEventRecord(ev[1], st);
  switch (force_lanes(m, b.N)) {
    case 16: launch_force<S, MULTI, 16>(m, b, st); break;
    case 8: launch_force<S, MULTI, 8>(m, b, st); break;
    case 4: launch_force<S, MULTI, 4>(m, b, st); break;
    case 2: launch_force<S, MULTI, 2>(m, b, st); break;
    default: launch_force<S, MULTI, 1>(m, b, st); break;
  }
  if (ev) (void)hipEventRecord(ev[2], st);
  return hipGetLastError();
}

template <class S>
hipError_t launch_shape(const ModelDev& m, int precision, const EvalBuffers& b, hipStream_t st,
                        hipEvent_t* ev) {
  const bool multi = m.T > 1;
  if (precision == 0)
    return multi ? launch_pair<S, 0, true>(m, b, st, ev) : launch_pair<S, 0, false>(m, b, st, ev);
  return multi ? launch_pair<S, 1, true>(m, b, st, ev) : launch_pair<S, 1, false>(m, b, st, ev);
}


// Derived radial tables (nep_fast.h) of coefficient blocks [nblk][N][K]: one thread per
// (block, channel) writes h_n0 = (c_n0 + sum_k c_nk) / 2, h_nk = c_nk / 2 and
// d_n(k-1) = k c_nk / 2 into that block's [N][2K - 1] table. Workgroup 0 derives the radial
// blocks, workgroup 1 the angular ones.
struct DeriveArgs {
  const float* c;
  float* h;
  int N, K;
};
__global__ void k_derive_coeffs(DeriveArgs r, DeriveArgs a, int nblk) {
  const DeriveArgs d = blockIdx.x == 0 ? r : a;
  const int N = d.N, K = d.K;
  for (int t = threadIdx.x; t < nblk * N; t += blockDim.x) {
    const int blk = t / N, n = t % N;
    const float* cn = d.c + ((int64_t)blk * N + n) * K;
    float* hb = d.h + (int64_t)blk * N * (2 * K - 1);
    float sum = 0.f;
    for (int k = 0; k < K; ++k) sum += cn[k];
    hb[n * K] = 0.5f * (cn[0] + sum);
    for (int k = 1; k < K; ++k) {
      hb[n * K + k] = 0.5f * cn[k];
      hb[N * K + n * (K - 1) + k - 1] = (0.5f * (float)k) * cn[k];
    }
  }
}

}  // namespace

int64_t derived_coeff_floats(int T, int nR, int kR, int nA, int kA) {
  return (int64_t)T * T * (nR * (2 * kR - 1) + nA * (2 * kA - 1));
}

hipError_t launch_derive_coeffs(int T, int nR, int kR, int nA, int kA, const float* cR, const float* cA, float* hR,
                                float* hA, hipStream_t st) {
  hipLaunchKernelGGL(k_derive_coeffs, dim3(2), dim3(64), 0, st, DeriveArgs{cR, hR, nR, kR}, DeriveArgs{cA, hA, nA, kA},
                     T * T);
  return hipGetLastError();
}

bool eval_supported(const ModelDev& m) { return is_shape<FullShape>(m) || is_shape<SurShape>(m); }

int eval_rows(const ModelDev& m, int64_t N) { return grid_blocks(N, kBlock / force_lanes(m, N)); }

hipError_t launch_eval(const ModelDev& m, int precision, const EvalBuffers& b, hipStream_t st,
                       hipEvent_t* ev) {
  if (is_shape<FullShape>(m)) return launch_shape<FullShape>(m, precision, b, st, ev);
  if (is_shape<SurShape>(m)) return launch_shape<SurShape>(m, precision, b, st, ev);
  return hipErrorInvalidValue;
}

}  // namespace nep
