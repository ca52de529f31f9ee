// Velocity-Verlet integration in FP64, the rebuild trigger, FP64 reductions and
// the conversions between the caller's original atom order ([N][3] rows) and
// the cell-sorted structure-of-arrays layout ([3][N]) used on the device.
// Section VI.A: 1 fs steps, neighbour lists refreshed every 10 steps with the
// displacement check enabled.
#include "nep_common.h"

namespace nep {
namespace {

// Sums of slots first .. first + nvals - 1 over the rows of partials, one workgroup of
// kRedBlock threads: 64 rows of 16 slots per pass (whole 128-byte rows, every slot at once),
// then the 64 row groups of each slot in a fixed order. sh holds kRedBlock doubles.
constexpr int kRedBlock = 1024;

__device__ __forceinline__ void reduce_rows(const double* __restrict__ partial, int nblocks, int first, int nvals,
                                            double* __restrict__ out, double* sh) {
  constexpr int kRows = kRedBlock / kPartialStride;
  const int slot = threadIdx.x % kPartialStride, row = threadIdx.x / kPartialStride;
  double s = 0.0;
#pragma unroll 4
  for (int b = row; b < nblocks; b += kRows) s += partial[(int64_t)b * kPartialStride + slot];
  sh[threadIdx.x] = s;
  __syncthreads();
  const int k = threadIdx.x - first;
  if (k >= 0 && k < nvals) {
    double t = 0.0;
#pragma unroll 8
    for (int r = 0; r < kRows; ++r) t += sh[r * kPartialStride + threadIdx.x];
    out[k] = t;
  }
}

__global__ void __launch_bounds__(kRedBlock)
k_reduce_partials(const double* __restrict__ partial, int nblocks, int first, int nvals, double* __restrict__ out) {
  __shared__ double sh[kRedBlock];
  reduce_rows(partial, nblocks, first, nvals, out, sh);
}

// An evaluation's results in one launch: the first workgroup sums the energy and virial
// partials, the others write forces [3 o + c] and (or) per-atom energies [o] in the
// caller's order as FP64. R: the type the evaluation holds them in. gate: the flag words, where
// the state and the lists are not checked on the host yet; an error there leaves the caller's
// arrays as they are.
template <class R>
__global__ void __launch_bounds__(kRedBlock)
k_results(const double* __restrict__ ew, int ew_rows, double* __restrict__ out, int64_t N,
          const int32_t* __restrict__ perm, const R* __restrict__ F, const R* __restrict__ U,
          double* __restrict__ forces, double* __restrict__ energies, const int32_t* __restrict__ gate) {
  __shared__ double sh[kRedBlock];
  if (blockIdx.x == 0) return reduce_rows(ew, ew_rows, P_ENERGY, 10, out, sh);
  const int64_t p = (int64_t)(blockIdx.x - 1) * kRedBlock + threadIdx.x;
  if (p >= N) return;
  if (gate && (gate[FLAG_OVF_R] | gate[FLAG_OVF_A] | gate[FLAG_TYPE] | gate[FLAG_NONFINITE])) return;
  const int64_t o = perm[p];
  if (forces)
    for (int c = 0; c < 3; ++c) forces[3 * o + c] = (double)F[c * N + p];
  if (energies) energies[o] = (double)U[p];
}

// The same for the training forward: FP32 forces in the caller's order.
__global__ void __launch_bounds__(kRedBlock)
k_results_f32(const double* __restrict__ ew, int ew_rows, double* __restrict__ out, int64_t N,
              const int32_t* __restrict__ perm, const float* __restrict__ F, float* __restrict__ forces) {
  __shared__ double sh[kRedBlock];
  if (blockIdx.x == 0) return reduce_rows(ew, ew_rows, P_ENERGY, 10, out, sh);
  const int64_t p = (int64_t)(blockIdx.x - 1) * kRedBlock + threadIdx.x;
  if (p >= N) return;
  const int64_t o = perm[p];
  for (int c = 0; c < 3; ++c) forces[3 * o + c] = F[c * N + p];
}

__device__ __forceinline__ double wrap_coord(double xv, double L) {
  if (xv < 0.0) xv += L;
  else if (xv >= L) xv -= L;
  return xv;
}

// v += dt/2 F/(m xi); x += dt v; wrap; the largest squared displacement since the build per
// workgroup, for the rebuild decision. PENDING: the half kick that ends the step before comes
// first (the same forces: one pass over v and F and one launch for both); NHC: before the
// kicks v is scaled by the chain's trailing and leading factors. Strides over a capped grid (kIntegrateGrid
// workgroups), so that these maxima are few.
constexpr int kIntegrateGrid = 8192;

template <bool PENDING, bool NHC>
__global__ void k_kick_drift(int64_t N, double dt, CellGrid g, const float* __restrict__ F,
                             const int32_t* __restrict__ type, MassTable mt, double* __restrict__ x,
                             double* __restrict__ v, uint4* __restrict__ pos, const double* __restrict__ xb,
                             const double* __restrict__ nhc, double* __restrict__ d2_out) {
  __shared__ double sh[kBlock / 64];
  double d2max = 0.0;
  const double s0 = NHC ? nhc[kNhcTrail] : 1.0, s1 = NHC ? nhc[kNhcLead] : 1.0;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += (int64_t)gridDim.x * blockDim.x) {
    const int32_t tp = type[p];
    const double inv = mt.inv_mxi[tp];
    double xn[3];
    double d2 = 0.0;
    for (int c = 0; c < 3; ++c) {
      const double a = (double)F[c * N + p];
      double vv = v[c * N + p];
      if (NHC) vv = vv * s0 * s1;
      if (PENDING) vv = vv + 0.5 * dt * a * inv;
      vv = vv + 0.5 * dt * a * inv;
      const double xx = wrap_coord(x[c * N + p] + dt * vv, g.box[c]);
      v[c * N + p] = vv;
      x[c * N + p] = xx;
      xn[c] = xx;
      const double d = min_image(xx - xb[c * N + p], g.box[c]);
      d2 += d * d;
    }
    pos_put(pos, p, xn[0], xn[1], xn[2], tp, g.box);
    if (!(d2 == d2)) d2 = 1e300;
    d2max = fmax(d2max, d2);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) d2max = fmax(d2max, __shfl_xor(d2max, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = d2max;
  __syncthreads();
  if (threadIdx.x == 0) d2_out[blockIdx.x] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

// v += dt (Fa - Fb)/(m xi)
__global__ void k_kick_diff(int64_t N, double dt, const float* __restrict__ Fa, const float* __restrict__ Fb,
                            const int32_t* __restrict__ type, MassTable mt, double* __restrict__ v) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  const double inv = mt.inv_mxi[type[p]];
  for (int c = 0; c < 3; ++c)
    v[c * N + p] += dt * ((double)Fa[c * N + p] - (double)Fb[c * N + p]) * inv;
}

__device__ __forceinline__ void block_partial(double val, double* sh, double* out) {
  __syncthreads();
  sh[threadIdx.x] = val;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < (unsigned)off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

template <bool KE>
__global__ void k_kick(int64_t N, double dt, const float* __restrict__ F, const int32_t* __restrict__ type,
                       MassTable mt, double* __restrict__ v, double* __restrict__ partial) {
  __shared__ double sh[kBlock];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double ke = 0.0;
  if (p < N) {
    const int32_t t = type[p];
    const double inv = mt.inv_mxi[t];
    for (int c = 0; c < 3; ++c) {
      const double vv = v[c * N + p] + 0.5 * dt * (double)F[c * N + p] * inv;
      v[c * N + p] = vv;
      ke += vv * vv;
    }
    ke *= 0.5 * mt.mass[t] * 103.642697;
  }
  if constexpr (KE) block_partial(ke, sh, partial + (int64_t)blockIdx.x * kPartialStride + P_KE);
}

__global__ void k_kinetic(int64_t N, const double* __restrict__ v, const int32_t* __restrict__ type,
                          MassTable mt, double* __restrict__ partial) {
  __shared__ double sh[kBlock];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double ke = 0.0;
  if (p < N) {
    const double m = mt.mass[type[p]];
    for (int c = 0; c < 3; ++c) ke += v[c * N + p] * v[c * N + p];
    ke *= 0.5 * m * 103.642697;
  }
  block_partial(ke, sh, partial + (int64_t)blockIdx.x * kPartialStride + P_KE);
}

__global__ void k_force_error(int64_t N, const float* __restrict__ Fa, const float* __restrict__ Fb,
                              double* __restrict__ partial) {
  __shared__ double sh[kBlock];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double e2 = 0.0, f2 = 0.0;
  if (p < N) {
    for (int c = 0; c < 3; ++c) {
      const double a = (double)Fa[c * N + p];
      const double d = a - (double)Fb[c * N + p];
      e2 += d * d;
      f2 += a * a;
    }
  }
  block_partial(e2, sh, partial + (int64_t)blockIdx.x * kPartialStride + P_ERR2);
  block_partial(f2, sh, partial + (int64_t)blockIdx.x * kPartialStride + P_F2);
  // maximum |e| over the block
  __syncthreads();
  sh[threadIdx.x] = sqrt(e2);
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < (unsigned)off) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[(int64_t)blockIdx.x * kPartialStride + P_ERRMAX] = sh[0];
}

// One half step (h = dt/2) of a Nose-Hoover chain in the explicit reversible
// Trotter form of Martyna, Tuckerman, Tobias and Klein (1996), FP64, one thread.
// ke = the current kinetic energy, scaled on return; returns the velocity scale.
// Chain masses Q_1 = Nf kT tau^2, Q_k = kT tau^2; forces G_1 = (2 KE - Nf kT)/Q_1,
// G_k = (Q_{k-1} v_{k-1}^2 - kT)/Q_k. The outermost velocity takes a quarter-step kick,
// the chain is swept inwards (each v_k damped by exp(-v_{k+1} h/4) around its kick),
// the particle velocities are to be scaled by exp(-v_1 h), the positions advance by
// v_k h, and the chain is swept outwards again with the forces recomputed.
__device__ double nhc_half(double& ke, double* eta, double* ve, int M, double kT, double Nf, double tau2, double h) {
  const double Q1 = Nf * kT * tau2, Qk = kT * tau2;
  auto force = [&](int k) {
    return k == 0 ? (2.0 * ke - Nf * kT) / Q1 : ((k == 1 ? Q1 : Qk) * ve[k - 1] * ve[k - 1] - kT) / Qk;
  };
  const int L = M - 1;
  ve[L] += 0.5 * h * force(L);
  for (int k = L - 1; k >= 0; --k) {
    const double d = exp(-0.25 * h * ve[k + 1]);
    ve[k] = (ve[k] * d + 0.5 * h * force(k)) * d;
  }
  const double sc = exp(-h * ve[0]);
  ke *= sc * sc;
  for (int k = 0; k < M; ++k) eta[k] += h * ve[k];
  for (int k = 0; k < L; ++k) {
    const double d = exp(-0.25 * h * ve[k + 1]);
    ve[k] = (ve[k] * d + 0.5 * h * force(k)) * d;
  }
  ve[L] += 0.5 * h * force(L);
  return sc;
}

// The kinetic energy from the nblocks P_KE partials, in every thread of a workgroup of
// kRedBlock; sh holds kRedBlock / 64 doubles.
__device__ double kinetic_sum(const double* partial, int nblocks, double* sh) {
  double ke = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < nblocks; b += kRedBlock) ke += partial[(int64_t)b * kPartialStride + P_KE];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ke += __shfl_xor(ke, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ke;
  __syncthreads();
  ke = 0.0;
  for (int k = 0; k < kRedBlock / 64; ++k) ke += sh[k];
  return ke;
}

// What k_kinetic leaves in the P_KE partials for the velocities v scale, by one workgroup of
// kRedBlock threads (the same additions in the same order, four of its workgroups at a time).
__device__ void kinetic_partials(int64_t N, const double* v, double scale, const int32_t* type, const MassTable& mt,
                                 double* partial, int nblocks, double* sh) {
  const int t = threadIdx.x % kBlock, g = threadIdx.x / kBlock;
  double* s = sh + g * kBlock;
  for (int b0 = 0; b0 < nblocks; b0 += kRedBlock / kBlock) {
    const int b = b0 + g;
    const int64_t p = (int64_t)b * kBlock + t;
    double ke = 0.0;
    if (p < N) {
      const double m = mt.mass[type[p]];
      for (int c = 0; c < 3; ++c) {
        const double vv = v[c * N + p] * scale;
        ke += vv * vv;
      }
      ke *= 0.5 * m * 103.642697;
    }
    __syncthreads();
    s[t] = ke;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
      if (t < off) s[t] += s[t + off];
      __syncthreads();
    }
    if (t == 0 && b < nblocks) partial[(int64_t)b * kPartialStride + P_KE] = s[0];
  }
  __syncthreads();
}

// The chain's half steps between two kicks (see launch_nhc): the sum of the kinetic energy's
// partials and both half steps in one launch, where each half step took four (kinetic
// energy, its sum, the chain, the scaling of v, which the next kick now does): 36 of the 240 us
// of a 33,660-atom step. flags (nullable): after a step that rebuilt its lists early the
// kinetic energy is taken from the scaled velocities, as a run resumed from that step takes
// it, not carried through the scaling (the two differ in the last places); rare, so that
// this one workgroup may do it.
__global__ void __launch_bounds__(kRedBlock)
k_nhc(double* partial, int nblocks, double* __restrict__ nhc, int M, double kT, double Nf, double tau2, double h,
      int trail, int lead, const int32_t* __restrict__ flags, int64_t N, const double* __restrict__ v,
      const int32_t* __restrict__ type, MassTable mt) {
  __shared__ double sh[kRedBlock], scale;
  const bool rebuilt = flags && flags[FLAG_REBUILD] != 0;
  double ke = partial ? kinetic_sum(partial, nblocks, sh) : nhc[kNhcKe];
  if (threadIdx.x != 0 && !rebuilt) return;
  double eta[kMaxChain], ve[kMaxChain];
  if (threadIdx.x == 0) {
    for (int k = 0; k < M; ++k) {
      eta[k] = nhc[k];
      ve[k] = nhc[kMaxChain + k];
    }
    const double s = trail ? nhc_half(ke, eta, ve, M, kT, Nf, tau2, h) : 1.0;
    nhc[kNhcTrail] = s;
    scale = s;
  }
  if (rebuilt) {
    __syncthreads();
    kinetic_partials(N, v, scale, type, mt, partial, nblocks, sh);
    ke = kinetic_sum(partial, nblocks, sh);
    if (threadIdx.x != 0) return;
  }
  nhc[kNhcLead] = lead ? nhc_half(ke, eta, ve, M, kT, Nf, tau2, h) : 1.0;
  nhc[kNhcKe] = ke;
  for (int k = 0; k < M; ++k) {
    nhc[k] = eta[k];
    nhc[kMaxChain + k] = ve[k];
  }
}

// v *= scale (the chain's velocity scaling), all 3N components.
__global__ void k_scale_v(int64_t n3, const double* __restrict__ scale, double* __restrict__ v) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n3) v[k] *= *scale;
}

__global__ void k_max_partials(const double* __restrict__ partial, int nblocks, int slot,
                               double* __restrict__ out) {
  __shared__ double sh[kBlock];
  double m = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += kBlock) m = fmax(m, partial[(int64_t)b * kPartialStride + slot]);
  sh[threadIdx.x] = m;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < (unsigned)off) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

__global__ void k_sum_i32(int64_t N, const int32_t* __restrict__ a, double* __restrict__ partial, int slot) {
  __shared__ double sh[kBlock];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  block_partial(p < N ? (double)a[p] : 0.0, sh, partial + (int64_t)blockIdx.x * kPartialStride + slot);
}

// A place in the box for a coordinate that is no number, which keeps what is queued before the
// host has seen the error in bounds and at its ordinary cost: fractional parts of multiples of
// the golden ratio and of two more irrationals fill the box evenly. One place for all of them
// would make one cell of a whole bad configuration, whose 20,000 atoms the list build would sort
// and pair in seconds.
__device__ __forceinline__ double stand_in(int64_t p, int c, double L) {
  const double a = c == 0 ? 0.6180339887498949 : (c == 1 ? 0.7548776662466927 : 0.8191725133961645);
  const double t = a * (double)(p + 1);
  return L * (t - floor(t));
}

// err: the words that report a bad species or value, the flags themselves or host words at the
// same indices (then the flags start from zero here).
__global__ void k_state_in(int64_t N, const double* __restrict__ xa, const double* __restrict__ va,
                           const int32_t* __restrict__ tin, int n_types, CellGrid g, double* __restrict__ x,
                           double* __restrict__ v, int32_t* __restrict__ type, int32_t* __restrict__ perm,
                           uint4* __restrict__ pos, int32_t* flags, int32_t* err) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < FLAG_COUNT && err != flags) flags[p] = 0;
  if (p >= N) return;
  double xn[3];
  for (int c = 0; c < 3; ++c) {
    double xv = xa[3 * p + c];
    if (!isfinite(xv)) {
      err[FLAG_NONFINITE] = 1;
      xv = stand_in(p, c, g.box[c]);
    }
    if (xv < 0.0 || xv >= g.box[c]) {
      xv = xv - g.box[c] * floor(xv / g.box[c]);
      if (xv >= g.box[c]) xv -= g.box[c];
    }
    x[c * N + p] = xv;
    xn[c] = xv;
    const double vv = va ? va[3 * p + c] : 0.0;
    if (!isfinite(vv)) err[FLAG_NONFINITE] = 1;
    v[c * N + p] = vv;
  }
  const int t = tin[p];
  const bool bad = t < 0 || t >= n_types;
  if (bad) err[FLAG_TYPE] = 1;
  pos_put(pos, p, xn[0], xn[1], xn[2], bad ? 0 : t, g.box);
  type[p] = bad ? 0 : t;
  perm[p] = (int32_t)p;
}

__global__ void k_state_out(int64_t N, const int32_t* __restrict__ perm, const double* __restrict__ soa,
                            double* __restrict__ aos) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  const int64_t o = perm[p];
  for (int c = 0; c < 3; ++c) aos[3 * o + c] = soa[c * N + p];
}

}  // namespace

hipError_t launch_reduce_partials(const double* partial, int nblocks, int first, int nvals, double* out,
                                  hipStream_t st) {
  hipLaunchKernelGGL(k_reduce_partials, dim3(1), dim3(kRedBlock), 0, st, partial, nblocks, first, nvals, out);
  return hipGetLastError();
}

hipError_t launch_max_partials(const double* partial, int nblocks, int slot, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_max_partials, dim3(1), dim3(kBlock), 0, st, partial, nblocks, slot, out);
  return hipGetLastError();
}

int kick_drift_blocks(int64_t N) {
  const int nb = grid_blocks(N);
  return nb < kIntegrateGrid ? nb : kIntegrateGrid;
}

hipError_t launch_kick_drift(int64_t N, double dt, CellGrid g, const float* F, const int32_t* type,
                             MassTable mt, double* x, double* v, uint4* pos, const double* x_build, bool pending,
                             const double* nhc, double* d2, hipStream_t st) {
  auto kern = nhc ? (pending ? k_kick_drift<true, true> : k_kick_drift<false, true>)
                  : (pending ? k_kick_drift<true, false> : k_kick_drift<false, false>);
  hipLaunchKernelGGL(kern, dim3(kick_drift_blocks(N)), dim3(kBlock), 0, st, N, dt, g, F, type, mt, x, v, pos, x_build,
                     nhc, d2);
  return hipGetLastError();
}

hipError_t launch_nhc(int64_t N, double* partial, int nblocks, double* nhc, int M, double kT, double tau, double h,
                      bool trail, bool lead, const int32_t* flags, const double* v, const int32_t* type, MassTable mt,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_nhc, dim3(1), dim3(kRedBlock), 0, st, partial, nblocks, nhc, M, kT, 3.0 * (double)N - 3.0,
                     tau * tau, h, trail ? 1 : 0, lead ? 1 : 0, flags, N, v, type, mt);
  return hipGetLastError();
}

hipError_t launch_scale_v(int64_t N, const double* nhc, double* v, hipStream_t st) {
  hipLaunchKernelGGL(k_scale_v, dim3(grid_blocks(3 * N)), dim3(kBlock), 0, st, 3 * N, nhc + kNhcTrail, v);
  return hipGetLastError();
}

hipError_t launch_kick(int64_t N, double dt, const float* F, const int32_t* type, MassTable mt, double* v,
                       double* ke_partial, hipStream_t st) {
  if (ke_partial)
    hipLaunchKernelGGL(k_kick<true>, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, dt, F, type, mt, v, ke_partial);
  else
    hipLaunchKernelGGL(k_kick<false>, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, dt, F, type, mt, v, ke_partial);
  return hipGetLastError();
}

hipError_t launch_kick_diff(int64_t N, double dt, const float* Fa, const float* Fb, const int32_t* type,
                            MassTable mt, double* v, hipStream_t st) {
  hipLaunchKernelGGL(k_kick_diff, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, dt, Fa, Fb, type, mt, v);
  return hipGetLastError();
}

hipError_t launch_kinetic(int64_t N, const double* v, const int32_t* type, MassTable mt, double* partial,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_kinetic, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, v, type, mt, partial);
  return hipGetLastError();
}

hipError_t launch_force_error(int64_t N, const float* Fa, const float* Fb, double* partial,
                              hipStream_t st) {
  hipLaunchKernelGGL(k_force_error, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, Fa, Fb, partial);
  return hipGetLastError();
}

hipError_t launch_sum_i32(int64_t N, const int32_t* a, double* partial, int slot, hipStream_t st) {
  hipLaunchKernelGGL(k_sum_i32, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, a, partial, slot);
  return hipGetLastError();
}

hipError_t launch_state_in(int64_t N, const double* x_aos, const double* v_aos, const int32_t* type_in,
                           int n_types, CellGrid g, double* x, double* v, int32_t* type, int32_t* perm,
                           uint4* pos, int32_t* flags, int32_t* err, hipStream_t st) {
  hipLaunchKernelGGL(k_state_in, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, x_aos, v_aos, type_in,
                     n_types, g, x, v, type, perm, pos, flags, err);
  return hipGetLastError();
}

hipError_t launch_state_out(int64_t N, const int32_t* perm, const double* soa, double* aos, hipStream_t st) {
  hipLaunchKernelGGL(k_state_out, dim3(grid_blocks(N)), dim3(kBlock), 0, st, N, perm, soa, aos);
  return hipGetLastError();
}

template <class R>
static hipError_t results(const double* ew, int ew_rows, double* out, int64_t N, const int32_t* perm, const R* F,
                          const R* U, double* forces, double* energies, const int32_t* gate, hipStream_t st) {
  const int nb = 1 + (forces || energies ? grid_blocks(N, kRedBlock) : 0);
  hipLaunchKernelGGL(k_results<R>, dim3(nb), dim3(kRedBlock), 0, st, ew, ew_rows, out, N, perm, F, U, forces,
                     energies, gate);
  return hipGetLastError();
}
hipError_t launch_results(const double* ew, int ew_rows, double* out, int64_t N, const int32_t* perm, const float* F,
                          const float* U, double* forces, double* energies, const int32_t* gate, hipStream_t st) {
  return results(ew, ew_rows, out, N, perm, F, U, forces, energies, gate, st);
}
hipError_t launch_results64(const double* ew, int ew_rows, double* out, int64_t N, const int32_t* perm,
                            const double* F, const double* U, double* forces, double* energies, const int32_t* gate,
                            hipStream_t st) {
  return results(ew, ew_rows, out, N, perm, F, U, forces, energies, gate, st);
}
hipError_t launch_results_f32(const double* ew, int ew_rows, double* out, int64_t N, const int32_t* perm,
                              const float* F, float* forces, hipStream_t st) {
  hipLaunchKernelGGL(k_results_f32, dim3(1 + (forces ? grid_blocks(N, kRedBlock) : 0)), dim3(kRedBlock), 0, st, ew,
                     ew_rows, out, N, perm, F, forces);
  return hipGetLastError();
}

}  // namespace nep
