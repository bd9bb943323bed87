// Direct-form (VALU) kernels for float and double: model fold, LWPR
// prediction, sampled rollouts, sub-rollout averaging, the path-integral
// update and the receding-horizon shift.  One lane evaluates one input
// against every local model; model records are staged through LDS tiles and
// read as broadcasts.  (PI^2-RH with LWPR dynamics, arXiv:1503.00330.)
#include <algorithm>

#include "direct.hpp"

namespace pi2rh {

// ----------------------------------------------------------------- fold
// One block per 16 local models, 16 lanes each (one input coordinate per lane).
// The lanes of a model fold its PLS chain (Sec. 2) into y = beta_0 + b . (z - c)
// -- b is the derivative of y w.r.t. the centred input, accumulated backwards
// through the deflation steps in double -- then all lanes write the 16
// contiguous records, coalesced:
// [c | theta (upper triangle of D + D^T, diagonal D_aa) | b | beta_0 | sigma^2].
// Bound by latency: 1536 models of d = 16 28 us with one lane per model and
// the pair of every entry searched for, 15 us so.
template <typename Real>
__global__ void __launch_bounds__(256) fold_direct_kernel(ModelArgs m, Real *__restrict__ rec) {
  __shared__ Real bv[16][kMaxD];
  __shared__ Real Dl[16][kMaxD * kMaxD + 1];
  __shared__ unsigned char pa[kMaxD * (kMaxD + 1) / 2], pb[kMaxD * (kMaxD + 1) / 2];
  const int j0 = blockIdx.x * 16, d = m.d, R = m.R, RS = d + d * (d + 1) / 2 + d + 2;
  const int nj = min(16, m.Ltot - j0), np = d * (d + 1) / 2;
  for (int e = threadIdx.x; e < nj * d * d; e += 256)
    Dl[e / (d * d)][e % (d * d)] = ((const Real *)m.metric)[(size_t)j0 * d * d + e];
  if ((int)threadIdx.x < np) {
    int a = 0, rem = threadIdx.x;
    while (rem >= d - a) {
      rem -= d - a;
      ++a;
    }
    pa[threadIdx.x] = (unsigned char)a;
    pb[threadIdx.x] = (unsigned char)(a + rem);
  }
  {
    const int col = threadIdx.x >> 4, a = threadIdx.x & 15;
    const bool on = col < nj && a < d;
    const size_t j = (size_t)j0 + (col < nj ? col : 0);
    const Real *U = (const Real *)m.proj_u + j * R * d;
    const Real *P = m.proj_p ? (const Real *)m.proj_p + j * R * d : U;
    const Real *B = (const Real *)m.beta + j * (R + 1);
    Real ru[kMaxR], rp[kMaxR], rbeta[kMaxR];
#pragma unroll
    for (int r = 0; r < kMaxR; ++r) {
      const bool use = r < R && on;
      ru[r] = use ? U[r * d + a] : (Real)0;
      rp[r] = use ? P[r * d + a] : (Real)0;
      rbeta[r] = r < R && col < nj ? B[r + 1] : (Real)0;
    }
    double rb = 0.0;
#pragma unroll
    for (int r = kMaxR - 1; r >= 0; --r) {
      if (r >= R) continue;
      double pr = (double)rp[r] * rb;
#pragma unroll
      for (int k = 8; k >= 1; k >>= 1) pr += __shfl_xor(pr, k);
      // lanes without a coordinate stay 0: an infinite coefficient times 0 is not
      rb += on ? ((double)rbeta[r] - pr) * (double)ru[r] : 0.0;
    }
    if (on) bv[col][a] = (Real)rb;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < nj * RS; e += 256) {
    const int jj = e / RS, f = e % RS, j = j0 + jj;
    Real v;
    if (f < d) {
      v = ((const Real *)m.centre)[(size_t)j * d + f];
    } else if (f < d + np) {
      const int a = pa[f - d], b = pb[f - d];
      v = (a == b) ? Dl[jj][a * d + a] : Dl[jj][a * d + b] + Dl[jj][b * d + a];
    } else if (f < d + np + d) {
      v = bv[jj][f - d - np];
    } else if (f == d + np + d) {
      v = ((const Real *)m.beta)[(size_t)j * (R + 1)];
    } else {
      v = ((const Real *)m.sigma2)[j];
    }
    rec[(size_t)j0 * RS + e] = v;
  }
}

hipError_t launch_fold_direct(int dtype, const ModelArgs &m, void *rec, hipStream_t s) {
  const int nb = (m.Ltot + 15) / 16;
  if (dtype == PI_F64)
    hipLaunchKernelGGL(fold_direct_kernel<double>, dim3(nb), dim3(256), 0, s, m, (double *)rec);
  else
    hipLaunchKernelGGL(fold_direct_kernel<float>, dim3(nb), dim3(256), 0, s, m, (float *)rec);
  return hipGetLastError();
}

template <typename Real, int D>
__global__ void __launch_bounds__(128) predict_direct_kernel(ModelArgs m, const Real *__restrict__ rec,
                                                             const Real *__restrict__ Z, int64_t N,
                                                             Real *__restrict__ mean,
                                                             Real *__restrict__ var) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Real *tile = (Real *)smem_raw;
  Real *out = tile + tile_models<Real, D>() * rec_stride<Real, D>() + threadIdx.x * 2 * kMaxOut;
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  Real z[D];
#pragma unroll
  for (int a = 0; a < D; ++a) z[a] = n < N ? Z[n * D + a] : (Real)0;
  direct_mixture<Real, D>(m, rec, z, tile, out);
  if (n < N)
    for (int o = 0; o < m.n_out; ++o) {
      mean[n * m.n_out + o] = out[o];
      var[n * m.n_out + o] = out[kMaxOut + o];
    }
}

template <typename Real, int D>
static hipError_t predict_direct_d(const ModelArgs &m, const void *rec, const void *Z, int64_t N,
                                   void *mean, void *var, hipStream_t s) {
  const size_t sh = (size_t)(tile_models<Real, D>() * rec_stride<Real, D>() + 128 * 2 * kMaxOut) *
                    sizeof(Real);
  const int64_t nb = (N + 127) / 128;
  hipLaunchKernelGGL((predict_direct_kernel<Real, D>), dim3((unsigned)nb), dim3(128), sh, s, m,
                     (const Real *)rec, (const Real *)Z, N, (Real *)mean, (Real *)var);
  return hipGetLastError();
}

template <typename Real>
static hipError_t predict_direct_t(const ModelArgs &m, const void *rec, const void *Z, int64_t N,
                                   void *mean, void *var, hipStream_t s) {
  switch (m.d) {
#define PI_CASE(DD) \
  case DD:          \
    return predict_direct_d<Real, DD>(m, rec, Z, N, mean, var, s);
    PI_CASE(1) PI_CASE(2) PI_CASE(3) PI_CASE(4) PI_CASE(5) PI_CASE(6) PI_CASE(7) PI_CASE(8)
    PI_CASE(9) PI_CASE(10) PI_CASE(11) PI_CASE(12) PI_CASE(13) PI_CASE(14) PI_CASE(15) PI_CASE(16)
#undef PI_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_predict_direct(int dtype, const ModelArgs &m, const void *rec, const void *Z,
                                 int64_t N, void *mean, void *var, hipStream_t s) {
  if (N == 0) return hipSuccess;
  return dtype == PI_F64 ? predict_direct_t<double>(m, rec, Z, N, mean, var, s)
                         : predict_direct_t<float>(m, rec, Z, N, mean, var, s);
}

// Predictions of few inputs from a model as given: one wave per (input, output), a lane
// per local model, statistics merged by xor shuffles, all in double.  It spares the
// fold and its launch.  Bound by launch and memory latency: 33 inputs, models
// 16/16, whole call 17.6 us with the fold, 14.6 us so.
template <typename Real, int D>
__global__ void __launch_bounds__(256) predict_raw_kernel(ModelArgs m, const Real *__restrict__ Z, int64_t N,
                                                          Real *__restrict__ mean, Real *__restrict__ var) {
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), n = w / m.n_out;
  const int o = (int)(w - n * m.n_out);
  if (n >= N) return;
  double z[D];
#pragma unroll
  for (int a = 0; a < D; ++a) z[a] = (double)Z[n * D + a];
  MixStat<double> st = mix_empty<double>();
  for (int j = m.L_off[o] + lane; j < m.L_off[o + 1]; j += 64) {
    const Real *c = (const Real *)m.centre + (size_t)j * D, *M = (const Real *)m.metric + (size_t)j * D * D;
    const Real *U = (const Real *)m.proj_u + (size_t)j * m.R * D;
    const Real *P = m.proj_p ? (const Real *)m.proj_p + (size_t)j * m.R * D : U;
    const Real *B = (const Real *)m.beta + (size_t)j * (m.R + 1);
    double dl[D], r[D], q = 0.0, y = (double)B[0];
#pragma unroll
    for (int a = 0; a < D; ++a) r[a] = dl[a] = z[a] - (double)c[a];
#pragma unroll
    for (int a = 0; a < D; ++a) {
      double row = 0.0;
#pragma unroll
      for (int b = 0; b < D; ++b) row += (double)M[a * D + b] * dl[b];
      q += dl[a] * row;
    }
    for (int k = 0; k < m.R; ++k) {
      double s = 0.0;
#pragma unroll
      for (int a = 0; a < D; ++a) s += (double)U[k * D + a] * r[a];
#pragma unroll
      for (int a = 0; a < D; ++a) r[a] -= s * (double)P[k * D + a];
      y += (double)B[k + 1] * s;
    }
    mix_add<false>(st, -0.5 * q, y, (double)((const Real *)m.sigma2)[j]);
  }
#pragma unroll
  for (int msk = 32; msk >= 1; msk >>= 1) st = mix_merge<false>(st, shfl_stat(st, msk));
  double mu, v;
  mix_finish(st, &mu, &v);
  if (lane == 0) {
    mean[n * m.n_out + o] = (Real)mu;
    var[n * m.n_out + o] = (Real)v;
  }
}

hipError_t launch_predict_raw(int dtype, const ModelArgs &m, const void *Z, int64_t N, void *mean, void *var,
                              hipStream_t s) {
  const dim3 grid((unsigned)((N * m.n_out + 3) / 4)), block(256);
#define PI_RAW(T, DD) \
  hipLaunchKernelGGL((predict_raw_kernel<T, DD>), grid, block, 0, s, m, (const T *)Z, N, (T *)mean, (T *)var)
  if (dtype == PI_F64) {
    if (m.d == 4) PI_RAW(double, 4);
    else PI_RAW(double, 6);
  } else {
    if (m.d == 4) PI_RAW(float, 4);
    else PI_RAW(float, 6);
  }
#undef PI_RAW
  return hipGetLastError();
}

// One lane per sub-rollout (k, m): every step draws eps_{k,t} (shared by the
// sub-rollouts of k) and xi_{k,m,t}, evaluates Eq. (1) at z = [x ; u_nom + eps],
// samples the accelerations, steps Euler and writes dt * q(x_{t+1}).
template <typename Real, int DYN>
__global__ void __launch_bounds__(128) rollout_direct_kernel(RolloutArgs<Real> ra, ModelArgs m,
                                                             const Real *__restrict__ rec) {
  using DD = DynDims<DYN>;
  constexpr int D = DD::D, NX = DD::NX, NU = DD::NU, NO = DD::NO;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Real *tile = (Real *)smem_raw;
  Real *outb = tile + tile_models<Real, D>() * rec_stride<Real, D>();
  Real *out = outb + threadIdx.x * 2 * kMaxOut;
  Real *obs = outb + blockDim.x * 2 * kMaxOut;
  const ProbDev<Real> &p = ra.p;
  for (int i = threadIdx.x; i < 3 * p.n_obs; i += blockDim.x) obs[i] = p.obs[i];
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool active = s < (int64_t)p.K * p.Ms;
  const uint32_t k = (uint32_t)(s / p.Ms), mm = (uint32_t)(s % p.Ms);
  const uint32_t it = *ra.iter;
  const uint32_t wc = stream_word(kTagCtrl, p.problem_id, it);
  const uint32_t wd = stream_word(kTagDyn, p.problem_id, it);
  Real x[NX];
#pragma unroll
  for (int a = 0; a < NX; ++a) x[a] = ra.x0[a];
  __syncthreads();
  for (int t = 0; t < p.T; ++t) {
    Real eps[4], u[NU], pert[NU];
    normals<Real, NU>(p.key0, p.key1, wc, k, 0u, (uint32_t)t, eps);
#pragma unroll
    for (int a = 0; a < NU; ++a) {
      pert[a] = p.noise_std[a] * eps[a];
      u[a] = ra.u_nom[t * NU + a] + pert[a];
    }
    Real cu = 0;
    if constexpr (DYN == kDynQuadHybrid)
      if (p.ctrl_cost) cu = control_cost<Real>(p, ra.u_nom + t * NU, pert);
    Real z[D];
    lwpr_input<DYN>(x, u, z);
    direct_mixture<Real, D>(m, rec, z, tile, out);
    Real acc[NO];
    if (p.M > 0) {
      Real xi[8];
      normals<Real, NO>(p.key0, p.key1, wd, k, mm, (uint32_t)t, xi);
#pragma unroll
      for (int o = 0; o < NO; ++o) acc[o] = out[o] + sqrt_(out[kMaxOut + o]) * xi[o];
    } else {
#pragma unroll
      for (int o = 0; o < NO; ++o) acc[o] = out[o];
    }
    Real xn[NX];
    euler_step<Real>(DYN, p.dt, x, acc, u, xn);
#pragma unroll
    for (int a = 0; a < NX; ++a) x[a] = xn[a];
    const Real c = p.dt * state_cost<Real>(p, obs, x) + cu;
    if (active) ra.cost[s * p.T + t] = c;
  }
}

// Small problems: 16 lanes per sub-rollout split the local models of every
// output (merged by xor shuffles in a fixed order), 16 sub-rollouts per block;
// lane 0 of each sub-rollout samples, steps Euler and writes the cost.  The
// lanes draw the noise of the next 16 steps together (lane l: step t + l), and
// a model that fits in LDS is staged once, so a step has a single barrier.
// Sixteen times the threads of the lane-per-sub-rollout kernel, for grids
// that would otherwise leave most of the chip idle.
constexpr int kGroupLanes = 16, kGroupRows = 16, kGroupChunk = 16;
template <typename Real, int DYN>
__global__ void __launch_bounds__(kGroupLanes *kGroupRows) rollout_group_kernel(RolloutArgs<Real> ra, ModelArgs m,
                                                                              const Real *__restrict__ rec) {
  using DD = DynDims<DYN>;
  constexpr int D = DD::D, NX = DD::NX, NU = DD::NU, NO = DD::NO;
  constexpr int RS = rec_stride<Real, D>(), TM = tile_models<Real, D>();
  __shared__ Real tile[TM * RS];
  __shared__ Real zs[kGroupRows][D];
  // applied controls u_nom + sigma eps and next-state draws of the chunk's steps
  __shared__ Real us_s[kGroupChunk][kGroupRows][4], xi_s[kGroupChunk][kGroupRows][8];
  __shared__ Real obs[kMaxObs * 3];
  const ProbDev<Real> &p = ra.p;
  for (int i = threadIdx.x; i < 3 * p.n_obs; i += blockDim.x) obs[i] = p.obs[i];
  const bool resident = m.Ltot <= TM;   // the whole model in LDS for the whole rollout
  if (resident)
    for (int i = threadIdx.x; i < m.Ltot * RS; i += blockDim.x) tile[i] = rec[i];
  const int g = threadIdx.x / kGroupLanes, l = threadIdx.x % kGroupLanes;
  const int64_t s = (int64_t)blockIdx.x * kGroupRows + g;
  const bool active = s < (int64_t)p.K * p.Ms;
  const uint32_t k = active ? (uint32_t)(s / p.Ms) : 0u, mm = active ? (uint32_t)(s % p.Ms) : 0u;
  const uint32_t it = *ra.iter;
  const uint32_t wc = stream_word(kTagCtrl, p.problem_id, it);
  const uint32_t wd = stream_word(kTagDyn, p.problem_id, it);
  Real x[NX], u[NU];
#pragma unroll
  for (int a = 0; a < NX; ++a) x[a] = ra.x0[a];
  for (int t = 0; t < p.T; ++t) {
    const int tc = t % kGroupChunk;
    if (tc == 0) {
      __syncthreads();   // lane 0 of every row is done with the previous chunk
      if (active && t + l < p.T) {
        Real e[NU], pert[NU];
        normals<Real, NU>(p.key0, p.key1, wc, k, 0u, (uint32_t)(t + l), e);
#pragma unroll
        for (int a = 0; a < NU; ++a) {
          pert[a] = p.noise_std[a] * e[a];
          us_s[l][g][a] = ra.u_nom[(t + l) * NU + a] + pert[a];
        }
        if (p.M > 0) normals<Real, NO>(p.key0, p.key1, wd, k, mm, (uint32_t)(t + l), xi_s[l][g]);
        // the step's control terms ride in the draw slot the hybrid model leaves unused
        if constexpr (DYN == kDynQuadHybrid)
          if (p.ctrl_cost) xi_s[l][g][7] = control_cost<Real>(p, ra.u_nom + (t + l) * NU, pert);
      }
    }
    if (l == 0) {
      Real z[D];
      if (active) {
#pragma unroll
        for (int a = 0; a < NU; ++a) u[a] = us_s[tc][g][a];
        lwpr_input<DYN>(x, u, z);
      } else {
#pragma unroll
        for (int a = 0; a < D; ++a) z[a] = 0;
      }
#pragma unroll
      for (int a = 0; a < D; ++a) zs[g][a] = z[a];
    }
    __syncthreads();
    Real zz[D];
#pragma unroll
    for (int a = 0; a < D; ++a) zz[a] = zs[g][a];
    Real acc[NO];
    for (int o = 0; o < NO; ++o) {
      MixStat<Real> st = mix_empty<Real>();
      for (int j0 = m.L_off[o]; j0 < m.L_off[o + 1]; j0 += TM) {
        const int nj = min(TM, m.L_off[o + 1] - j0);
        const Real *base = tile;
        if (resident) {
          base = tile + (size_t)j0 * RS;
        } else {
          __syncthreads();
          for (int i = threadIdx.x; i < nj * RS; i += blockDim.x) tile[i] = rec[(size_t)j0 * RS + i];
          __syncthreads();
        }
        for (int jj = l; jj < nj; jj += kGroupLanes) {
          Real q, y;
          eval_record<Real, D>(base + jj * RS, zz, q, y);
          mix_add<false>(st, (Real)-0.5 * q, y, base[jj * RS + RS - 1]);
        }
      }
#pragma unroll
      for (int msk = 8; msk >= 1; msk >>= 1) st = mix_merge<false>(st, shfl_stat(st, msk));
      if (l == 0) {   // every lane holds the merged statistics; lane 0 owns the draws
        Real mu, v;
        mix_finish(st, &mu, &v);
        acc[o] = p.M > 0 ? mu + sqrt_(v) * xi_s[tc][g][o] : mu;
      }
    }
    if (l == 0 && active) {
      Real xn[NX];
      euler_step<Real>(DYN, p.dt, x, acc, u, xn);
#pragma unroll
      for (int a = 0; a < NX; ++a) x[a] = xn[a];
      Real c = p.dt * state_cost<Real>(p, obs, x);
      if constexpr (DYN == kDynQuadHybrid)
        if (p.ctrl_cost) c += xi_s[tc][g][7];
      ra.cost[s * p.T + t] = c;
    }
  }
}

template <typename Real>
static hipError_t rollout_group_t(const RolloutArgs<Real> &ra, const ModelArgs &m, const void *rec,
                                  hipStream_t s) {
  const int64_t n = (int64_t)ra.p.K * ra.p.Ms;
  const dim3 grid((unsigned)((n + kGroupRows - 1) / kGroupRows)), block(kGroupLanes * kGroupRows);
  if (ra.p.dyn == kDynPointMass2D)
    hipLaunchKernelGGL((rollout_group_kernel<Real, kDynPointMass2D>), grid, block, 0, s, ra, m, (const Real *)rec);
  else if (ra.p.dyn == kDynQuadHybrid)
    hipLaunchKernelGGL((rollout_group_kernel<Real, kDynQuadHybrid>), grid, block, 0, s, ra, m, (const Real *)rec);
  else
    hipLaunchKernelGGL((rollout_group_kernel<Real, kDynQuad12>), grid, block, 0, s, ra, m, (const Real *)rec);
  return hipGetLastError();
}

// -------------------------------------------------- small-model rollouts
// P lanes share one sub-rollout and its models (lane l: models l, l + P, ..), a wave
// holds 64 / P of them, and nothing but the wave's own lanes takes part in a step: the
// state is stepped by all P lanes alike, statistics cross lanes by DPP, there is no
// barrier.  The mixture is evaluated in two passes over registers (maximum, weights
// and mean; then the spread about the mean), one exponential per model.  Bound by
// the serial chain of a step where the chip is not full (P = 16), by vector
// instructions where it is (P = 4).  The whole step of 256 rollouts x 20, models
// 16/16, in double: 144 -> 55 us; 1000 x 50, models 15/15/24, in float 162 us (matrix
// cores) -> 65 us, 30400 sub-rollouts 366 -> 209 us.
__device__ __forceinline__ float exp_act(float x) { return __builtin_amdgcn_exp2f(x); }   // base 2, x <= 0
__device__ __forceinline__ double exp_act(double x) { return exp(x); }
__device__ __forceinline__ float root_(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double root_(double x) { return sqrt(x); }

template <typename Real, int D>
constexpr int rec_pad() {   // record stride in LDS: whole 16-byte words
  return (rec_stride<Real, D>() * (int)sizeof(Real) + 15) / 16 * 16 / (int)sizeof(Real);
}

template <typename Real, int DYN, int P, int NJ>
__global__ void __launch_bounds__(64, NJ > 2 ? 2 : 1) rollout_wave_kernel(RolloutArgs<Real> ra, ModelArgs m,
                                                                        const Real *__restrict__ rec) {
  using DD = DynDims<DYN>;
  constexpr int D = DD::D, NX = DD::NX, NU = DD::NU, NO = DD::NO;
  constexpr int RS = rec_stride<Real, D>(), RSP = rec_pad<Real, D>();
  extern __shared__ __attribute__((aligned(16))) char wave_lds[];
  Real *tile = (Real *)wave_lds;
  __shared__ Real obs[kMaxObs * 3];
  const ProbDev<Real> &p = ra.p;
  for (int i = threadIdx.x; i < 3 * p.n_obs; i += 64) obs[i] = p.obs[i];
  // Behind each output's records one of zeros, for the lanes past its last model, whose
  // weight is 0 (a repeated model's infinite parameter times that weight would be NaN).
  for (int i = threadIdx.x; i < m.Ltot * RS; i += 64) {
    const int j = i / RS;
    int slot = j;
#pragma unroll
    for (int o = 1; o < NO; ++o) slot += j >= m.L_off[o];
    tile[slot * RSP + i % RS] = rec[i];
  }
  for (int i = threadIdx.x; i < NO * RS; i += 64) {
    const int o = i / RS;
    tile[(m.L_off[o + 1] + o) * RSP + i % RS] = 0;
  }
  __syncthreads();
  const int l = threadIdx.x % P;
  const int64_t n = (int64_t)p.K * p.Ms, row = (int64_t)blockIdx.x * (64 / P) + threadIdx.x / P;
  const uint32_t s = (uint32_t)min(row, n - 1);   // lanes past the last sub-rollout repeat it
  const uint32_t k = p.Ms == 1 ? s : s / (uint32_t)p.Ms, mm = s - k * (uint32_t)p.Ms;
  const uint32_t it = *ra.iter;
  const uint32_t wc = stream_word(kTagCtrl, p.problem_id, it);
  const uint32_t wd = stream_word(kTagDyn, p.problem_id, it);
  const Real kAct = (Real)(sizeof(Real) == 4 ? -0.72134752044448170368 : -0.5);   // -log2(e) / 2 in float
  const Real ninf = -(Real)(1.0 / 0.0);
  auto add = [](Real a, Real b) { return a + b; };
  auto mx2 = [](Real a, Real b) { return a > b ? a : b; };
  Real x[NX], lo[NX];
#pragma unroll
  for (int a = 0; a < NX; ++a) x[a] = ra.x0[a], lo[a] = 0;
  for (int tb = 0; tb < p.T; tb += P) {
    // lane l draws step tb + l
    Real uc[NU], xc[NO], cc = 0, keep = 0;
    {
      const int t = min(tb + l, p.T - 1);
      Real e[NU], pert[NU];
      normals<Real, NU>(p.key0, p.key1, wc, k, 0u, (uint32_t)t, e);
#pragma unroll
      for (int a = 0; a < NU; ++a) {
        pert[a] = p.noise_std[a] * e[a];
        uc[a] = ra.u_nom[t * NU + a] + pert[a];
      }
#pragma unroll
      for (int o = 0; o < NO; ++o) xc[o] = 0;
      if (p.M > 0) normals<Real, NO>(p.key0, p.key1, wd, k, mm, (uint32_t)t, xc);
      if constexpr (DYN == kDynQuadHybrid)
        if (p.ctrl_cost) cc = control_cost<Real>(p, ra.u_nom + t * NU, pert);
    }
    const int nt = min(P, p.T - tb);
    for (int tc = 0; tc < nt; ++tc) {
      Real u[NU], xi[NO], z[D], acc[NO];
#pragma unroll
      for (int a = 0; a < NU; ++a) u[a] = __shfl(uc[a], tc, P);
#pragma unroll
      for (int o = 0; o < NO; ++o) xi[o] = p.M > 0 ? __shfl(xc[o], tc, P) : (Real)0;
      lwpr_input<DYN>(x, u, z);
      int off = 0;
      if constexpr (NJ > 2) asm volatile("" : "+s"(off));   // keep the records in LDS
// every model's distance and prediction, then the statistics of all
      // outputs side by side, whose chains hide each other's latency
      Real act[NO][NJ], y[NO][NJ], s2[NO][NJ], mx[NO], Z[NO], S1[NO], S2[NO], mu[NO];
      constexpr int G = NJ > 2 ? 2 : NJ;   // models between two looks at the output's end
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        const int j0 = m.L_off[o], L = m.L_off[o + 1] - j0;
#pragma unroll
        for (int g = 0; g < NJ; g += G) {
#pragma unroll
          for (int jj = g; jj < g + G; ++jj) act[o][jj] = ninf, y[o][jj] = 0, s2[o][jj] = 0;
          if (NJ > 2 && g * P >= L) continue;
#pragma unroll
          for (int jj = g; jj < g + G; ++jj) {
            const int j = jj * P + l;
            const Real *r = tile + off + (j0 + o + min(j, L)) * RSP;
            Real q;
            eval_record<Real, D>(r, z, q, y[o][jj]);
            act[o][jj] = j < L ? kAct * q : ninf;
            s2[o][jj] = r[RS - 1];
          }
        }
      }
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        mx[o] = act[o][0];
#pragma unroll
        for (int jj = 1; jj < NJ; ++jj) mx[o] = mx2(act[o][jj], mx[o]);
        mx[o] = lanes_reduce<P>(mx[o], mx2);
      }
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        Z[o] = S1[o] = S2[o] = 0;
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
          act[o][jj] = exp_act(act[o][jj] - mx[o]);
          Z[o] += act[o][jj];
          S1[o] += act[o][jj] * y[o][jj];
          S2[o] += act[o][jj] * s2[o][jj];
        }
        Z[o] = lanes_reduce<P>(Z[o], add);
        S1[o] = lanes_reduce<P>(S1[o], add);
      }
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        mu[o] = ratio(S1[o], Z[o]);
        acc[o] = mu[o];
      }
      if (p.M > 0) {
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          Real M2 = 0;
#pragma unroll
          for (int jj = 0; jj < NJ; ++jj) {
            const Real dy = y[o][jj] - mu[o];
            M2 += act[o][jj] * dy * dy;
          }
          acc[o] += root_(ratio(lanes_reduce<P>(M2 + S2[o], add), Z[o])) * xi[o];
        }
      }
      Real xn[NX];
      if constexpr (sizeof(Real) == 4)
        euler_step_comp(DYN, p.dt, x, acc, u, xn, lo);
      else
        euler_step<Real>(DYN, p.dt, x, acc, u, xn);
#pragma unroll
      for (int a = 0; a < NX; ++a) x[a] = xn[a];
      Real c = p.dt * state_cost_quad<Real, DYN>(p, obs, x, l % 4);
      if constexpr (DYN == kDynQuadHybrid)
        if (p.ctrl_cost) c += __shfl(cc, tc, P);
      keep = l == tc ? c : keep;
    }
    // lane l holds the cost of step tb + l
    if (row < n && l < nt) ra.cost[row * p.T + tb + l] = keep;
  }
}

// The lanes per sub-rollout: 16 while their waves leave the chip's vector units idle,
// then 4 (8 for more than 32 models per output), which reduce less and hold each
// lane's whole share of the models.  50 steps, models 15/15/24, float: 4000
// sub-rollouts 77 us with 16 lanes and 159 with 4, 16000 172 and 168, 30400 319 and
// 213; 16/16: 16000 97 and 139, 30400 177 and 182; 30/40/35: 4000 157 (8 lanes 183),
// 8000 195 (181); 16/16 in double: 8000 163 and 236, 16000 301 and 259.
template <typename Real, int DYN>
static hipError_t rollout_wave_t(const RolloutArgs<Real> &ra, const ModelArgs &m, const void *rec, hipStream_t s) {
  const int64_t n = (int64_t)ra.p.K * ra.p.Ms;
  const int L = max_models(m.n_out, m.L_off);
  const int64_t wide = L > 32 ? 6144 : L <= 16 && sizeof(Real) == 4 ? 24576 : 12288;
  const size_t lds = wave_lds_bytes(sizeof(Real) == 8 ? PI_F64 : PI_F32, m.d, m.Ltot + m.n_out);   // + the records of zeros
  auto go = [&](auto kernel, int lanes) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n * lanes + 63) / 64)), dim3(64), lds, s, ra, m, (const Real *)rec);
  };
  if (n <= wide) {
    if (L <= 16)
      go(rollout_wave_kernel<Real, DYN, 16, 1>, 16);
    else if (L <= 32)
      go(rollout_wave_kernel<Real, DYN, 16, 2>, 16);
    else
      go(rollout_wave_kernel<Real, DYN, 16, 4>, 16);
  } else if (L <= 16) {
    go(rollout_wave_kernel<Real, DYN, 4, 4>, 4);
  } else if (L <= 32) {
    go(rollout_wave_kernel<Real, DYN, 4, 8>, 4);
  } else {
    go(rollout_wave_kernel<Real, DYN, 8, 8>, 8);
  }
  return hipGetLastError();
}

template <typename Real>
static hipError_t rollout_direct_t(const RolloutArgs<Real> &ra, const ModelArgs &m, const void *rec,
                                   hipStream_t s) {
  const int64_t n = (int64_t)ra.p.K * ra.p.Ms;
  if (rollout_wave_ok(ra.p.dyn, sizeof(Real) == 8 ? PI_F64 : PI_F32, m.d, m.n_out, m.L_off, n))
    return ra.p.dyn == kDynPointMass2D ? rollout_wave_t<Real, kDynPointMass2D>(ra, m, rec, s)
                                       : rollout_wave_t<Real, kDynQuadHybrid>(ra, m, rec, s);
  // fewer sub-rollouts than 32 lanes per compute unit: split the models over lanes
  if (n < 256 * 32) return rollout_group_t(ra, m, rec, s);
  const unsigned nb = (unsigned)((n + 127) / 128);
  if (ra.p.dyn == kDynPointMass2D) {
    constexpr int D = 6;
    const size_t sh = (size_t)(tile_models<Real, D>() * rec_stride<Real, D>() + 128 * 2 * kMaxOut +
                               3 * kMaxObs) * sizeof(Real);
    hipLaunchKernelGGL((rollout_direct_kernel<Real, kDynPointMass2D>), dim3(nb), dim3(128), sh, s,
                       ra, m, (const Real *)rec);
  } else if (ra.p.dyn == kDynQuadHybrid) {
    constexpr int D = 4;
    const size_t sh = (size_t)(tile_models<Real, D>() * rec_stride<Real, D>() + 128 * 2 * kMaxOut +
                               3 * kMaxObs) * sizeof(Real);
    hipLaunchKernelGGL((rollout_direct_kernel<Real, kDynQuadHybrid>), dim3(nb), dim3(128), sh, s,
                       ra, m, (const Real *)rec);
  } else {
    constexpr int D = 16;
    const size_t sh = (size_t)(tile_models<Real, D>() * rec_stride<Real, D>() + 128 * 2 * kMaxOut +
                               3 * kMaxObs) * sizeof(Real);
    hipLaunchKernelGGL((rollout_direct_kernel<Real, kDynQuad12>), dim3(nb), dim3(128), sh, s, ra, m,
                       (const Real *)rec);
  }
  return hipGetLastError();
}

hipError_t launch_rollout_direct(int dtype, const void *rargs, const ModelArgs &m, const void *rec,
                                 hipStream_t s) {
  return dtype == PI_F64 ? rollout_direct_t<double>(*(const RolloutArgs<double> *)rargs, m, rec, s)
                         : rollout_direct_t<float>(*(const RolloutArgs<float> *)rargs, m, rec, s);
}

// -------------------------------------------------- sub-rollout average
// cbar_{k,t} = (1/M) sum_m c_{k,m,t} (Sec. 3.2), summed in order of m.
template <typename Real>
__global__ void subcost_reduce_kernel(const Real *__restrict__ sub, Real *__restrict__ cost, int K,
                                      int Ms, int T) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)K * T) return;
  const int64_t k = i / T, t = i % T;
  Real acc = 0;
  for (int mm = 0; mm < Ms; ++mm) acc += sub[(k * Ms + mm) * T + t];
  cost[i] = acc / (Real)Ms;
}

hipError_t launch_subcost_reduce(int dtype, const void *sub, void *cost, int K, int Ms, int T,
                                 hipStream_t s) {
  const int64_t n = (int64_t)K * T;
  const unsigned nb = (unsigned)((n + 255) / 256);
  if (dtype == PI_F64)
    hipLaunchKernelGGL(subcost_reduce_kernel<double>, dim3(nb), dim3(256), 0, s,
                       (const double *)sub, (double *)cost, K, Ms, T);
  else
    hipLaunchKernelGGL(subcost_reduce_kernel<float>, dim3(nb), dim3(256), 0, s, (const float *)sub,
                       (float *)cost, K, Ms, T);
  return hipGetLastError();
}

// ------------------------------------------------------------- update
// Eq. (2) with the cost-to-go of Sec. 3.1, all sums in double:
//  (1) the cost-to-go at the segment boundaries, S_b[j][k] = sum of row k's costs
//      from step j seg_len on (only where (2) does not sum the rows itself);
//  (2) one wave per (chunk of rollouts, segment of steps) walks its steps
//      backwards with the cost-to-go of its rollouts in registers: the local
//      minimum m_c, Z_c = sum exp(-(S - m_c)/lambda), N_c = sum exp(...) eps_{k,i};
//  (3) one block per step merges the chunks (log-sum-exp shifts) and applies
//      u_i += N / Z.  If the weights P_{k,i} are asked for, (4) writes
//      them, walking the rows once more.
// (2) is bound by its arithmetic: per (rollout, step) ten Philox rounds, two
// Box-Muller pairs and one double exp.  (1) and (2) read the costs once each; S is
// not stored.  K = 65536, T = 200 in float: 176 us with S and separate passes over it,
// 98 us so (boundaries 12, partials 78 -- 230 vector instructions per pair --, merge 5).
constexpr int kUpdChunk = 2048;   // the workspace holds one partial per so many rollouts and step, and S
constexpr int kUpdSteps = 4, kUpdTiles = 2;   // steps and 64-rollout tiles per wave of stage 2
constexpr int kUpdSegLen = 8;     // steps between boundaries (a multiple of it for long rows)
constexpr int kUpdRows = 32;      // rows per block of stage 1
constexpr int kUpdMaxSeg = 64;    // boundaries per row
constexpr int kUpdQ = 2 + kMaxU;  // values per partial: m, Z, N
constexpr int kUpdMaxGrid = 1 << 20;   // blocks of stages 1 and 3 (a launch has fewer than 2^32 threads)

size_t update_ws_bytes(int K, int T) {
  const int C = (K + kUpdChunk - 1) / kUpdChunk;
  return align_up((size_t)K * T * 8, 256) + align_up((size_t)T * C * kUpdQ * 8, 256) +
         align_up((size_t)T * 2 * 8, 256);
}

// The weights W[t][k] = exp(-(S - m_t) / lambda) / Z_t of the merged minima and sums,
// S = sum_{t' >= t} cost[k][t'] (t = 0 for a trajectory's weight).  A block holds 64
// rollouts and splits the horizon into segments, one wave each: every lane
// sums its (rollout, segment), the segment totals meet in LDS, and each lane
// walks its segment backwards from the total of the later segments; the
// stores of a wave cover 64 consecutive rollouts.  Two ways to read the costs:
// each lane straight along its own row (every load of a wave touches 64 rows,
// but all of a lane's loads are in flight at once: best when the grid is
// small), or through a per-wave LDS tile in chunks of 16 steps (each load
// covers 16 consecutive steps of 4 rollouts: best when bandwidth matters).
constexpr int kWgtK = 64, kWgtChunk = 16;
template <typename Real, bool kStaged, int kSeg>
__global__ void __launch_bounds__(kWgtK * kSeg) update_weights_kernel(const Real *__restrict__ cost, int K, int T,
                                                                         double lambda, int weighting,
                                                                         const double *__restrict__ norm,
                                                                         double *__restrict__ W) {
  __shared__ double tile[kStaged ? kSeg : 1][kWgtK][kWgtChunk + 1];
  __shared__ double tot[kSeg][kWgtK];
  const int lane = threadIdx.x % kWgtK, seg = threadIdx.x / kWgtK;
  const int k0 = blockIdx.x * kWgtK, k = k0 + lane;
  const int lo = (int)((int64_t)seg * T / kSeg), hi = (int)((int64_t)(seg + 1) * T / kSeg);
  const Real *row = cost + (int64_t)min(k, K - 1) * T;
  double (*tl)[kWgtChunk + 1] = tile[kStaged ? seg : 0];
  // chunk [c0, c0 + w) of the segment into this wave's tile (rows past K read row K-1)
  auto load = [&](int c0, int w) {
    for (int e = lane; e < kWgtK * kWgtChunk; e += kWgtK) {
      const int r = e / kWgtChunk, c = e % kWgtChunk;
      if (c < w) tl[r][c] = (double)cost[(int64_t)min(k0 + r, K - 1) * T + c0 + c];
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
  };
  double sum = 0.0;
  if constexpr (kStaged) {
    for (int c0 = lo; c0 < hi; c0 += kWgtChunk) {
      const int w = min(kWgtChunk, hi - c0);
      load(c0, w);
      for (int c = 0; c < w; ++c) sum += tl[lane][c];
      __builtin_amdgcn_wave_barrier();
    }
  } else {
    for (int t = lo; t < hi; ++t) sum += (double)row[t];
  }
  tot[seg][lane] = sum;
  __syncthreads();
  double acc = 0.0;
  for (int j = kSeg - 1; j > seg; --j) acc += tot[j][lane];
  double whole = 0.0;
  for (int j = kSeg - 1; j >= 0; --j) whole += tot[j][lane];
  auto weight = [&](int t) {
    const double S = weighting == PI_W_TRAJECTORY ? whole : acc;
    W[(int64_t)t * K + k] = exp(-(S - norm[2 * t]) / lambda) / norm[2 * t + 1];
  };
  if constexpr (kStaged) {
    for (int c1 = hi; c1 > lo; c1 -= kWgtChunk) {
      const int c0 = max(lo, c1 - kWgtChunk), w = c1 - c0;
      load(c0, w);
      for (int c = w - 1; c >= 0; --c) {
        acc += tl[lane][c];
        if (k < K) weight(c0 + c);
      }
      __builtin_amdgcn_wave_barrier();
    }
  } else {
    if (k >= K) return;
    for (int t = hi - 1; t >= lo; --t) {
      acc += (double)row[t];
      weight(t);
    }
  }
}

// Four consecutive costs of a row as doubles; steps from te on read as 0.  vec: every
// row and the base are 16-byte aligned and T is a multiple of four.
template <typename Real>
__device__ __forceinline__ void load_cost4(const Real *__restrict__ row, int t, int te, bool vec, Real (&c)[4]) {
  if (vec) {
    if (t >= te) {
      c[0] = c[1] = c[2] = c[3] = (Real)0;
    } else if constexpr (sizeof(Real) == 4) {
      const float4 v = *(const float4 *)(row + t);
      c[0] = v.x, c[1] = v.y, c[2] = v.z, c[3] = v.w;
    } else {
      const double2 v = *(const double2 *)(row + t), w = *(const double2 *)(row + t + 2);
      c[0] = v.x, c[1] = v.y, c[2] = w.x, c[3] = w.y;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = t + i < te ? row[t + i] : (Real)0;
  }
}

// Stage 1: lanes take (row, segment) pairs in memory order, the segment sums meet
// in LDS, one lane per row walks them backwards, and the boundaries go out
// transposed, 32 rows at a time.  Bound by reading the costs.
// kLoop: more rows than kUpdMaxGrid blocks take.
template <typename Real, bool kLoop>
__global__ void __launch_bounds__(256) update_bound_kernel(const Real *__restrict__ cost, int K, int T, int seg_len,
                                                           int nseg, int vec, double *__restrict__ Sb) {
  __shared__ double tot[kUpdRows][kUpdMaxSeg + 1];
  // (k0 stays below 2^31 + 2^25)
  for (uint32_t k0 = blockIdx.x * kUpdRows; k0 < (uint32_t)K; k0 += gridDim.x * kUpdRows) {
    for (int e = threadIdx.x; e < kUpdRows * nseg; e += 256) {
      const int r = e / nseg, j = e - r * nseg;
      const Real *row = cost + (int64_t)min(k0 + r, (uint32_t)K - 1) * T;
      const int te = min(T, (j + 1) * seg_len);
      double sum = 0.0;
      for (int t = j * seg_len; t < te; t += 8) {
        Real a[4], b[4];
        load_cost4(row, t, te, vec, a);
        load_cost4(row, t + 4, te, vec, b);
        sum += (((double)a[0] + (double)a[1]) + ((double)a[2] + (double)a[3])) +
               (((double)b[0] + (double)b[1]) + ((double)b[2] + (double)b[3]));
      }
      tot[r][j] = sum;
    }
    __syncthreads();
    if (threadIdx.x < kUpdRows) {
      double acc = 0.0;
      for (int j = nseg - 1; j >= 0; --j) {
        acc += tot[threadIdx.x][j];
        tot[threadIdx.x][j] = acc;
      }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kUpdRows * nseg; e += 256) {
      const int r = e % kUpdRows, j = e / kUpdRows;
      if (k0 + r < (uint32_t)K) Sb[(int64_t)j * K + k0 + r] = tot[r][j];
    }
    if (!kLoop) return;
    __syncthreads();   // the sums have been read
  }
}

// Cross-lane sums of doubles.  fold32 / fold16 add lane pairs 32 / 16 apart of two
// values at once: a's sums end in the lower half-wave / even rows, b's in the upper / odd.
template <int STEP>
__device__ __forceinline__ void swap_rows(double &a, double &b) {
  const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
  uint32_t w[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t x = (uint32_t)(ua >> (32 * h)), y = (uint32_t)(ub >> (32 * h));
    if constexpr (STEP == 32) {
      auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
      w[h][0] = r[0], w[h][1] = r[1];
    } else {
      auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
      w[h][0] = r[0], w[h][1] = r[1];
    }
  }
  a = __longlong_as_double((long long)((uint64_t)w[0][0] | ((uint64_t)w[1][0] << 32)));
  b = __longlong_as_double((long long)((uint64_t)w[0][1] | ((uint64_t)w[1][1] << 32)));
}
template <int STEP>
__device__ __forceinline__ double fold_rows(double a, double b) {
  swap_rows<STEP>(a, b);
  return a + b;
}
__device__ __forceinline__ double row_sum(double v) {   // over 16 lanes, in every lane
  v += dpp<0x128>(v);
  v += dpp<0x124>(v);
  v += dpp<0x122>(v);
  return v + dpp<0x121>(v);
}
__device__ __forceinline__ double wave_min(double v) {
  v = fmin(v, dpp<0x128>(v));
  v = fmin(v, dpp<0x124>(v));
  v = fmin(v, dpp<0x122>(v));
  v = fmin(v, dpp<0x121>(v));
  double a = v, b = v;
  swap_rows<16>(a, b);
  v = fmin(a, b);
  a = b = v;
  swap_rows<32>(a, b);
  return fmin(a, b);
}
__device__ __forceinline__ double wave_sum(double v) {
  v = row_sum(v);
  v = fold_rows<16>(v, v);
  return fold_rows<32>(v, v);
}

// d / lambda with the quotient's rounding error corrected once (d >= 0, inv = 1/lambda;
// infinities and NaN pass through).
__device__ __forceinline__ double scaled(double d, double lambda, double inv) {
  const double q = d * inv, r = fma(-q, lambda, d);
  return fabs(r) < 1.0 / 0.0 ? fma(r, inv, q) : (d > 0.0 ? q : d);
}

// Stage 2.  A wave holds NT tiles of 64 rollouts and SEG steps; it sums the costs
// between its last step and the next boundary (nseg = 0: the row's end) itself.
// Partials go to part[step][q][chunk].  Rollouts past K weigh exp(-inf) = 0.
template <typename Real, int NU, int NT, int SEG>
__global__ void __launch_bounds__(256) update_part_kernel(ProbDev<Real> p, double lambda, double inv, int weighting,
                                                          const uint32_t *__restrict__ iter,
                                                          const Real *__restrict__ cost,
                                                          const double *__restrict__ Sb, int seg_len, int nseg,
                                                          int vec, int C, double *__restrict__ part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, K = p.K, T = p.T;
  // waves of a block: neighbouring segments of the same rows, or neighbouring chunks
  const int chunk = SEG > 1 ? blockIdx.x : blockIdx.x * 4 + wave;
  const int t0 = SEG > 1 ? (blockIdx.y * 4 + wave) * SEG : blockIdx.y;
  if (chunk >= C || t0 >= T) return;
  const bool whole = weighting == PI_W_TRAJECTORY;
  const uint32_t wc = stream_word(kTagCtrl, p.problem_id, *iter);
  const Real *row[NT];
  double acc[NT];
  bool in[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int64_t k = ((int64_t)chunk * NT + n) * 64 + lane;
    in[n] = k < K;
    const int64_t kc = in[n] ? k : K - 1;
    row[n] = cost + kc * T;
    acc[n] = 0.0;
    // the cost-to-go behind the wave's last step (of the whole row for a
    // trajectory's weight)
    int from = whole ? 0 : min(T, t0 + SEG), to = T;
    if (nseg > 0) {
      const int j = whole ? 0 : t0 / seg_len + 1;
      if (j < nseg) acc[n] = Sb[(int64_t)j * K + kc];
      to = whole ? 0 : min(T, j * seg_len);
    }
    for (int t = from; t < to; t += 4) {
      Real c[4];
      load_cost4(row[n], t, to, false, c);   // from need not be a multiple of four
      acc[n] += ((double)c[0] + (double)c[1]) + ((double)c[2] + (double)c[3]);
    }
  }
  constexpr int W = SEG > 1 ? 4 : 1;   // steps per load
#pragma unroll 1
  for (int h = SEG - W; h >= 0; h -= W) {
    if (t0 + h >= T) continue;
    Real c[NT][4];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      if (W > 1)
        load_cost4(row[n], t0 + h, T, vec, c[n]);
      else
        c[n][0] = row[n][t0];
    }
#pragma unroll
    for (int w = W - 1; w >= 0; --w) {
      const int i = t0 + h + w;
      if (i >= T) continue;
      double S[NT], mn = 1.0 / 0.0;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        if (!whole) acc[n] += (double)c[n][w];
        S[n] = in[n] ? acc[n] : 1.0 / 0.0;
        mn = fmin(mn, S[n]);
      }
      mn = wave_min(mn);
      // a chunk of infinite costs only: no weight, and no inf - inf
      const double base = mn < 1.0 / 0.0 ? mn : 0.0;
      double z = 0.0, N[NU];
#pragma unroll
      for (int a = 0; a < NU; ++a) N[a] = 0.0;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const double om = exp(-scaled(S[n] - base, lambda, inv));
        Real eps[4];
        normals<Real, NU>(p.key0, p.key1, wc, (uint32_t)((chunk * NT + n) * 64 + lane), 0u, (uint32_t)i, eps);
        z += om;
#pragma unroll
        for (int a = 0; a < NU; ++a) N[a] += om * (double)(p.noise_std[a] * eps[a]);
      }
      double *o = part + (int64_t)i * kUpdQ * C + chunk;
      if constexpr (NU == 2) {
        const double x = row_sum(fold_rows<16>(fold_rows<32>(N[0], N[1]), fold_rows<32>(z, z)));
        // rows: N0, z, N1, z
        if (lane == 0) o[0] = mn, o[2 * C] = x;
        if (lane == 16) o[C] = x;
        if (lane == 32) o[3 * C] = x;
      } else {
        const double x = row_sum(fold_rows<16>(fold_rows<32>(N[0], N[1]), fold_rows<32>(N[2], N[3])));
        z = wave_sum(z);
        // rows: N0, N2, N1, N3
        if (lane == 0) o[0] = mn, o[C] = z, o[2 * C] = x;
        if (lane == 16) o[4 * C] = x;
        if (lane == 32) o[3 * C] = x;
        if (lane == 48) o[5 * C] = x;
      }
    }
  }
}

// Stage 3, one block per step: every lane reads its chunks' partials at once, so the
// block waits for memory once; then minima and sums over the waves and through LDS.
// kLoop: more steps than kUpdMaxGrid.
template <typename Real, bool kLoop>
__global__ void __launch_bounds__(256) update_apply_kernel(int T, int C, int n_u, double lambda,
                                                           const double *__restrict__ part,
                                                           Real *__restrict__ u_nom, double *__restrict__ norm,
                                                           uint32_t *__restrict__ iter) {
  __shared__ double wmin[4], wsum[4][1 + kMaxU];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the iteration's draws have all been consumed: advance the iteration word
  if (blockIdx.x == 0 && threadIdx.x == 0) *iter += 1u;
  for (uint32_t i = blockIdx.x; i < (uint32_t)T; i += gridDim.x) {
    const double *pi_ = part + (int64_t)i * kUpdQ * C;
    double m = 1.0 / 0.0, v[1 + kMaxU] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int c = threadIdx.x; c < C; c += 256) {
      const double mc = pi_[c], mn = fmin(m, mc);
      const double f = m == mn ? 1.0 : exp(-(m - mn) / lambda), fc = mc == mn ? 1.0 : exp(-(mc - mn) / lambda);
#pragma unroll
      for (int q = 0; q <= kMaxU; ++q)
        if (q <= n_u) v[q] = v[q] * f + pi_[(int64_t)(1 + q) * C + c] * fc;
      m = mn;
    }
    const double wm = wave_min(m);
    if (lane == 0) wmin[wave] = wm;
    __syncthreads();
    const double mn = fmin(fmin(wmin[0], wmin[1]), fmin(wmin[2], wmin[3]));
    const double f = m == mn ? 1.0 : exp(-(m - mn) / lambda);
#pragma unroll
    for (int q = 0; q <= kMaxU; ++q) {
      const double w = q <= n_u ? wave_sum(v[q] * f) : 0.0;
      if (lane == 0) wsum[wave][q] = w;
    }
    __syncthreads();
    auto total = [&](int q) { return (wsum[0][q] + wsum[1][q]) + (wsum[2][q] + wsum[3][q]); };
    const int a = threadIdx.x;
    if (a < n_u) u_nom[(int64_t)i * n_u + a] = (Real)((double)u_nom[(int64_t)i * n_u + a] + total(1 + a) / total(0));
    if (a == 0) {
      norm[2 * (int64_t)i] = mn;
      norm[2 * (int64_t)i + 1] = total(0);
    }
    if (!kLoop) return;
    __syncthreads();   // the sums have been read
  }
}

template <typename Real, int NU>
static void update_part(const ProbDev<Real> &p, const Real *cost, const uint32_t *iter, double *ws, double **part,
                        int *nchunk, double lambda, int weighting, hipStream_t s) {
  const int K = p.K, T = p.T;
  const double inv = 1.0 / lambda;
  // Up to 12 (tile, step) pairs per compute unit (of 256), every wave takes one: at
  // 2048 x 50 in float 12.8 us against 16.6 with tiles and steps grouped, at 4096 x 100
  // 19.3 against 16.9.  Rows of up to 40 steps are then summed by the waves themselves,
  // which spares a launch: 3000 x 20 9.9 us against 11.1, 1000 x 50 13.2 against 11.9.
  // So are rows of one segment at any K, as S_b and the partials need the place of
  // more than that many steps of S.
  const bool single = (int64_t)((K + 63) / 64) * T <= 3072, direct = T <= kUpdSegLen || (single && T <= 40);
  const int nt = direct || single ? 1 : kUpdTiles, C = (K + 64 * nt - 1) / (64 * nt);
  *nchunk = C;
  if (direct) {
    *part = ws;
    hipLaunchKernelGGL((update_part_kernel<Real, NU, 1, 1>), dim3((C + 3) / 4, T), dim3(256), 0, s, p, lambda, inv,
                       weighting, iter, cost, (const double *)nullptr, 0, 0, 0, C, ws);
    return;
  }
  const int seg_len = kUpdSegLen * ((T + kUpdSegLen * kUpdMaxSeg - 1) / (kUpdSegLen * kUpdMaxSeg));
  const int nseg = (T + seg_len - 1) / seg_len;
  const int vec = T % 4 == 0 && (uintptr_t)cost % 16 == 0;
  *part = (double *)((char *)ws + align_up((size_t)K * nseg * 8, 256));
  const int nb = (K - 1) / kUpdRows + 1;
  if (nb > kUpdMaxGrid)
    hipLaunchKernelGGL((update_bound_kernel<Real, true>), dim3(kUpdMaxGrid), dim3(256), 0, s, cost, K, T, seg_len, nseg,
                       vec, ws);
  else
    hipLaunchKernelGGL((update_bound_kernel<Real, false>), dim3(nb), dim3(256), 0, s, cost, K, T, seg_len, nseg, vec, ws);
  if (single)
    hipLaunchKernelGGL((update_part_kernel<Real, NU, 1, 1>), dim3((C + 3) / 4, T), dim3(256), 0, s, p, lambda, inv,
                       weighting, iter, cost, (const double *)ws, seg_len, nseg, vec, C, *part);
  else
    hipLaunchKernelGGL((update_part_kernel<Real, NU, kUpdTiles, kUpdSteps>),
                       dim3(C, (T + 4 * kUpdSteps - 1) / (4 * kUpdSteps)), dim3(256), 0, s, p, lambda, inv, weighting,
                       iter, cost, (const double *)ws, seg_len, nseg, vec, C, *part);
}

template <typename Real>
static hipError_t update_t(const ProbDev<Real> &p, const Real *cost, const uint32_t *iter,
                           Real *u_nom, double *W, void *ws, double lambda, int weighting,
                           hipStream_t s) {
  const int K = p.K, T = p.T;
  double *part;
  double *norm = (double *)((char *)ws + update_ws_bytes(K, T) - align_up((size_t)T * 2 * 8, 256));
  int C;
  if (p.n_u <= 2)
    update_part<Real, 2>(p, cost, iter, (double *)ws, &part, &C, lambda, weighting, s);
  else
    update_part<Real, 4>(p, cost, iter, (double *)ws, &part, &C, lambda, weighting, s);
  if (T > kUpdMaxGrid)
    hipLaunchKernelGGL((update_apply_kernel<Real, true>), dim3(kUpdMaxGrid), dim3(256), 0, s, T, C, p.n_u, lambda,
                       (const double *)part, u_nom, norm, const_cast<uint32_t *>(iter));
  else
    hipLaunchKernelGGL((update_apply_kernel<Real, false>), dim3(T), dim3(256), 0, s, T, C, p.n_u, lambda,
                       (const double *)part, u_nom, norm, const_cast<uint32_t *>(iter));
  if (W) {
    const unsigned nb = (unsigned)((K + kWgtK - 1) / kWgtK);
    if (nb >= 256)   // enough blocks to cover the compute units: read through LDS
      hipLaunchKernelGGL((update_weights_kernel<Real, true, 4>), dim3(nb), dim3(kWgtK * 4), 0, s, cost, K, T, lambda,
                         weighting, (const double *)norm, W);
    else             // more waves per block instead
      hipLaunchKernelGGL((update_weights_kernel<Real, false, 16>), dim3(nb), dim3(kWgtK * 16), 0, s, cost, K, T,
                         lambda, weighting, (const double *)norm, W);
  }
  return hipGetLastError();
}

hipError_t launch_update(int dtype, const void *pargs, const void *cost, const uint32_t *iter,
                         void *u_nom, double *weights, void *ws, int, double lambda, int weighting,
                         hipStream_t s) {
  if (dtype == PI_F64)
    return update_t<double>(*(const ProbDev<double> *)pargs, (const double *)cost, iter,
                            (double *)u_nom, weights, ws, lambda, weighting, s);
  return update_t<float>(*(const ProbDev<float> *)pargs, (const float *)cost, iter, (float *)u_nom,
                         weights, ws, lambda, weighting, s);
}

// ------------------------------------------------------------ RH shift
// The plant step executes u_nom[0] under the PLANT stream.  Kernel 1: block
// (o, c) evaluates 64 local models of output o at z = [x0 ; u_nom[0]], one per
// lane, and merges them into one partial statistic (fixed tree order).
// Kernel 2 (one block, a lane per output): merges the partials of every output in order,
// samples the accelerations, steps Euler and shifts the plan left by one step (last
// control repeated).  The iteration word is read, not advanced.
constexpr int kShiftThreads = 64;

size_t shift_partial_bytes(const ModelArgs &m, int dtype) {
  int Lmax = 1;
  for (int o = 0; o < m.n_out; ++o) Lmax = max(Lmax, m.L_off[o + 1] - m.L_off[o]);
  const int C = (Lmax + kShiftThreads - 1) / kShiftThreads;
  return align_up((size_t)m.n_out * C * 5 * (dtype == PI_F64 ? 8 : 4), 256);
}

template <typename Real, int DYN>
__global__ void __launch_bounds__(kShiftThreads) plant_partial_kernel(ModelArgs m,
                                                                      const Real *__restrict__ rec,
                                                                      const Real *__restrict__ x0,
                                                                      const Real *__restrict__ u_nom,
                                                                      MixStat<Real> *__restrict__ part) {
  using DD = DynDims<DYN>;
  constexpr int D = DD::D, NX = DD::NX, NU = DD::NU;
  constexpr int RS = rec_stride<Real, D>();
  __shared__ MixStat<Real> red[kShiftThreads];
  const int o = blockIdx.y, c = blockIdx.x, C = gridDim.x;
  Real z[D], x[NX], u[NU];
#pragma unroll
  for (int a = 0; a < NX; ++a) x[a] = x0[a];
#pragma unroll
  for (int a = 0; a < NU; ++a) u[a] = u_nom[a];
  lwpr_input<DYN>(x, u, z);
  MixStat<Real> st = mix_empty<Real>();
  const int j = m.L_off[o] + c * kShiftThreads + threadIdx.x;
  if (j < m.L_off[o + 1]) {
    Real q, y;
    eval_record<Real, D>(rec + (size_t)j * RS, z, q, y);
    mix_add<false>(st, (Real)-0.5 * q, y, rec[(size_t)j * RS + RS - 1]);
  }
  red[threadIdx.x] = st;
  __syncthreads();
  for (int w = kShiftThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = mix_merge<false>(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[o * C + c] = red[0];
}

// The rest of the shift by one block, behind a barrier after `part`: a lane per output
// merges its partials in order and samples its acceleration, one lane steps Euler, all
// shift the plan.  acc, xnew: LDS.
template <typename Real, int DYN>
__device__ __forceinline__ void plant_finish(const ProbDev<Real> &p, int C, const MixStat<Real> *part,
                                             Real *__restrict__ x0, Real *__restrict__ u_nom,
                                             const uint32_t *__restrict__ iter, Real *acc, Real *xnew) {
  using DD = DynDims<DYN>;
  constexpr int NX = DD::NX, NU = DD::NU, NO = DD::NO;
  if ((int)threadIdx.x < NO) {
    const int o = threadIdx.x;
    Real xi[8], xo = 0, mu, v;
    normals<Real, NO>(p.key0, p.key1, stream_word(kTagPlant, p.problem_id, *iter), 0u, 0u, 0u, xi);
#pragma unroll
    for (int i = 0; i < NO; ++i) xo = i == o ? xi[i] : xo;
    MixStat<Real> st = part[o * C];
    for (int c = 1; c < C; ++c) st = mix_merge<false>(st, part[o * C + c]);
    mix_finish(st, &mu, &v);
    acc[o] = mu + sqrt_(v) * xo;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    Real x[NX], u[NU], ac[NO], xn[NX];
    for (int a = 0; a < NX; ++a) x[a] = x0[a];
    for (int a = 0; a < NU; ++a) u[a] = u_nom[a];
    for (int o = 0; o < NO; ++o) ac[o] = acc[o];
    euler_step<Real>(DYN, p.dt, x, ac, u, xn);
    for (int a = 0; a < NX; ++a) xnew[a] = xn[a];
  }
  __syncthreads();
  // Shift left by one control in place.  Chunk by chunk every lane reads its
  // new value before any lane writes; a chunk only reads indices at or above
  // its own start, which no earlier chunk has written.
  const int n = p.T * NU;
  for (int base = 0; base < n; base += blockDim.x) {
    const int i = base + threadIdx.x;
    Real v = 0;
    if (i < n) v = (i + NU < n) ? u_nom[i + NU] : u_nom[i];
    __syncthreads();
    if (i < n) u_nom[i] = v;
    __syncthreads();
  }
  if (threadIdx.x < NX) x0[threadIdx.x] = xnew[threadIdx.x];
}

template <typename Real, int DYN>
__global__ void __launch_bounds__(1024) plant_apply_kernel(ProbDev<Real> p, int C,
                                                           const MixStat<Real> *__restrict__ part,
                                                           Real *__restrict__ x0, Real *__restrict__ u_nom,
                                                           const uint32_t *__restrict__ iter) {
  __shared__ Real acc[kMaxOut], xnew[kMaxX];
  plant_finish<Real, DYN>(p, C, part, x0, u_nom, iter, acc, xnew);
}

// Both kernels in one block, a wave per (output, chunk), where there are at most
// kPlantWaves of these: the same sums in the same order, one launch less (control
// step of 256 x 20 point-mass rollouts in double 54.3 -> 52.5 us).
constexpr int kPlantWaves = 8;
template <typename Real, int DYN>
__global__ void __launch_bounds__(kPlantWaves * 64) plant_small_kernel(ProbDev<Real> p, ModelArgs m, int C,
                                                                      const Real *__restrict__ rec,
                                                                      Real *__restrict__ x0,
                                                                      Real *__restrict__ u_nom,
                                                                      const uint32_t *__restrict__ iter) {
  using DD = DynDims<DYN>;
  constexpr int D = DD::D, NX = DD::NX, NU = DD::NU, NO = DD::NO;
  constexpr int RS = rec_stride<Real, D>();
  __shared__ MixStat<Real> part[kPlantWaves];
  __shared__ Real acc[kMaxOut], xnew[kMaxX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave < NO * C) {
    const int o = wave / C, c = wave - o * C;
    Real z[D], x[NX], u[NU];
#pragma unroll
    for (int a = 0; a < NX; ++a) x[a] = x0[a];
#pragma unroll
    for (int a = 0; a < NU; ++a) u[a] = u_nom[a];
    lwpr_input<DYN>(x, u, z);
    MixStat<Real> st = mix_empty<Real>();
    const int j = m.L_off[o] + c * kShiftThreads + lane;
    if (j < m.L_off[o + 1]) {
      Real q, y;
      eval_record<Real, D>(rec + (size_t)j * RS, z, q, y);
      mix_add<false>(st, (Real)-0.5 * q, y, rec[(size_t)j * RS + RS - 1]);
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) st = mix_merge<false>(st, shfl_stat(st, w));
    if (lane == 0) part[wave] = st;
  }
  __syncthreads();
  plant_finish<Real, DYN>(p, C, part, x0, u_nom, iter, acc, xnew);
}

template <typename Real>
static hipError_t rh_shift_t(const ProbDev<Real> &p, const ModelArgs &m, const void *rec, void *part,
                             void *x0, void *u_nom, const uint32_t *iter, hipStream_t s) {
  int Lmax = 1;
  for (int o = 0; o < m.n_out; ++o) Lmax = max(Lmax, m.L_off[o + 1] - m.L_off[o]);
  const int C = (Lmax + kShiftThreads - 1) / kShiftThreads;
  if (C * m.n_out <= kPlantWaves) {
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(1), dim3(kPlantWaves * 64), 0, s, p, m, C, (const Real *)rec, (Real *)x0,
                         (Real *)u_nom, iter);
    };
    if (p.dyn == kDynPointMass2D)
      go(plant_small_kernel<Real, kDynPointMass2D>);
    else if (p.dyn == kDynQuadHybrid)
      go(plant_small_kernel<Real, kDynQuadHybrid>);
    else
      go(plant_small_kernel<Real, kDynQuad12>);
    return hipGetLastError();
  }
  const dim3 grid(C, m.n_out);
  const int apply = p.T * p.n_u > 256 ? 1024 : 256;   // the plan's shift in one pass, mostly
  if (p.dyn == kDynPointMass2D) {
    hipLaunchKernelGGL((plant_partial_kernel<Real, kDynPointMass2D>), grid, dim3(kShiftThreads), 0, s, m,
                       (const Real *)rec, (const Real *)x0, (const Real *)u_nom, (MixStat<Real> *)part);
    hipLaunchKernelGGL((plant_apply_kernel<Real, kDynPointMass2D>), dim3(1), dim3(apply), 0, s, p, C,
                       (const MixStat<Real> *)part, (Real *)x0, (Real *)u_nom, iter);
  } else if (p.dyn == kDynQuadHybrid) {
    hipLaunchKernelGGL((plant_partial_kernel<Real, kDynQuadHybrid>), grid, dim3(kShiftThreads), 0, s, m,
                       (const Real *)rec, (const Real *)x0, (const Real *)u_nom, (MixStat<Real> *)part);
    hipLaunchKernelGGL((plant_apply_kernel<Real, kDynQuadHybrid>), dim3(1), dim3(apply), 0, s, p, C,
                       (const MixStat<Real> *)part, (Real *)x0, (Real *)u_nom, iter);
  } else {
    hipLaunchKernelGGL((plant_partial_kernel<Real, kDynQuad12>), grid, dim3(kShiftThreads), 0, s, m,
                       (const Real *)rec, (const Real *)x0, (const Real *)u_nom, (MixStat<Real> *)part);
    hipLaunchKernelGGL((plant_apply_kernel<Real, kDynQuad12>), dim3(1), dim3(apply), 0, s, p, C,
                       (const MixStat<Real> *)part, (Real *)x0, (Real *)u_nom, iter);
  }
  return hipGetLastError();
}

hipError_t launch_rh_shift(int dtype, const void *pargs, const ModelArgs &m, const void *rec,
                           void *part, void *x0, void *u_nom, const uint32_t *iter, hipStream_t s) {
  return dtype == PI_F64
             ? rh_shift_t<double>(*(const ProbDev<double> *)pargs, m, rec, part, x0, u_nom, iter, s)
             : rh_shift_t<float>(*(const ProbDev<float> *)pargs, m, rec, part, x0, u_nom, iter, s);
}

// Clears one counter with a kernel (graph-capture friendly, no memset node).
__global__ void zero_int_kernel(int *p) { *p = 0; }
__global__ void zero_u32_kernel(uint32_t *p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}
hipError_t launch_zero_u32(uint32_t *p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = std::min<int64_t>((n + 255) / 256, 1024);
  hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)nb), dim3(256), 0, s, p, n);
  return hipGetLastError();
}
hipError_t launch_zero_int(int *p, hipStream_t s) {
  hipLaunchKernelGGL(zero_int_kernel, dim3(1), dim3(1), 0, s, p);
  return hipGetLastError();
}

// ------------------------------------------------------ stream access
__global__ void philox_kernel(const uint32_t *__restrict__ ctr, uint32_t k0, uint32_t k1,
                              uint32_t *__restrict__ out, int64_t N) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const Philox4 r = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1);
  for (int q = 0; q < 4; ++q) out[4 * i + q] = r.v[q];
}

hipError_t launch_philox(const uint32_t *ctr, uint32_t k0, uint32_t k1, uint32_t *out, int64_t N,
                         hipStream_t s) {
  if (N == 0) return hipSuccess;
  hipLaunchKernelGGL(philox_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, ctr, k0, k1,
                     out, N);
  return hipGetLastError();
}

// One lane per (k, t): the same normals<> calls as the rollout, update and
// shift kernels.
template <typename Real>
__global__ void noise_kernel(ProbDev<Real> p, int tag, const uint32_t *__restrict__ iter, int k0,
                             int nk, int m, Real *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t word = stream_word((uint32_t)tag, p.problem_id, *iter);
  Real v[8];
  if (tag == kTagPlant) {
    if (i != 0) return;
    normals_n<Real>(p.n_out, p.key0, p.key1, word, 0u, 0u, 0u, v);
    for (int o = 0; o < p.n_out; ++o) out[o] = v[o];
    return;
  }
  if (i >= (int64_t)nk * p.T) return;
  const uint32_t k = (uint32_t)(k0 + i / p.T), t = (uint32_t)(i % p.T);
  if (tag == kTagCtrl) {
    normals_n<Real>(p.n_u, p.key0, p.key1, word, k, 0u, t, v);
    for (int a = 0; a < p.n_u; ++a) out[i * p.n_u + a] = p.noise_std[a] * v[a];
  } else {
    normals_n<Real>(p.n_out, p.key0, p.key1, word, k, (uint32_t)m, t, v);
    for (int o = 0; o < p.n_out; ++o) out[i * p.n_out + o] = v[o];
  }
}

hipError_t launch_noise(int dtype, const void *pargs, int tag, const uint32_t *iter, int k0, int nk,
                        int m, void *out, hipStream_t s) {
  const int T = dtype == PI_F64 ? ((const ProbDev<double> *)pargs)->T : ((const ProbDev<float> *)pargs)->T;
  const int64_t n = tag == kTagPlant ? 1 : (int64_t)nk * T;
  if (n == 0) return hipSuccess;
  const unsigned nb = (unsigned)((n + 255) / 256);
  if (dtype == PI_F64)
    hipLaunchKernelGGL(noise_kernel<double>, dim3(nb), dim3(256), 0, s,
                       *(const ProbDev<double> *)pargs, tag, iter, k0, nk, m, (double *)out);
  else
    hipLaunchKernelGGL(noise_kernel<float>, dim3(nb), dim3(256), 0, s, *(const ProbDev<float> *)pargs,
                       tag, iter, k0, nk, m, (float *)out);
  return hipGetLastError();
}

}  // namespace pi2rh
