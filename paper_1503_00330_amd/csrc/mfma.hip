// FP32 matrix-core kernels for gfx950 (v_mfma_f32_16x16x4f32).
//
// The kernel distance of Eq. (1) is recast as a dense contraction: with
// Phi(z) = [z_a z_b (a <= b), z, 1] the activation of model j is
//   alpha * q_j = Phi(z) . w_j,   w_j = alpha [theta_j, -(D_j + D_j^T) c_j, c_j^T D_j c_j],
// alpha = -log2(e)/2, and the local prediction is y_j = [z, 1] . [b_j, beta0_j - b_j.c_j].
// A workgroup owns 16*MT samples (staged in LDS as lane-major fragments); its
// NW waves split the model tiles (16 models, streamed from L2 as 1 KB
// coalesced loads).  In the rollout contraction the model tile is the A
// operand and the samples' features the B operand (both have the same
// register layout), so each lane ends with four models of one sample.
//
// Anchored accumulation.  Every (sample, output) carries an anchor m (an
// activation close to the largest one) and a reference mean r, both taken
// from the previous step and fed through one extra feature of each
// contraction, so the matrix core returns a' = a - m and d = y - r directly.
// Per model a lane then only accumulates
//   Z += 2^a', S1 += 2^a' d, S2 += 2^a' d^2, S3 += 2^a' sigma^2, mx = max(mx, a'),
// and the normalised mixture of Eq. (1) is
//   mu = r + S1/Z,  var = (max(S2 - S1^2/Z, 0) + S3)/Z;
// the spread term is non-negative in exact arithmetic, and the clamp keeps its
// rounding (FP32 cancellation when the models' predictions differ widely) from
// turning the variance negative.
// Partial sums merge within a lane (its four models), across the four lane
// groups (two cross-lane shuffles) and across waves (LDS) as plain sums in a
// fixed order.  The sums are exact up to rounding whatever
// the anchor, as long as none of them overflowed and the largest term kept
// full precision; so the step is evaluated again, with the anchor moved to the
// observed maximum, only if a sum is not finite or the largest shifted
// activation fell below -100 (its term near the denormal range).  The first
// step always takes this second pass so its reference mean is the first
// pass's mean.
// (PI^2-RH with LWPR dynamics, arXiv:1503.00330.)
#include <stdlib.h>

#include <algorithm>
#include <type_traits>

#include "internal.hpp"

namespace pi2rh {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

template <int D>
struct Geo {
  static constexpr int NP = D * (D + 1) / 2;
  static constexpr int KQ = NP + D + 2;
  static constexpr int KQB = (KQ + 3) / 4;
  static constexpr int KY = D + 2;
  static constexpr int KYB = (KY + 3) / 4;
  static constexpr int KB = KQB + KYB;
  static constexpr int KB4 = (KB + 3) / 4;
  static constexpr int FQS = NP + D + 1;         // activation anchor feature
  static constexpr int FYS = 4 * KQB + D + 1;    // prediction reference feature
  static constexpr int NE = KB4 * 256;           // fragment floats per row tile
};

// alpha = -log2(e) / 2
constexpr double kAlpha = -0.72134752044448170368;
constexpr float kPadAct = -1.0e30f;
constexpr float kAnchorLo = -100.0f;
// Word 3 of a raw (untyped) buffer descriptor: 32-bit data format, no swizzle.
constexpr int kBufferWord3 = 0x00020000;

// Model-tile reads through buffer descriptors over the whole array: the tile's
// offset is a scalar and the lane's a fixed register, so no vector
// instruction goes into addressing.  The hardware range check covers only the
// lane's offset, so callers keep tile indices in range themselves (the
// prefetches clamp them).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void *base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, bytes, kBufferWord3);
}
__device__ __forceinline__ f32x4 buffer_f32x4(__amdgpu_buffer_rsrc_t r, int lane_off, int tile_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, tile_off, 0));
}
__device__ __forceinline__ float buffer_f32(__amdgpu_buffer_rsrc_t r, int lane_off, int tile_off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, lane_off, tile_off, 0));
}

// Three bf16 pieces hi + mid + lo of a float32 value, each rounded to nearest
// (ties to even) from the remainder of the previous ones: hi holds the top 8
// significand bits, mid the next 8, lo the rest exactly, so the pieces sum to
// the value exactly (for values whose pieces stay above the float32 normal
// range).  Products of two such values, summed over the six piece pairs whose
// weight is at least 2^-24 (hi hi, hi mid, mid hi, hi lo, mid mid, lo hi),
// reproduce the float32 product to within float32 rounding.  The conversion
// instruction keeps a NaN a NaN (adding half a unit to the bits would carry a
// mantissa of ones into the sign and leave a zero).
__device__ __forceinline__ void bf16_split3(float v, uint16_t *pc) {
  const __bf16 h = (__bf16)v;
  const float r1 = v - (float)h;
  const __bf16 m = (__bf16)r1;
  const __bf16 l = (__bf16)(r1 - (float)m);
  pc[0] = __builtin_bit_cast(uint16_t, h);
  pc[1] = __builtin_bit_cast(uint16_t, m);
  pc[2] = __builtin_bit_cast(uint16_t, l);
}

// Two fp16 pieces hi + lo of a float32 value of magnitude below 2^15, each
// rounded to nearest (ties to even): hi holds the top 11 significand bits, lo
// the next 11 (lo may be subnormal: the matrix cores keep fp16 subnormal
// inputs, so its absolute precision stays 2^-24).  The three piece products
// hi hi, hi lo, lo hi of two such values give the float32 product to about
// 2^-22 relative (lo lo, below 2^-22, is left out).
__device__ __forceinline__ void f16_split2(float v, uint16_t *pc) {
  const _Float16 h = (_Float16)v;
  const _Float16 l = (_Float16)(v - (float)h);
  pc[0] = __builtin_bit_cast(uint16_t, h);
  pc[1] = __builtin_bit_cast(uint16_t, l);
}

// ----------------------------------------------------------------- fold
// One block per tile of 16 model slots.  Phase 1: 16 lanes per model (one input
// coordinate each) compute in double the derived vectors (h = -(D + D^T) c,
// kappa = c^T D c, the folded PLS map b and y0 = beta0 - b.c); phase 2: the float32
// feature values of every slot go into LDS once; phase 3: every lane writes
// whole 16-byte fragments of each form, coalesced.  Bound by latency (a block
// reads 21 KB and writes 42 KB at d = 16): 96 tiles 114 us with one lane per
// model and every value recomputed for every form, 16 us so.
constexpr int kFoldThreads = 256;
static_assert(kFoldThreads >= kHfMeta, "one fold thread per per-tile value of the fp16 form");
constexpr int kFoldVals = kMaxD * (kMaxD + 1) / 2 + kMaxD + 2 + kMaxD + 2;   // quadratic-form, then prediction features

// Sum (or maximum) over the 16 lanes of a model, in every lane.
template <typename T, class Op>
__device__ __forceinline__ T fold_reduce(T v, Op op) {
#pragma unroll
  for (int m = 8; m >= 1; m >>= 1) v = op(v, __shfl_xor(v, m));
  return v;
}

__global__ void __launch_bounds__(kFoldThreads) fold_mfma_kernel(ModelArgs m, MfmaLayout l,
                                                                 float *__restrict__ W,
                                                                 float *__restrict__ sig2,
                                                                 uint32_t *__restrict__ Wb,
                                                                 uint32_t *__restrict__ Wh,
                                                                 float *__restrict__ hmeta) {
  __shared__ float Dl[16][kMaxD * kMaxD + 1];
  __shared__ double cs[16][kMaxD];
  __shared__ float val[16][kFoldVals + 1];
  __shared__ unsigned char pa[kMaxD * (kMaxD + 1) / 2], pb[kMaxD * (kMaxD + 1) / 2];
  __shared__ int eq[16], ey[16], big[16];
  const int tile = blockIdx.x, d = m.d, R = m.R, tid = threadIdx.x;
  const MfmaGeom g = MfmaGeom::make(d);
  int o = 0;
  while (o + 1 < m.n_out && tile >= l.tile_off[o + 1]) ++o;
  const int jfirst = m.L_off[o] + (tile - l.tile_off[o]) * 16;
  const int nvalid = min(16, m.L_off[o + 1] - jfirst);
  // the metrics and centres of the tile's models, and the feature pairs
  for (int e = tid; e < nvalid * d * d; e += kFoldThreads)
    Dl[e / (d * d)][e % (d * d)] = ((const float *)m.metric)[(size_t)jfirst * d * d + e];
  for (int e = tid; e < nvalid * d; e += kFoldThreads)
    cs[e / d][e % d] = (double)((const float *)m.centre)[(size_t)jfirst * d + e];
  if (tid < g.NP) {
    int a = 0, rem = tid;
    while (rem >= d - a) {
      rem -= d - a;
      ++a;
    }
    pa[tid] = (unsigned char)a;
    pb[tid] = (unsigned char)(a + rem);
  }
  const int col = tid >> 4, a = tid & 15;
  const bool valid = col < nvalid, on = valid && a < d;
  const size_t j = (size_t)jfirst + (valid ? col : 0);
  float ru[kMaxR], rp[kMaxR], rbeta[kMaxR];
  {
    const float *U = (const float *)m.proj_u + j * R * d;
    const float *P = m.proj_p ? (const float *)m.proj_p + j * R * d : U;
    const float *B = (const float *)m.beta + j * (R + 1);
#pragma unroll
    for (int r = 0; r < kMaxR; ++r) {
      const bool use = r < R && on;
      ru[r] = use ? U[r * d + a] : 0.0f;
      rp[r] = use ? P[r * d + a] : 0.0f;
      rbeta[r] = r < R && valid ? B[r + 1] : 0.0f;
    }
  }
  const float beta0 = valid ? ((const float *)m.beta)[j * (R + 1)] : 0.0f;
  const float s2 = valid ? ((const float *)m.sigma2)[j] : 0.0f;
  __syncthreads();
  auto add = [](double x, double y) { return x + y; };
  double h = 0.0, kap = 0.0;
  const double ca = on ? cs[col][a] : 0.0;
  if (on)
    for (int b = 0; b < d; ++b) {
      const double cb = cs[col][b], Dab = (double)Dl[col][a * d + b];
      h += (Dab + (double)Dl[col][b * d + a]) * cb;
      kap += ca * Dab * cb;
    }
  const double kappa = fold_reduce(kap, add);
  // y = beta0 + b.(z - c): b by reverse accumulation through the deflation chain
  double rb = 0.0;
#pragma unroll
  for (int r = kMaxR - 1; r >= 0; --r) {
    if (r >= R) continue;
    const double pr = fold_reduce((double)rp[r] * rb, add);
    // lanes without a coordinate stay 0: an infinite coefficient times 0 is not
    rb += on ? ((double)rbeta[r] - pr) * (double)ru[r] : 0.0;
  }
  const double y0 = (double)beta0 - fold_reduce(rb * ca, add);
  // padded slots: activation kPadAct, everything else 0
  if (a < d) {
    val[col][g.NP + a] = on ? (float)(kAlpha * -h) : 0.0f;
    val[col][g.KQ + a] = on ? (float)rb : 0.0f;
  }
  if (a == 0) {
    val[col][g.NP + d] = valid ? (float)(kAlpha * kappa) : kPadAct;
    val[col][g.NP + d + 1] = 1.0f;
    val[col][g.KQ + d] = valid ? (float)y0 : 0.0f;
    val[col][g.KQ + d + 1] = 1.0f;
    sig2[tile * 16 + col] = s2;
  }
  for (int f = a; f < g.NP; f += 16) {
    const int x = pa[f], y = pb[f];
    const double th = x == y ? (double)Dl[col][x * d + x] : (double)Dl[col][x * d + y] + (double)Dl[col][y * d + x];
    val[col][f] = valid ? (float)(kAlpha * th) : 0.0f;
  }
  __syncthreads();
  // float32 fragments: feature f of the contraction is quadratic-form feature f,
  // or from 4 KQB on prediction feature f - 4 KQB
  float4 *dst = (float4 *)(W + (size_t)tile * g.KB4 * 256);
  for (int e = tid; e < g.KB4 * 64; e += kFoldThreads) {
    const int lane = e & 63, kb4 = e >> 6;
    float v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int f = 4 * (4 * kb4 + c) + lane / 16, fy = f - 4 * g.KQB;
      v[c] = f < g.KQ ? val[lane & 15][f] : fy >= 0 && fy < g.KY ? val[lane & 15][g.KQ + fy] : 0.0f;
    }
    dst[e] = make_float4(v[0], v[1], v[2], v[3]);
  }
  if (Wb == nullptr) return;
  // the value of piece-form feature k of block kb: blocks 0 .. kBfNKQ-1 hold the
  // quadratic-form features, the last the prediction features
  auto piece_value = [&](int kb, int k, int slot) {
    return kb < kBfNKQ ? (k < g.KQ ? val[slot][k] : 0.0f) : (k < g.KY ? val[slot][g.KQ + k] : 0.0f);
  };
  // the same values as three bf16 pieces, in the A-operand layout of the bf16
  // 16x16x32 instruction: block kb, piece p, lane (model lane%16, features
  // 8 (lane/16) .. +7 of the block)
  u32x4 *dstb = (u32x4 *)(Wb + (size_t)tile * kBfTileU32);
  for (int e = tid; e < kBfNKB * 64; e += kFoldThreads) {
    const int lane = e & 63, kb = e >> 6, k0 = 32 * (kb < kBfNKQ ? kb : 0) + 8 * (lane / 16);
    uint16_t pc[8][3];
#pragma unroll
    for (int i = 0; i < 8; ++i) bf16_split3(piece_value(kb, k0 + i, lane & 15), pc[i]);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      u32x4 w;
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = (uint32_t)pc[2 * i][p] | ((uint32_t)pc[2 * i + 1][p] << 16);
      dstb[(kb * 3 + p) * 64 + lane] = w;
    }
  }
  if (Wh == nullptr) return;
  // the two-piece fp16 form: each model's quadratic-form values and its
  // prediction values, then split into hi + lo fp16 pieces.  A set whose
  // largest magnitude m is 2^-2 <= m < 2^14 is taken as it is (the pieces of
  // m then hold 22 bits, and every smaller value of the set is kept to
  // within 2^-25 absolute, 2^-23 of m, the lo piece's subnormal step); any
  // other set is scaled by the power of two 2^-e that brings m to [2^13,
  // 2^14) (fp16 holds up to 65504).
  // A padded slot beside models of the first kind, all below 2^13, is one of them:
  // -2 x 65504 (1 + sum_a z_a^2), in both pieces, lies below every such model's
  // activation at any z, which is at least -2^13 (9 + 9 sum_a z_a^2) -- by far
  // enough that it has no weight and is never the largest.  So outputs whose models
  // do not fill their last tile need no scales (a rollout with some runs the slower
  // loop of mixture_tiles_sh: 32768 rollouts, 6 x 61 models, 27.3 us per step against
  // 24.5).  Beside any other model the slot holds kPadAct, scaled.
  {
    float mq = 0.0f, my = 0.0f;
    for (int f = a; f < g.KQ; f += 16) mq = fmaxf(mq, fabsf(val[col][f]));
    for (int f = a; f < g.KY; f += 16) my = fmaxf(my, fabsf(val[col][g.KQ + f]));
    auto mx = [](float x, float y) { return fmaxf(x, y); };
    mq = fold_reduce(mq, mx);
    my = fold_reduce(my, mx);
    if (a < 2) {
      const float mm = a == 0 ? mq : my;
      int ex = 0;
      if (mm > 0.0f) frexpf(mm, &ex);   // mm < 2^ex
      (a == 0 ? eq : ey)[col] = (ex > 14 || ex < -1) ? ex - 14 : 0;
      if (a == 0) big[col] = ex > 13;
    }
    if (a == 2) hmeta[(size_t)tile * kHfMeta + col] = s2;
  }
  __syncthreads();
  int any = 0, any_big = 0;   // over the tile's models
  for (int c = 0; c < nvalid; ++c) {
    any |= eq[c] | ey[c];
    any_big |= big[c];
  }
  const bool pad16 = any == 0 && any_big == 0;   // padded slots in fp16's own range
  if (tid >= 16 && tid < 64) {
    const int slot = tid & 15, part = tid >> 4;
    float v = 0.0f;
    if (part < 3)
      v = slot >= nvalid && pad16 ? 1.0f : ldexpf(1.0f, part == 1 ? eq[slot] : ey[slot]);
    else if (slot == kHfPlain - 48)
      v = any == 0 && (nvalid == 16 || pad16) ? 1.0f : 0.0f;
    hmeta[(size_t)tile * kHfMeta + tid] = v;
  }
  u32x4 *dsth = (u32x4 *)(Wh + (size_t)tile * kHfTileU32);
  for (int e = tid; e < kBfNKB * 64; e += kFoldThreads) {
    const int lane = e & 63, kb = e >> 6, k0 = 32 * (kb < kBfNKQ ? kb : 0) + 8 * (lane / 16);
    const bool pad = (lane & 15) >= nvalid && pad16;
    const int sc = pad ? 0 : kb < kBfNKQ ? eq[lane & 15] : ey[lane & 15];
    uint16_t pc[8][2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = k0 + i;
      if (pad && kb < kBfNKQ && ((k < g.NP && pa[k] == pb[k]) || k == g.NP + d))
        pc[i][0] = pc[i][1] = 0xFBFF;   // -65504
      else
        f16_split2(ldexpf(piece_value(kb, k, lane & 15), -sc), pc[i]);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      u32x4 w;
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = (uint32_t)pc[2 * i][p] | ((uint32_t)pc[2 * i + 1][p] << 16);
      dsth[(kb * 2 + p) * 64 + lane] = w;
    }
  }
}

hipError_t launch_fold_mfma(int, const ModelArgs &m, const MfmaLayout &l, void *base, hipStream_t s) {
  float *W = (float *)base;
  float *sig = (float *)((char *)base + align_up(l.w_floats * 4, 256));
  uint32_t *Wb = l.wb_u32 ? (uint32_t *)((char *)sig + align_up(l.sig_floats * 4, 256)) : nullptr;
  uint32_t *Wh = l.wh_u32 ? (uint32_t *)((char *)Wb + align_up(l.wb_u32 * 4, 256)) : nullptr;
  float *hm = l.hm_floats ? (float *)((char *)Wh + align_up(l.wh_u32 * 4, 256)) : nullptr;
  hipLaunchKernelGGL(fold_mfma_kernel, dim3(l.n_tiles), dim3(kFoldThreads), 0, s, m, l, W, sig, Wb, Wh, hm);
  return hipGetLastError();
}

static MfmaModel mfma_view(const MfmaLayout &l, const void *base) {
  MfmaModel md;
  md.W = (const float4 *)base;
  md.sig2 = (const float *)((const char *)base + align_up(l.w_floats * 4, 256));
  md.Wb = l.wb_u32 ? (const uint4 *)((const char *)md.sig2 + align_up(l.sig_floats * 4, 256)) : nullptr;
  md.Wh = l.wh_u32 ? (const uint4 *)((const char *)md.Wb + align_up(l.wb_u32 * 4, 256)) : nullptr;
  md.hmeta = l.hm_floats ? (const float *)((const char *)md.Wh + align_up(l.wh_u32 * 4, 256)) : nullptr;
  md.n_out = l.n_out;
  md.n_tiles = l.n_tiles;
  for (int o = 0; o <= kMaxOut; ++o) md.tile_off[o] = l.tile_off[o];
  return md;
}

// ------------------------------------------------------ shared mixture

// Partial sums of one (sample, output) over a subset of local models.
struct Acc {
  float Z, S1, S2, S3, mx;
};

__device__ __forceinline__ Acc acc_empty() { return Acc{0.f, 0.f, 0.f, 0.f, -3.0e38f}; }
__device__ __forceinline__ Acc acc_sum(const Acc &a, const Acc &b) {
  return Acc{a.Z + b.Z, a.S1 + b.S1, a.S2 + b.S2, a.S3 + b.S3, fmaxf(a.mx, b.mx)};
}

// The sums of the four lane groups that hold the same sample (lanes l, l + 16,
// l + 32, l + 48), in every lane: (g0 + g1) + (g2 + g3).  The row and half-wave
// swaps stay in the vector ALU, where shuffles are two dependent LDS round trips
// per sum.
__device__ __forceinline__ Acc sum_groups(Acc s) {
  auto fold = [](float v, auto op) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const float h = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(h), __float_as_uint(h), false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
  };
  auto add = [](float x, float y) { return x + y; };
  s.Z = fold(s.Z, add);
  s.S1 = fold(s.S1, add);
  s.S2 = fold(s.S2, add);
  s.S3 = fold(s.S3, add);
  s.mx = fold(s.mx, [](float x, float y) { return fmaxf(x, y); });
  return s;
}

// BF (a pieces form): the samples' fragments as pieces (d = 16): per row
// tile, 32-feature block and piece, 64 lanes x 8 bf16 (16 bytes per lane,
// kept in the float4 slots), sample lane%16, features 8 (lane/16) .. +7.
//
// SH (a pieces form with MT > 2 row tiles): the shared-tile form.  The
// workgroup stages each model tile once in LDS (ring) instead of every wave
// streaming its own range; each wave holds RT row tiles, and the TS waves of a
// row group share the model tiles (NPART = TS sets of sums).  The samples'
// pieces are built in registers by their waves (no A).
template <int D, int MT, int NW, int PF = 0>
struct MixSmem {
  static constexpr bool BF = PF != kPfF32;
  static constexpr bool SH = BF && MT > 2;
  static_assert(!BF || (D == kBfD && (MT <= 2 || MT == 4 || MT == 8)), "the pieces forms cover d = 16");
  static constexpr int NPC = PF == kPfF16x2 ? 2 : 3;   // pieces per value
  static constexpr int ROWS = 16 * MT;
  static constexpr int NFRAG = BF ? kBfNKB * NPC : Geo<D>::KB4;   // 16-byte fragments per lane and row tile
  static constexpr int NSRC = BF ? kBfNKB * 32 : Geo<D>::NE;
  // row tiles per wave and waves per row group of the shared-tile form: the
  // bf16 pieces of two row tiles would not fit an eight-wave workgroup's
  // registers beside the rest
  static constexpr int RT = PF == kPfBf16x3 && NW == 8 ? 1 : 2;
  static constexpr int TS = SH ? NW * RT / MT : 1;
  static constexpr int NPART = SH ? TS : NW;
  // outputs held per row: the shared-tile form runs the quadrotor's six
  static constexpr int NOUT = SH ? 6 : kMaxOut;
  static constexpr int XIS = SH ? 6 : 8;   // next-state draws held per row
  // ring of stages of two tiles' piece chunks (1 KiB each, lane-major)
  static constexpr int kChunks = kBfNKB * NPC;
  static constexpr int kRingStages = 3;
  std::conditional_t<SH, char[16], float4[MT][NFRAG][64]> A;   // sample fragments, lane-major (anchor slots 0)
  std::conditional_t<SH, u32x4[kRingStages][2 * kChunks][64], char[16]> ring;
  Acc part[NPART][NOUT][ROWS];           // per-wave partial sums
  float z[ROWS][D + 2];                  // [z, 1, 0]: fragment entries are products of two
  float mref[ROWS][NOUT], yref[ROWS][NOUT];
  float mprev[ROWS][NOUT];               // previous step's largest activation
  // sampled accelerations (rollouts); the shared-tile form, whose LDS is full,
  // leaves them in the Z slots of the sums they come from
  float acc[SH ? 1 : ROWS][NOUT];
  __device__ __forceinline__ float &accel(int row, int o) {
    if constexpr (SH)
      return part[0][o][row].Z;
    else
      return acc[row][o];
  }
  unsigned short fsrc[NSRC];             // entry (BF: feature slot) -> (ia << 8) | ib into z[row][]
  int redo[2];                           // second-pass requests, by evaluation parity
  int pair_fail;                         // a partner wait ran out (results invalid)
  int model_scaled;                      // SH, fp16 form: some tile's scales are not all 1
};

// fp16 form: the exponent e >= 0 of the power of two 2^-e that scales every
// feature of sample row `row` (products of two entries of [z, 1]) and its
// anchors below 2^14 in magnitude; the fragment build, the anchors and the
// epilogue all take it from here, so they agree.
template <int D, int MT, int NW, int PF>
__device__ __forceinline__ int row_scale_exp(const MixSmem<D, MT, NW, PF> &sm, int row) {
  float mx = 1.0f;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const float za = fabsf(sm.z[row][a]);
    mx = fmaxf(mx, fmaxf(za, za * za));
  }
#pragma unroll
  for (int o = 0; o < MixSmem<D, MT, NW, PF>::NOUT; ++o)
    mx = fmaxf(mx, fmaxf(fabsf(sm.mref[row][o]), fabsf(sm.yref[row][o])));
  int ex = 0;
  frexpf(mx, &ex);   // mx < 2^ex
  return ex > 14 ? ex - 14 : 0;
}

// Fragment entry e = ((kb4 * 64 + lane) * 4 + comp) of row tile mt holds
// feature f = 4 (4 kb4 + comp) + lane/16 of row 16 mt + lane%16; every feature
// is a product z'[ia] z'[ib] of the extended input z' = [z, 1, 0].
// In the bf16 form (BF) entry e is feature slot e: slots 0 .. 32 kBfNKQ - 1
// the quadratic-form features (f = e), the last block's the prediction
// features (f = 4 KQB + e - 32 kBfNKQ in the numbering above).
template <int D, int MT, int NW, int PF>
__device__ void mix_setup(MixSmem<D, MT, NW, PF> &sm) {
  using G = Geo<D>;
  for (int e = threadIdx.x; e < MixSmem<D, MT, NW, PF>::NSRC; e += NW * 64) {
    int f;
    if constexpr (MixSmem<D, MT, NW, PF>::BF) {
      const int g = e - 32 * kBfNKQ;
      f = e < 32 * kBfNKQ ? (e < G::KQ ? e : -1) : (g < G::KY ? 4 * G::KQB + g : -1);
    } else {
      const int comp = e & 3, lane = (e >> 2) & 63, kb4 = e >> 8;
      f = 4 * (4 * kb4 + comp) + lane / 16;
    }
    int ia = D + 1, ib = D + 1;  // zero
    if (f < 0) {
      // padding slot of the bf16 form
    } else if (f < G::NP) {
      int a = 0, rem = f;
      while (rem >= D - a) {
        rem -= D - a;
        ++a;
      }
      ia = a;
      ib = a + rem;
    } else if (f < G::NP + D) {
      ia = f - G::NP;
      ib = D;
    } else if (f == G::NP + D) {
      ia = D;
      ib = D;
    } else if (f >= 4 * G::KQB && f < 4 * G::KQB + D) {
      ia = f - 4 * G::KQB;
      ib = D;
    } else if (f == 4 * G::KQB + D) {
      ia = D;
      ib = D;
    }
    sm.fsrc[e] = (unsigned short)((ia << 8) | ib);
  }
  if (threadIdx.x == 0) {
    sm.redo[0] = sm.redo[1] = 0;
    sm.pair_fail = 0;
  }
}

// Stage 1 (all lanes): the samples' fragments sm.A from sm.z (named for the
// parameter pass, where they are the A operand; the rollout and the reverse
// sweep use them as the B operand).
template <int D, int MT, int NW, int PF>
__device__ __forceinline__ void build_fragments(MixSmem<D, MT, NW, PF> &sm) {
  using G = Geo<D>;
  if constexpr (MixSmem<D, MT, NW, PF>::SH) {
    return;   // built in registers by mixture_tiles_sh
  } else if constexpr (MixSmem<D, MT, NW, PF>::BF) {
    // one (block, lane group, row) per thread: the group's 8 features of the
    // row, each split into its pieces (three bf16, or two fp16 of the value
    // scaled by the row's power of two), one 16-byte store per piece
    constexpr int NPC = MixSmem<D, MT, NW, PF>::NPC;
    constexpr int NWORK = MT * kBfNKB * 4 * 16;
    u32x4 *Ab = (u32x4 *)&sm.A[0][0][0];
    for (int w = threadIdx.x; w < NWORK; w += NW * 64) {
      const int r16 = w & 15, grp = (w >> 4) & 3, kb = (w >> 6) % kBfNKB, mt = (w >> 6) / kBfNKB;
      const int row = 16 * mt + r16;
      const float rsi = PF == kPfF16x2 ? ldexpf(1.0f, -row_scale_exp(sm, row)) : 1.0f;
      uint32_t pk[NPC][4];
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        uint16_t lo[3], hi[3];
        const unsigned s0 = sm.fsrc[32 * kb + 8 * grp + i], s1 = sm.fsrc[32 * kb + 8 * grp + i + 1];
        const float v0 = sm.z[row][s0 >> 8] * sm.z[row][s0 & 0xFF], v1 = sm.z[row][s1 >> 8] * sm.z[row][s1 & 0xFF];
        if constexpr (PF == kPfF16x2) {
          f16_split2(v0 * rsi, lo);
          f16_split2(v1 * rsi, hi);
        } else {
          bf16_split3(v0, lo);
          bf16_split3(v1, hi);
        }
#pragma unroll
        for (int p = 0; p < NPC; ++p) pk[p][i / 2] = (uint32_t)lo[p] | ((uint32_t)hi[p] << 16);
      }
#pragma unroll
      for (int p = 0; p < NPC; ++p)
        Ab[((mt * kBfNKB + kb) * NPC + p) * 64 + 16 * grp + r16] = u32x4{pk[p][0], pk[p][1], pk[p][2], pk[p][3]};
    }
  } else {
    float *Af = (float *)&sm.A[0][0][0];
    // fixed trip count, fully unrolled: every thread's reads go out together
    // (a rolled loop waits for two dependent LDS round trips per element)
    constexpr int NIT = (MT * G::NE + NW * 64 - 1) / (NW * 64);
    unsigned src[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int e = threadIdx.x + it * NW * 64;
      src[it] = e < MT * G::NE ? sm.fsrc[e % G::NE] : 0u;
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int e = threadIdx.x + it * NW * 64;
      if (e < MT * G::NE) {
        const int row = 16 * (e / G::NE) + (((e % G::NE) >> 2) & 15);
        Af[e] = sm.z[row][src[it] >> 8] * sm.z[row][src[it] & 0xFF];
      }
    }
  }
}

// Empty per-wave partial sums: a wave flushes only the outputs its tiles
// meet, and the merge adds every wave's slot in order.
template <int D, int MT, int NW, int PF>
__device__ __forceinline__ void clear_parts(MixSmem<D, MT, NW, PF> &sm) {
  Acc *pp = &sm.part[0][0][0];
  using SM = MixSmem<D, MT, NW, PF>;
  for (int i = threadIdx.x; i < SM::NPART * SM::NOUT * SM::ROWS; i += NW * 64) pp[i] = acc_empty();
}

// Stage 2 (each wave): its contiguous range of model tiles, one MFMA chain per
// tile with the model tile as the A operand: lane l holds models 4(l/16) + i
// (i < 4) of sample l%16.  Partial sums are flushed per output into
// sm.part[wave][o][row].
template <int D, int MT, int NW, int PF>
__device__ __forceinline__ void mixture_tiles(const MfmaModel &md, MixSmem<D, MT, NW, PF> &sm, int T0, int T1) {
  static_assert(PF == kPfF32, "float32 products: the pieces forms have their own tile loops");
  using G = Geo<D>;
  constexpr int KQS = G::FQS / 4, GQS = G::FQS % 4;   // kblock / lane group of the anchors
  constexpr int KYS = G::FYS / 4, GYS = G::FYS % 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the wave's tile range is uniform across its lanes: held in scalar
  // registers, the tile loop's control and the model addresses stay off the
  // vector ALU
  const int t0 = __builtin_amdgcn_readfirstlane(T0 + (int)((int64_t)wave * (T1 - T0) / NW));
  const int t1 = __builtin_amdgcn_readfirstlane(T0 + (int)((int64_t)(wave + 1) * (T1 - T0) / NW));
  if (t0 >= t1) return;
  f32x4 A[MT][G::KB4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int q = 0; q < G::KB4; ++q) {
      const float4 v = sm.A[mt][q][lane];
      A[mt][q] = f32x4{v.x, v.y, v.z, v.w};
    }
  // Output of a tile and the next output boundary, from compile-time indexed
  // scans of tile_off (scalar registers): a runtime-indexed read would be a
  // vector memory load whose wait would also drain the B prefetch.
  auto output_of = [&](int tile) {
    int oo = 0;
#pragma unroll
    for (int i = 1; i < kMaxOut; ++i) oo += (i < md.n_out && md.tile_off[i] <= tile) ? 1 : 0;
    return oo;
  };
  auto next_boundary = [&](int tile) {
    int nb = md.n_tiles;
#pragma unroll
    for (int i = 1; i <= kMaxOut; ++i) {
      const int v = md.tile_off[i];
      nb = (v > tile && v < nb) ? v : nb;
    }
    return nb;
  };
  int o = output_of(t0);
  int nb = next_boundary(t0);
  // anchors of output o go into the lanes of the shift features
  auto set_anchor = [&](int oo) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int row = 16 * mt + (lane & 15);
      if ((lane >> 4) == GQS) A[mt][KQS / 4][KQS % 4] = -sm.mref[row][oo];
      if ((lane >> 4) == GYS) A[mt][KYS / 4][KYS % 4] = -sm.yref[row][oo];
    }
  };
  set_anchor(o);
  // st[mt][i]: sums over this lane's model 4(lane/16) + i of every tile so
  // far, for sample 16 mt + lane%16
  Acc st[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) st[mt][i] = acc_empty();

  // the four models of the lane, then the four lane groups holding the same
  // sample (lanes l, l^16, l^32, l^48); every lane ends with the same sums
  auto flush = [&](int oo) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      Acc s = acc_sum(acc_sum(st[mt][0], st[mt][1]), acc_sum(st[mt][2], st[mt][3]));
      s = sum_groups(s);
      if (lane < 16) sm.part[wave][oo][16 * mt + lane] = s;
#pragma unroll
      for (int i = 0; i < 4; ++i) st[mt][i] = acc_empty();
    }
  };

  // Software pipeline over tiles with two buffers: the loads of tile i+1 are
  // issued before the MFMA chain of tile i, and scheduling barriers keep the
  // compiler from sinking them next to their use.  sigma^2 of the lane's four
  // models travels with its tile (loads complete in order, so a later load
  // would make the wait drain the prefetch too).
  f32x4 B0[G::KB4], B1[G::KB4];
  f32x4 s2_0, s2_1;
  // Tile loads of the large feature set through buffer descriptors.
  constexpr int kTileBytes = G::KB4 * 64 * 16;
  const __amdgpu_buffer_rsrc_t wrs = buffer_rsrc(md.W, md.n_tiles * kTileBytes);
  const __amdgpu_buffer_rsrc_t srs = buffer_rsrc(md.sig2, md.n_tiles * 16 * 4);
  const int lane_off = lane * 16, grp_off = 16 * (lane >> 4);
  auto load_tile = [&](f32x4 (&Bd)[G::KB4], f32x4 &s2d, int tile) {
    if constexpr (G::KB4 >= 4) {
      const int base = tile * kTileBytes;
#pragma unroll
      for (int q = 0; q < G::KB4; ++q) Bd[q] = buffer_f32x4(wrs, lane_off, base + q * 1024);
      s2d = buffer_f32x4(srs, grp_off, tile * 64);
    } else {
      // small feature sets (two or three fragments per lane) measured faster
      // with plain global loads
      const f32x4 *src = (const f32x4 *)md.W + (size_t)tile * G::KB4 * 64 + lane;
#pragma unroll
      for (int q = 0; q < G::KB4; ++q) Bd[q] = src[q * 64];
      s2d = *(const f32x4 *)(md.sig2 + tile * 16 + 4 * (lane >> 4));
    }
  };
  auto compute_tile = [&](const f32x4 (&Bc)[G::KB4], const f32x4 &s2, int tile) {
    if (tile >= nb) {
      flush(o);
      o = output_of(tile);
      nb = next_boundary(tile);
      set_anchor(o);
    }
    f32x4 qa[MT], qb[MT], ya[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      qa[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      qb[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      ya[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // two interleaved accumulators per row tile shorten the dependency chain;
    // the model tile is the A operand, the samples' fragments the B operand
#pragma unroll
    for (int kb = 0; kb < G::KQB; ++kb)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        if (kb & 1)
          qb[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(Bc[kb / 4][kb % 4], A[mt][kb / 4][kb % 4],
                                                        qb[mt], 0, 0, 0);
        else
          qa[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(Bc[kb / 4][kb % 4], A[mt][kb / 4][kb % 4],
                                                        qa[mt], 0, 0, 0);
      }
#pragma unroll
    for (int kb = G::KQB; kb < G::KB; ++kb)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        ya[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(Bc[kb / 4][kb % 4], A[mt][kb / 4][kb % 4],
                                                      ya[mt], 0, 0, 0);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float a = qa[mt][i] + qb[mt][i], dd = ya[mt][i];
        // bare v_exp_f32: arguments below -126 (weights under 2^-126 next to a
        // largest term of at least 2^-100) need none of exp2f's denormal scaling
        const float e = __builtin_amdgcn_exp2f(a);
        const float te = e * dd;
        st[mt][i].Z += e;
        st[mt][i].S1 += te;
        st[mt][i].S2 = fmaf(te, dd, st[mt][i].S2);
        st[mt][i].S3 = fmaf(e, s2[i], st[mt][i].S3);
        st[mt][0].mx = fmaxf(st[mt][0].mx, a);   // one running max per row
      }
  };

  // Prefetches are unconditional (a clamped index re-reads the last tile) so
  // that every wait counts exactly the loads issued after the needed ones.
  load_tile(B0, s2_0, t0);
  for (int tile = t0; tile < t1; tile += 2) {
    load_tile(B1, s2_1, min(tile + 1, t1 - 1));
    __builtin_amdgcn_sched_barrier(0);
    compute_tile(B0, s2_0, tile);
    __builtin_amdgcn_sched_barrier(0);
    if (tile + 1 >= t1) break;
    load_tile(B0, s2_0, min(tile + 2, t1 - 1));
    __builtin_amdgcn_sched_barrier(0);
    compute_tile(B1, s2_1, tile + 1);
    __builtin_amdgcn_sched_barrier(0);
  }
  flush(o);
}

// The same stage in the three-piece bf16 form (d = 16, one or two row tiles):
// per 32-feature block, six bf16 16x16x32 instructions take the piece pairs hi hi,
// hi mid, mid hi, hi lo, mid mid, lo hi (model tile as the A operand, the
// samples' pieces as the B operand), which reproduce the float32 products to
// within float32 rounding; five blocks of quadratic-form features into one
// accumulator, one block of prediction features into another.  With two row
// tiles every model piece loaded serves both, halving the loads per product
// (the loads, not the matrix cores, bound the one-tile form).  The model
// tile's pieces (18 KB) are held in registers once: as each block's products
// issue, the registers of that block take the next tile's block (loads one
// tile ahead).  The softmax epilogue and the flush are the float32 form's.
// The two-piece fp16 form runs the same loop with three fp16 instructions per
// block (hi hi, hi lo, lo hi of scaled values; 12 KB of pieces per tile) and
// undoes the models' and rows' powers of two in the epilogue.
// NPU: pieces used per value, all of them or (a coarse pass, whose sums serve as
// anchors only) the leading one.
template <int D, int MT, int NW, int PF, int NPU = MixSmem<D, MT, NW, PF>::NPC, bool TWO = false>
__device__ __forceinline__ void mixture_tiles_bf(const MfmaModel &md, MixSmem<D, MT, NW, PF> &sm, int T0, int T1) {
  static_assert(PF != kPfF32 && D == kBfD && (MT == 1 || MT == 2), "pieces forms: d = 16, one or two row tiles");
  using G = Geo<D>;
  constexpr bool HF = PF == kPfF16x2;   // two fp16 pieces (else three bf16 pieces)
  constexpr int NPC = MixSmem<D, MT, NW, PF>::NPC;
  // bytes of per-model values per tile: sigma^2, or (fp16 form) sigma^2 and the two scales
  constexpr int kMetaBytes = HF ? kHfMeta * 4 : 16 * 4;
  // the activation anchor and the prediction reference: block, lane group, element
  constexpr int FQ = G::NP + D + 1, KQA = FQ / 32, GQA = (FQ % 32) / 8, IQA = FQ % 8;
  constexpr int FY = D + 1, KYA = kBfNKQ + FY / 32, GYA = (FY % 32) / 8, IYA = FY % 8;
  constexpr int kTileBytes = kBfNKB * NPC * 1024;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t0 = __builtin_amdgcn_readfirstlane(T0 + (int)((int64_t)wave * (T1 - T0) / NW));
  const int t1 = __builtin_amdgcn_readfirstlane(T0 + (int)((int64_t)(wave + 1) * (T1 - T0) / NW));
  if (t0 >= t1) return;
  u32x4 Bs[MT][kBfNKB][NPU];
  {
    const u32x4 *Ab = (const u32x4 *)&sm.A[0][0][0];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int kb = 0; kb < kBfNKB; ++kb)
#pragma unroll
        for (int p = 0; p < NPU; ++p) Bs[mt][kb][p] = Ab[((mt * kBfNKB + kb) * NPC + p) * 64 + lane];
  }
  // fp16 form: the lane's rows' powers of two (as in the fragment build)
  float rsc[MT], rsi[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    rsc[mt] = 1.0f;
    rsi[mt] = 1.0f;
    if constexpr (HF) {
      const int e = row_scale_exp(sm, 16 * mt + (lane & 15));
      rsc[mt] = ldexpf(1.0f, e);
      rsi[mt] = ldexpf(1.0f, -e);
    }
  }
  auto output_of = [&](int tile) {
    int oo = 0;
#pragma unroll
    for (int i = 1; i < kMaxOut; ++i) oo += (i < md.n_out && md.tile_off[i] <= tile) ? 1 : 0;
    return oo;
  };
  auto next_boundary = [&](int tile) {
    int nb = md.n_tiles;
#pragma unroll
    for (int i = 1; i <= kMaxOut; ++i) {
      const int v = md.tile_off[i];
      nb = (v > tile && v < nb) ? v : nb;
    }
    return nb;
  };
  // element I of the three pieces (blocks of 8 bf16) takes the pieces of x
  auto put = [&](u32x4 (&v)[NPU], auto I, float x, int mt) {
    constexpr int i = decltype(I)::value;
    uint16_t pc[3];
    if constexpr (HF)
      f16_split2(x * rsi[mt], pc);
    else
      bf16_split3(x, pc);
#pragma unroll
    for (int p = 0; p < NPU; ++p) {
      uint32_t w = v[p][i / 2];
      w = (i & 1) ? ((w & 0x0000FFFFu) | ((uint32_t)pc[p] << 16)) : ((w & 0xFFFF0000u) | pc[p]);
      v[p][i / 2] = w;
    }
  };
  int o = output_of(t0);
  int nb = next_boundary(t0);
  auto set_anchor = [&](int oo) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int row = 16 * mt + (lane & 15);
      if ((lane >> 4) == GQA) put(Bs[mt][KQA], std::integral_constant<int, IQA>{}, -sm.mref[row][oo], mt);
      if ((lane >> 4) == GYA) put(Bs[mt][KYA], std::integral_constant<int, IYA>{}, -sm.yref[row][oo], mt);
    }
  };
  set_anchor(o);
  Acc st[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) st[mt][i] = acc_empty();
  auto flush = [&](int oo) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      Acc s = acc_sum(acc_sum(st[mt][0], st[mt][1]), acc_sum(st[mt][2], st[mt][3]));
      s = sum_groups(s);
      if (lane < 16) sm.part[wave][oo][16 * mt + lane] = s;
#pragma unroll
      for (int i = 0; i < 4; ++i) st[mt][i] = acc_empty();
    }
  };
  const __amdgpu_buffer_rsrc_t wrs = buffer_rsrc(HF ? (const void *)md.Wh : (const void *)md.Wb,
                                                 md.n_tiles * kTileBytes);
  const __amdgpu_buffer_rsrc_t srs = buffer_rsrc(HF ? md.hmeta : md.sig2, md.n_tiles * kMetaBytes);
  const int lane_off = lane * 16, grp_off = 16 * (lane >> 4);
  u32x4 W[kBfNKB][NPU];
  auto load_blk = [&](int tile, int kb) {
#pragma unroll
    for (int p = 0; p < NPU; ++p)
      W[kb][p] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                               wrs, lane_off, tile * kTileBytes + (kb * NPC + p) * 1024, 0));
  };
  auto mm = [&](const u32x4 &a, const u32x4 &b, f32x4 c) {
    if constexpr (HF)
      return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                    0, 0);
    else
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                     0, 0, 0);
  };
  // the piece pairs of block kb of row tile mt into one accumulator (the pipe
  // takes a dependent product at full rate): bf16 hh, hm, mh, hl, mm, lh;
  // fp16 hh, hl, lh
  // TWO: the leading products (hh) and the others go into accumulators of their
  // own (lo: 2^-8 of hh and less), so that the sum rounds once per block at its
  // full magnitude instead of six times.  For predictions, whose error it is
  // (100003 inputs, 6 x 256 models, means against float64: 2.7e-7, 6.1e-7 in one
  // accumulator, 4.5e-7 in float32 products); a rollout's error does not feel it
  // and its loop would pay 7 %.
  auto block6 = [&](int mt, int kb, f32x4 &x, f32x4 &lo) {
    x = mm(W[kb][0], Bs[mt][kb][0], x);
    f32x4 &r = TWO ? lo : x;
    if constexpr (NPU > 1) {
      r = mm(W[kb][0], Bs[mt][kb][1], r);
      r = mm(W[kb][1], Bs[mt][kb][0], r);
    }
    if constexpr (NPU > 2) {
      r = mm(W[kb][0], Bs[mt][kb][2], r);
      r = mm(W[kb][1], Bs[mt][kb][1], r);
      r = mm(W[kb][2], Bs[mt][kb][0], r);
    }
  };
  // With two row tiles (one wave per SIMD, nothing else to overlap with) two
  // accumulator sets take turns: while the matrix cores take tile i into one,
  // the epilogue (exponentials and sums) of tile i-1 is issued between them
  // from the other.  Every element still meets the same operations in tile
  // order, so the sums match the unpipelined loop bit for bit; a pending set
  // with activation -inf, prediction 0 and sigma^2 0 adds exact zeros.  With
  // one row tile two waves per SIMD overlap instead, and the epilogue follows
  // the products.
  constexpr bool PIPE = MT == 2;
  // per accumulator set: sigma^2 of the tile's models and (fp16 form) their scales
  f32x4 qa[2][MT], ya[2][MT], s2[2], qsc[2], ysc[2];
  f32x4 ql[2][MT], yl[2][MT];   // (TWO) the lower products' sums
  auto clear_pending = [&](auto PI) {
    constexpr int p = decltype(PI)::value;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      qa[p][mt] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      ya[p][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      ql[p][mt] = ya[p][mt];
      yl[p][mt] = ya[p][mt];
    }
    s2[p] = f32x4{0.f, 0.f, 0.f, 0.f};
    qsc[p] = f32x4{1.f, 1.f, 1.f, 1.f};
    ysc[p] = qsc[p];
  };
  auto epi = [&](auto PI, int mt, int i) {
    constexpr int p = decltype(PI)::value;
    // fp16 form: the model's and the row's powers of two undone (exact)
    const float qv = TWO ? qa[p][mt][i] + ql[p][mt][i] : qa[p][mt][i];
    const float yv = TWO ? ya[p][mt][i] + yl[p][mt][i] : ya[p][mt][i];
    const float a = HF ? qv * (qsc[p][i] * rsc[mt]) : qv;
    const float dd = HF ? yv * (ysc[p][i] * rsc[mt]) : yv;
    // bare v_exp_f32: arguments below -126 (weights under 2^-126 next to a
    // largest term of at least 2^-100) need none of exp2f's denormal scaling
    const float e = __builtin_amdgcn_exp2f(a);
    const float te = e * dd;
    st[mt][i].Z += e;
    st[mt][i].S1 += te;
    st[mt][i].S2 = fmaf(te, dd, st[mt][i].S2);
    st[mt][i].S3 = fmaf(e, s2[p][i], st[mt][i].S3);
    st[mt][0].mx = fmaxf(st[mt][0].mx, a);   // one running max per row
  };
  auto epi_all = [&](auto PI) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) epi(PI, mt, i);
  };
  // tile `tile` into set c (and, pipelined, set p = tile - 1 finished); on
  // entry s2[c] holds tile's sigma^2 (and s2[p] tile - 1's), on exit the set
  // that takes tile + 1 holds tile + 1's
  auto body = [&](int tile, auto CI, auto PI) {
    constexpr int c = decltype(CI)::value, p = decltype(PI)::value;
    if (tile >= nb) {
      if constexpr (PIPE) {
        epi_all(PI);
        clear_pending(PI);
      }
      flush(o);
      o = output_of(tile);
      nb = next_boundary(tile);
      set_anchor(o);
    }
    // prefetches are unconditional (the last tile re-reads itself) so that
    // every wait counts a fixed number of loads
    const int tn = min(tile + 1, t1 - 1);
    const f32x4 s2n = buffer_f32x4(srs, grp_off, tn * kMetaBytes);
    f32x4 qsn, ysn;
    if constexpr (HF) {
      qsn = buffer_f32x4(srs, grp_off + 64, tn * kMetaBytes);
      ysn = buffer_f32x4(srs, grp_off + 128, tn * kMetaBytes);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      qa[c][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      ya[c][mt] = qa[c][mt];
      ql[c][mt] = qa[c][mt];
      yl[c][mt] = qa[c][mt];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kb = 0; kb < kBfNKB; ++kb) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) block6(mt, kb, kb < kBfNKQ ? qa[c][mt] : ya[c][mt], kb < kBfNKQ ? ql[c][mt] : yl[c][mt]);
      if constexpr (PIPE) {
        // this block's share of the pending epilogue, between its products
#pragma unroll
        for (int e = 0; e < 4 * MT; ++e)
          if (e * kBfNKB / (4 * MT) == kb) epi(PI, e / 4, e % 4);
      }
      load_blk(tn, kb);
      if constexpr (PIPE) {
#pragma unroll
        for (int j = 0; j < NPU * (NPU + 1) / 2 * MT; ++j) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one product
          __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // two vector ALU ops
        }
        __builtin_amdgcn_sched_group_barrier(0x020, NPU, 0);  // the piece loads
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!PIPE) epi_all(CI);
    s2[p] = s2n;
    if constexpr (HF) {
      qsc[p] = qsn;
      ysc[p] = ysn;
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // the first tile's loads in the loop's own order (block 0 first): the
  // loop's first wait is the merge of this order and the loop body's, and a
  // block 0 issued last here would make it wait for every load in flight on
  // every tile, the next tile's prefetch included
#pragma unroll
  for (int kb = 0; kb < kBfNKB; ++kb) {
    load_blk(t0, kb);
    __builtin_amdgcn_sched_barrier(0);
  }
  s2[0] = buffer_f32x4(srs, grp_off, t0 * kMetaBytes);
  if constexpr (HF) {
    qsc[0] = buffer_f32x4(srs, grp_off + 64, t0 * kMetaBytes);
    ysc[0] = buffer_f32x4(srs, grp_off + 128, t0 * kMetaBytes);
  }
  if constexpr (PIPE) {
    clear_pending(I1{});
    int tile = t0;
    for (; tile + 1 < t1; tile += 2) {
      body(tile, I0{}, I1{});
      body(tile + 1, I1{}, I0{});
    }
    if (tile < t1) {
      body(tile, I0{}, I1{});
      epi_all(I0{});
    } else {
      epi_all(I1{});
    }
  } else {
    for (int tile = t0; tile < t1; ++tile) body(tile, I0{}, I0{});
  }
  flush(o);
}

// f(integral_constant<int, i>) for i = B .. E-1, unrolled at compile time.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// The shared-tile form of the pieces stage (MixSmem::SH): 128 or 64 rows in
// groups of 16 RT, every wave holding the pieces of one group.  With two row tiles per
// wave each model piece read from LDS serves two products; the workgroup reads
// each model tile from L2 once per step: the tile's piece chunks go straight
// from memory into an LDS ring (buffer loads to LDS, each wave issuing every
// NW-th chunk).  The tiles go in stages of two.  Where the waves just cover the
// rows each runs both tiles of a stage; where two waves hold the same rows
// (TS = 2: 64 rows on four waves, 128 on eight of two row tiles each) they take
// one tile of the stage each and their sums meet in the merge.  Three stages fit the
// ring: a stage's loads are issued two stages ahead, spread over the products
// of the stage in hand (all at once after the barrier they held every wave up
// for about 400 cycles).  Per stage a wave waits for its own loads and then for
// the other waves at a barrier: past it the stage is complete and every wave is
// done with the slots the next loads overwrite.
//
// Bound: the matrix pipe (36 fp16 products of 16 cycles per wave and tile) and,
// with it, the card's power: its clock falls as the pipe fills.  A product
// leaves room for two vector instructions beside it, so the softmax epilogue of
// the wave's previous tile (52 vector operations and 8 exponentials) is issued
// between the products of the tile in hand, from a second accumulator set, as
// in mixture_tiles_bf: a pending set with activation -inf, prediction 0 and
// sigma^2 0 adds exact zeros.  At 65536 rollouts x 200 steps x 6 x 1024 models
// (fp16 pieces, 8 waves) a stage of two tiles takes 1833 cycles at 2.06 GHz,
// the pipe 64 % busy, 68.9 ms in all (1350 TFLOP/s of executed fp16 products);
// one row tile per wave, every piece read for one product and the epilogue
// behind the products: 2540 cycles at 2.35 GHz, 83.7 ms on the same card.  bf16
// pieces, 40 steps: 25.8 against 26.5 ms.
// NPU and TWO as in mixture_tiles_bf.
template <int D, int MT, int NW, int PF, int NPU = MixSmem<D, MT, NW, PF>::NPC, bool TWO = false>
__device__ __forceinline__ void mixture_tiles_sh(const MfmaModel &md, MixSmem<D, MT, NW, PF> &sm, int T0, int T1) {
  using SM = MixSmem<D, MT, NW, PF>;
  static_assert(SM::SH && (NW == 4 || (NW == 8 && MT == 8)), "shared-tile form: 64 rows on four, 128 on four or eight waves");
  using G = Geo<D>;
  constexpr bool HF = PF == kPfF16x2;   // two fp16 pieces (else three bf16 pieces)
  constexpr int NPC = SM::NPC;
  constexpr int RT = SM::RT;     // row tiles per wave
  constexpr int RG = MT / RT;    // row groups
  constexpr int TS = SM::TS;     // waves per row group: each takes every TS-th tile
  static_assert(RG * TS == NW && (TS == 1 || TS == 2), "shared-tile form: the waves cover the rows");
  // two waves per SIMD: a stage outlasts its loads, so all of them are waited
  // for, and the next tile's first blocks are read before the barrier; one wave
  // per SIMD: the loads get two stages, the first reads wait behind the barrier
  constexpr bool XB = NW == 8;
  constexpr int FQ = G::NP + D + 1, KQA = FQ / 32, GQA = (FQ % 32) / 8, IQA = FQ % 8;
  constexpr int FY = D + 1, KYA = kBfNKQ + FY / 32, GYA = (FY % 32) / 8, IYA = FY % 8;
  constexpr int kTileBytes = kBfNKB * NPC * 1024;
  // bytes of per-model values per tile: sigma^2, or (fp16 form) sigma^2 and the two scales
  constexpr int kMetaBytes = HF ? kHfMeta * 4 : 16 * 4;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int half = TS == 2 ? wave / RG : 0;
  const int row0 = 16 * RT * (wave % RG) + (lane & 15);   // the lane's row of row tile 0
  const int n = T1 - T0;
  const __amdgpu_buffer_rsrc_t wrs = buffer_rsrc(HF ? (const void *)md.Wh : (const void *)md.Wb,
                                                 md.n_tiles * kTileBytes);
  const __amdgpu_buffer_rsrc_t srs = buffer_rsrc(HF ? md.hmeta : md.sig2, md.n_tiles * kMetaBytes);
  // Stage st_i: tiles 2 st_i and 2 st_i + 1, their chunks (contiguous in memory)
  // in ring stage st_i % NSTG.  Load q of this wave is chunk wave + NW q of the
  // stage.  The loads are unconditional: past the stage's last chunk they
  // repeat it, past the range's last tile they re-read that tile's end into
  // slots that nobody reads (no branch in the tile loop).
  constexpr int NSTG = SM::kRingStages;
  constexpr int kChunks = kBfNKB * NPU;   // of a tile
  constexpr int kLoads = (2 * kChunks + NW - 1) / NW;
  const int n_st = (n + 1) / 2;
  const int src_end = T1 * kTileBytes - 1024;
  auto issue = [&](int st_i, int ring, int q) {
    const int j = min(wave + NW * q, 2 * kChunks - 1);
    // chunk (block, piece) of the stage's two tiles: contiguous when every piece is used
    const int off = NPU == NPC ? j * 1024 : j / kChunks * kTileBytes + (j % kChunks) / NPU * (NPC * 1024) + j % NPU * 1024;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (__attribute__((address_space(3))) void *)&sm.ring[ring][j][0], 16,
                                             lane * 16, min((T0 + 2 * st_i) * kTileBytes + off, src_end), 0, 0);
  };
  auto issue_stage = [&](int st_i) {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) issue(st_i, st_i % NSTG, q);
  };
  if (n > 0) {
    issue_stage(0);
    issue_stage(1);
  }
  // fp16 form: each row's features (and its anchors) scaled by a power of two
  // 2^-e (e >= 0) that keeps them below 2^14 in magnitude; rsc[mt] = 2^e
  // undoes it in the epilogue
  float rsc[RT], rsi[RT];
#pragma unroll
  for (int mt = 0; mt < RT; ++mt) {
    rsc[mt] = 1.0f;
    rsi[mt] = 1.0f;
    if constexpr (HF) {
      const int e = row_scale_exp(sm, row0 + 16 * mt);
      rsc[mt] = ldexpf(1.0f, e);
      rsi[mt] = ldexpf(1.0f, -e);
    }
  }
  // the pieces of one feature value (scaled in the fp16 form)
  auto split = [&](float x, int mt, uint16_t *pc) {
    if constexpr (HF)
      f16_split2(x * rsi[mt], pc);
    else
      bf16_split3(x, pc);
  };
  // the wave's sample pieces, built in registers (rows row0 + 16 mt, features
  // 32 kb + 8 (lane/16) .. +7 of block kb)
  u32x4 Bs[RT][kBfNKB][NPU];
  {
    const int grp = lane >> 4;
#pragma unroll
    for (int kb = 0; kb < kBfNKB; ++kb) {
      unsigned src[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) src[i] = sm.fsrc[32 * kb + 8 * grp + i];
#pragma unroll
      for (int mt = 0; mt < RT; ++mt) {
        const int row = row0 + 16 * mt;
        uint32_t pk[NPU][4];
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          uint16_t lo[3], hi[3];
          split(sm.z[row][src[i] >> 8] * sm.z[row][src[i] & 0xFF], mt, lo);
          split(sm.z[row][src[i + 1] >> 8] * sm.z[row][src[i + 1] & 0xFF], mt, hi);
#pragma unroll
          for (int p = 0; p < NPU; ++p) pk[p][i / 2] = (uint32_t)lo[p] | ((uint32_t)hi[p] << 16);
        }
#pragma unroll
        for (int p = 0; p < NPU; ++p) Bs[mt][kb][p] = u32x4{pk[p][0], pk[p][1], pk[p][2], pk[p][3]};
      }
    }
  }
  // the output of a tile and the first tile past it: every output has a tile,
  // so tile_off grows up to n_tiles; scalar selects only
  auto locate = [&](int tile, int &oo, int &nb) {
#pragma unroll
    for (int i = kMaxOut; i >= 1; --i) {
      const bool past = md.tile_off[i] > tile;
      nb = past ? md.tile_off[i] : nb;
      oo = past ? i - 1 : oo;
    }
    oo = __builtin_amdgcn_readfirstlane(oo);
    nb = __builtin_amdgcn_readfirstlane(nb);
  };
  // output oo's anchors into their feature slots: one LDS round trip, and a
  // select instead of a branch for the lanes that hold the slots
  auto set_anchor = [&](int oo) {
    float m[RT], y[RT];
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
      m[mt] = sm.mref[row0 + 16 * mt][oo];
      y[mt] = sm.yref[row0 + 16 * mt][oo];
    }
    auto put = [&](u32x4 (&v)[NPU], auto I, bool mine, float x, int mt) {
      constexpr int i = decltype(I)::value;
      uint16_t pc[3];
      split(x, mt, pc);
#pragma unroll
      for (int p = 0; p < NPU; ++p) {
        const uint32_t w = v[p][i / 2];
        const uint32_t n = (i & 1) ? ((w & 0x0000FFFFu) | ((uint32_t)pc[p] << 16)) : ((w & 0xFFFF0000u) | pc[p]);
        v[p][i / 2] = mine ? n : w;
      }
    };
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
      put(Bs[mt][KQA], std::integral_constant<int, IQA>{}, (lane >> 4) == GQA, -m[mt], mt);
      put(Bs[mt][KYA], std::integral_constant<int, IYA>{}, (lane >> 4) == GYA, -y[mt], mt);
    }
  };
  // sums over the lane's models 4 (lane/16) + i: one per i, or (eight waves,
  // whose registers are all taken) i even and odd apart
  constexpr int NS = TS == 1 ? 4 : 2;
  Acc st[RT][NS];
  auto clear_sums = [&]() {
#pragma unroll
    for (int mt = 0; mt < RT; ++mt)
#pragma unroll
      for (int i = 0; i < NS; ++i) st[mt][i] = acc_empty();
  };
  clear_sums();
  auto flush = [&](int oo) {
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
      Acc s = acc_sum(st[mt][0], st[mt][1]);
      if constexpr (NS == 4) s = acc_sum(s, acc_sum(st[mt][2], st[mt][3]));
      s = sum_groups(s);
      if (lane < 16) sm.part[half][oo][row0 + 16 * mt] = s;
    }
    clear_sums();
  };
  auto mm = [&](const u32x4 &a, const u32x4 &b, f32x4 c) {
    if constexpr (HF)
      return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                    0, 0);
    else
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                     0, 0, 0);
  };
  // two accumulator sets: one takes the tile in hand, the other waits for its
  // epilogue, with sigma^2 and (fp16 form) the scales of its tile's models
  f32x4 qa[2][RT], ya[2][RT], s2[2], qs[2], ys[2];
  f32x4 ql[2][RT], yl[2][RT];
  auto clear_pending = [&](auto PI) {
    constexpr int p = decltype(PI)::value;
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
      qa[p][mt] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      ya[p][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      ql[p][mt] = ya[p][mt];
      yl[p][mt] = ya[p][mt];
    }
    s2[p] = f32x4{0.f, 0.f, 0.f, 0.f};
    qs[p] = f32x4{1.f, 1.f, 1.f, 1.f};
    ys[p] = qs[p];
  };
  // The epilogue of element (row tile el % RT, model el / RT of the lane's four)
  // in three steps, placed in consecutive slots so that none waits for the one
  // before: A the exponential (and the models' and rows' powers of two undone,
  // exactly, when SC), B and C the sums.
  float ea[4 * RT], ee[4 * RT], ed[4 * RT];   // activation, weight, prediction difference (live for two slots)
  auto epi_a = [&](auto PI, auto SC, int el) {
    constexpr int p = decltype(PI)::value;
    constexpr bool sc = decltype(SC)::value;
    const int mt = el % RT, i = el / RT;
    const float qv = TWO ? qa[p][mt][i] + ql[p][mt][i] : qa[p][mt][i];
    const float yv = TWO ? ya[p][mt][i] + yl[p][mt][i] : ya[p][mt][i];
    ea[el] = sc ? qv * (qs[p][i] * rsc[mt]) : qv;
    ed[el] = sc ? yv * (ys[p][i] * rsc[mt]) : yv;
    // bare v_exp_f32: arguments below -126 (weights under 2^-126 next to a
    // largest term of at least 2^-100) need none of exp2f's denormal scaling
    ee[el] = __builtin_amdgcn_exp2f(ea[el]);
  };
  float et[4 * RT];
  auto epi_b = [&](int el) {
    const int mt = el % RT, i = el / RT;
    et[el] = ee[el] * ed[el];
    st[mt][i % NS].Z += ee[el];
    st[mt][0].mx = fmaxf(st[mt][0].mx, ea[el]);   // one running max per row
  };
  auto epi_c = [&](auto PI, int el) {
    constexpr int p = decltype(PI)::value;
    const int mt = el % RT, i = el / RT;
    Acc &t = st[mt][i % NS];
    t.S1 += et[el];
    t.S2 = fmaf(et[el], ed[el], t.S2);
    t.S3 = fmaf(ee[el], s2[p][i], t.S3);
  };
  auto epi_all = [&](auto PI, auto SC) {
#pragma unroll
    for (int el = 0; el < 4 * RT; ++el) {
      epi_a(PI, SC, el);
      epi_b(el);
      epi_c(PI, el);
    }
  };
  // The tile's six blocks of model pieces go through a ring of three blocks in
  // registers, each read from LDS two blocks (12 products) ahead.
  u32x4 wb[3][NPU];
  auto ldb = [&](const u32x4(*W)[64], int kb) {
#pragma unroll
    for (int p = 0; p < NPU; ++p) wb[kb % 3][p] = W[kb * NPU + p][lane];
  };
  int o = 0, nb = 0;
  // the products of one tile (piece chunks W) into set c, the epilogue of the
  // tile before from set p, (LD) the loads of stage st_ld into ring stage
  // `ring_ld`, and (NEXT) the first blocks of the next tile (Wn); PRE: this
  // tile's were read so
  auto body = [&](int tile, const u32x4(*W)[64], const u32x4(*Wn)[64], int st_ld, int ring_ld, auto LD, auto PRE,
                  auto NEXT, auto CI, auto PI, auto SC) {
    constexpr int c = decltype(CI)::value;
    if constexpr (!decltype(PRE)::value) {
      ldb(W, 0);
      ldb(W, 1);
    }
    if (tile >= nb) {
      if (nb > 0) {
        epi_all(PI, SC);
        clear_pending(PI);
        flush(o);
      }
      locate(tile, o, nb);
      set_anchor(o);
    }
    constexpr int NPR = NPU * (NPU + 1) / 2;
    constexpr int PA[6] = {0, 0, 1, 0, 1, 2}, PB[6] = {0, 1, 0, 2, 1, 0};
    // slot: one product of each row tile (the chains alternate; piece pairs
    // (model, sample) bf16 hh, hm, mh, hl, mm, lh; fp16 hh, hl, lh) and about
    // four vector operations of the pending epilogue
    auto slot = [&](auto SI) {
      constexpr int sl = decltype(SI)::value, kb = sl / NPR, r = sl % NPR;
      // the wave further behind in its tile goes first: left to age order, the
      // older of the two waves of a SIMD would finish its tile early and leave
      // the other to run alone
      constexpr int kQuarter = (kBfNKB * NPR + 3) / 4;
      if constexpr (NW == 8 && sl % kQuarter == 0) __builtin_amdgcn_s_setprio(3 - sl / kQuarter);
      if constexpr (r == 0) {
        if constexpr (kb + 2 < kBfNKB)
          ldb(W, kb + 2);
        else if constexpr (decltype(NEXT)::value)
          ldb(Wn, kb + 2 - kBfNKB);
      }
      if constexpr (sl == 0) {   // for the epilogue, one tile later
        s2[c] = buffer_f32x4(srs, 16 * (lane >> 4), tile * kMetaBytes);
        if constexpr (decltype(SC)::value) {   // the models' scales 2^eq, 2^ey
          qs[c] = buffer_f32x4(srs, 16 * (lane >> 4) + 64, tile * kMetaBytes);
          ys[c] = buffer_f32x4(srs, 16 * (lane >> 4) + 128, tile * kMetaBytes);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mt = 0; mt < RT; ++mt) {
        constexpr bool low = TWO && r > 0;
        f32x4 &x = kb < kBfNKQ ? (low ? ql[c][mt] : qa[c][mt]) : (low ? yl[c][mt] : ya[c][mt]);
        x = mm(wb[kb % 3][PA[r]], Bs[mt][kb][PB[r]],
               r == (low ? 1 : 0) && (kb == 0 || kb == kBfNKQ) ? f32x4{0.f, 0.f, 0.f, 0.f} : x);
      }
      // the epilogue's steps in order: 2 el is A of element el and C of the one
      // before, 2 el + 1 its B; one step per slot where the slots suffice
      constexpr int kSteps = 8 * RT + 1, kPer = (kSteps + kBfNKB * NPR - 1) / (kBfNKB * NPR);
#pragma unroll
      for (int es = sl * kPer; es < (sl + 1) * kPer && es < kSteps; ++es) {
        if (es & 1) {
          epi_b(es / 2);
        } else {
          if (es / 2 < 4 * RT) epi_a(PI, SC, es / 2);
          if (es > 0) epi_c(PI, es / 2 - 1);
        }
      }
      // a memory load each: all at once they would hold every wave up
      if constexpr (decltype(LD)::value && sl % 2 == 1 && sl / 2 < kLoads) issue(st_ld, ring_ld, sl / 2);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_for<0, kBfNKB * NPR>(slot);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using Yes = std::true_type;
  using Cross = std::integral_constant<bool, XB>;
  auto enter = [&]() {
    // this wave's loads are complete (all, or all but the latest stage's); no
    // memory access moves across the barrier (compiler fences on both sides)
    __builtin_amdgcn_s_waitcnt(XB ? 0x0F70 : 0x0F70 | kLoads);   // vmcnt(0 or kLoads), expcnt and lgkmcnt untouched
    __asm__ __volatile__("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    __asm__ __volatile__("" ::: "memory");
  };
  auto run = [&](auto SC) {
    auto W = [&](int ring, int u) { return (const u32x4(*)[64]) & sm.ring[ring][u * kChunks]; };
    auto next = [&](int r) { return r + 1 == NSTG ? 0 : r + 1; };
    clear_pending(I1{});
    enter();
    if constexpr (XB) {
      ldb(W(0, half), 0);
      ldb(W(0, half), 1);
    }
    int ring = 0, done = 0;   // ring stage of the stage in hand; tiles this wave has run
    // one stage: the loads go to the stage whose ring slots the last barrier freed
    auto stage = [&](int st_i, auto CI, auto PI) {
      const int r1 = next(ring), rl = next(r1), sl = st_i + 2;
      if constexpr (TS == 2) {
        if (2 * st_i + half < n) {
          body(T0 + 2 * st_i + half, W(ring, half), W(r1, half), sl, rl, Yes{}, Cross{}, Cross{}, CI, PI, SC);
          ++done;
        }
      } else {
        body(T0 + 2 * st_i, W(ring, 0), W(ring, 1), sl, rl, Yes{}, Cross{}, Yes{}, CI, PI, SC);
        ++done;
        if (2 * st_i + 1 < n) {
          body(T0 + 2 * st_i + 1, W(ring, 1), W(r1, 0), n_st, rl, std::false_type{}, Yes{}, Cross{}, PI, CI, SC);
          ++done;
        }
      }
      ring = r1;
    };
    for (int st_i = 0; st_i < n_st;) {
      stage(st_i, I0{}, I1{});
      if (++st_i >= n_st) break;
      enter();
      if constexpr (TS == 2) {
        stage(st_i, I1{}, I0{});
        if (++st_i >= n_st) break;
        enter();
      }
    }
    // loads past the last stage must not land in the next evaluation's ring
    __builtin_amdgcn_s_waitcnt(0x0F70);
    if (done > 0) {
      if (done & 1)
        epi_all(I0{}, SC);
      else
        epi_all(I1{}, SC);
      flush(o);
    }
  };
  // Whether any power of two has to be undone: the wave's rows' (rarely) or
  // some model's (the models' scales are all 1 unless their values are far
  // from 1); products with a scale of 1 are exact, so both loops agree.
  bool scaled = false;
  if constexpr (HF)
    scaled = sm.model_scaled != 0 || __builtin_amdgcn_ballot_w64(rsc[0] != 1.0f || rsc[RT - 1] != 1.0f) != 0;
  if (HF && scaled)
    run(std::true_type{});
  else
    run(std::false_type{});
}

// Sampling of the next-state draw inside the mixture's last stage: with xi
// set, acc = mu + sqrt(var) xi[row][o] (a draw from N(mu, var)); without, mu.
struct SampleArgs {
  const float *xi;   // [rows][MixSmem::XIS] standard normals of this step, or null
  // optional per-step trace of the adjoint: for row r < trace_rows and output
  // o, trace[r * trace_stride + trace_off + 5 o + {0..4}] = (d1, var, log2 Z,
  // m, yref) of the evaluation's final pass: the activation anchor m and the
  // prediction reference yref it used, its normaliser Z = sum_j 2^(a_j) with
  // a_j = -q_j log2(e) / 2 - m, and d1 = mu - yref.  A reverse sweep that
  // contracts with the same anchors reproduces every a_j and y_j - yref
  // bitwise, so its weights 2^(a_j - log2 Z) are the forward's.
  float *trace = nullptr;
  int64_t trace_stride = 0;
  int trace_off = 0, trace_rows = 0;
  // optional moments (prediction): mean[row * n_out + o], var[...] of rows < moment_rows;
  // full: the pass takes every piece (mprev of a row and output then holds whether its
  // sums were usable)
  float *mean = nullptr, *var = nullptr;
  int moment_rows = 0, n_out = 0;
  bool full = true;
};

// Eq. (1) moments of one (row, output) from its complete sums, the sampled
// acceleration, the anchors of the next evaluation (observed maximum and
// mean), and the redo flag of evaluation `ev` when the sums are not usable
// (one overflowed, or the largest term came near the denormal range).
template <int D, int MT, int NW, int PF>
__device__ __forceinline__ void finish_sums(MixSmem<D, MT, NW, PF> &sm, int row, int o, const Acc &s, uint32_t ev,
                                            const SampleArgs &sa) {
  const float d1 = s.S1 / s.Z;
  const float mu = sm.yref[row][o] + d1;
  const float var = (fmaxf(s.S2 - s.S1 * d1, 0.f) + s.S3) / s.Z;
  if (sa.mean && row < sa.moment_rows) {
    sa.mean[row * sa.n_out + o] = mu;
    sa.var[row * sa.n_out + o] = var;
  }
  // the anchor in use is m (base-2 units): sum_j exp(-q_j/2) = 2^m Z.  A
  // redo pass rewrites the trace, so it ends with the final pass's values.
  if (sa.trace && row < sa.trace_rows) {
    float *dst = sa.trace + row * sa.trace_stride + sa.trace_off + 5 * o;
    dst[0] = d1;
    dst[1] = var;
    dst[2] = log2f(s.Z);
    dst[3] = sm.mref[row][o];
    dst[4] = sm.yref[row][o];
  }
  sm.accel(row, o) = sa.xi ? mu + sqrtf(var) * sa.xi[row * MixSmem<D, MT, NW, PF>::XIS + o] : mu;
  const bool valid = isfinite(s.Z) && isfinite(s.S1) && isfinite(s.S2) && isfinite(s.S3) && s.mx >= kAnchorLo;
  if (sa.mean) {
    // a prediction's reference far from its mean (a coarse pass, far inputs) costs
    // the variance its digits: 2^-24 d1^2 beside var.  A reference that is the mean of
    // a full pass is as near as rounding lets it (the variance may be 0), and sums that
    // no anchor or reference makes finite stay what they are.
    const bool off = d1 * d1 > 4.0f * var && sm.mprev[row][o] == 0.0f;
    const bool lost = isnan(s.Z) || (isfinite(s.Z) && s.mx >= kAnchorLo && !isfinite(mu));
    if ((!valid || off) && !lost && row < sa.moment_rows) sm.redo[ev & 1] = 1;
    sm.mprev[row][o] = sa.full && valid ? 1.0f : 0.0f;
  } else if (!valid) {
    sm.redo[ev & 1] = 1;
  }
  sm.mref[row][o] += s.mx;
  if (isfinite(mu)) sm.yref[row][o] = mu;
}


template <int D, int MT, int NW, int PF>
__device__ __forceinline__ Acc sum_waves(const MixSmem<D, MT, NW, PF> &sm, int row, int o) {
  Acc s = sm.part[0][o][row];
#pragma unroll
  for (int w = 1; w < MixSmem<D, MT, NW, PF>::NPART; ++w) s = acc_sum(s, sm.part[w][o][row]);
  return s;
}

// Stage 3 (lanes < ROWS * n_out): fixed-order sums over waves, then the
// moments.
template <int D, int MT, int NW, int PF>
__device__ __forceinline__ void merge_waves(MixSmem<D, MT, NW, PF> &sm, int n_out, uint32_t ev, const SampleArgs &sa) {
  constexpr int ROWS = MixSmem<D, MT, NW, PF>::ROWS;
  for (int i = threadIdx.x; i < ROWS * n_out; i += NW * 64) {
    const int row = i % ROWS, o = i / ROWS;
    finish_sums(sm, row, o, sum_waves(sm, row, o), ev, sa);
  }
}

// Paired workgroups: two workgroups (on two compute units) hold the same rows
// and each runs half of the model tiles.  After its own wave sums, each
// publishes them, waits for the partner's, and both add the two halves in
// the same order (half 0 + half 1), so both hold bit-identical moments and
// take the same redo decision.
//
// Protocol per evaluation (sequence number seq >= 1, slots double-buffered by
// parity): every published sum travels in a 64-bit word (sequence number in
// the high half, the float's bits in the low half) written with an
// agent-scope relaxed atomic store; the lane that needs the partner's word
// polls it with agent-scope loads until its sequence number is seq.  Aligned
// 64-bit accesses are single-copy atomic, so a word carrying seq carries
// this evaluation's value: no flag, fence or barrier orders the data.  A slot
// is rewritten two evaluations later, which the partner can only reach after
// every one of our lanes has read it (it needs our next evaluation's words,
// published after a barrier that follows the reads).  The slots are zeroed
// before each launch.  Every wait is bounded: on running out, pair_fail is
// set, no further waits are made and the rollout's costs are written as NaN
// from then on.  A workgroup that has given up no longer holds valid state,
// so every word it publishes afterwards carries the poison sequence number
// instead of a valid one; a partner that reads a poisoned word gives up too.
// Each workgroup that gave up is counted in pair_give_ups_total.
struct PairCtx {
  uint64_t *xbuf;       // the pair's slots: [half][parity][5][kXSlots] (sums Z, S1, S2, S3, mx)
  int half;             // 0 or 1; -1 when not paired
  uint32_t spin_limit;  // polls of one wait before giving up
};
__device__ __forceinline__ bool writer_of(const PairCtx *pc) { return pc == nullptr || pc->half == 0; }
constexpr int kXSlots = 16 * kMaxOut;
constexpr int kPairWords = 2 * 2 * kXSlots * 5;
constexpr uint32_t kSpinLimit = 1u << 20;
// Sequence number of the words of a workgroup that has given up; valid ones
// run from 1 to twice the horizon, far below it.
constexpr uint32_t kPoisonSeq = 0xFFFFFFFFu;
// Workgroups of paired launches on this device that gave up a wait, since load.
__device__ unsigned long long pair_give_ups_total = 0;

__device__ __forceinline__ void put_word(uint64_t *p, float v, uint32_t seq) {
  __hip_atomic_store(p, ((uint64_t)seq << 32) | (uint64_t)__float_as_uint(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

template <int D, int MT, int NW, int PF>
__device__ __forceinline__ void merge_pair(MixSmem<D, MT, NW, PF> &sm, int n_out, const PairCtx &pc, uint32_t seq,
                                           const SampleArgs &sa) {
  static_assert(MT == 1, "paired workgroups hold one 16-row tile");
  constexpr int ROWS = 16;
  const int i = threadIdx.x;
  if (i >= ROWS * n_out) return;
  const int row = i % ROWS, o = i / ROWS;
  const Acc loc = sum_waves(sm, row, o);
  // consecutive lanes write consecutive words of each sum
  uint64_t *dst = pc.xbuf + (size_t)(pc.half * 2 + (seq & 1)) * 5 * kXSlots + i;
  // pair_fail is read after the barrier that closed the previous evaluation:
  // every lane agrees whether this workgroup's state is still valid
  const uint32_t tag = sm.pair_fail ? kPoisonSeq : seq;
  put_word(dst + 0 * kXSlots, loc.Z, tag);
  put_word(dst + 1 * kXSlots, loc.S1, tag);
  put_word(dst + 2 * kXSlots, loc.S2, tag);
  put_word(dst + 3 * kXSlots, loc.S3, tag);
  put_word(dst + 4 * kXSlots, loc.mx, tag);
  const uint64_t *src = pc.xbuf + (size_t)((1 - pc.half) * 2 + (seq & 1)) * 5 * kXSlots + i;
  uint64_t w[5];
  uint32_t n = 0;
  for (;;) {
    bool ready = true, poisoned = false;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      w[k] = __hip_atomic_load(src + k * kXSlots, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ready = ready && (uint32_t)(w[k] >> 32) == seq;
      poisoned = poisoned || (uint32_t)(w[k] >> 32) == kPoisonSeq;
    }
    if (ready) break;
    if (poisoned || sm.pair_fail || ++n >= pc.spin_limit) {
      sm.pair_fail = 1;
      break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  Acc rem;
  rem.Z = __uint_as_float((uint32_t)w[0]);
  rem.S1 = __uint_as_float((uint32_t)w[1]);
  rem.S2 = __uint_as_float((uint32_t)w[2]);
  rem.S3 = __uint_as_float((uint32_t)w[3]);
  rem.mx = __uint_as_float((uint32_t)w[4]);
  finish_sums(sm, row, o, pc.half == 0 ? acc_sum(loc, rem) : acc_sum(rem, loc), seq, sa);
}

// The whole mixture of one step for the rows in sm.z over model tiles
// [T0, T1): one pass, a second one if an anchor was out of range or
// `force_second`.  Block-synchronous.  seq counts the evaluations (it numbers
// the pair exchanges and selects the redo flag, double-buffered so that one
// barrier per evaluation suffices); with a pair context the two halves' sums
// are exchanged every pass.
template <int D, int MT, int NW, int PF>
__device__ __forceinline__ void mixture_step(const MfmaModel &md, MixSmem<D, MT, NW, PF> &sm, bool force_second,
                                             int T0, int T1, const PairCtx *pc, uint32_t &seq,
                                             const SampleArgs &sa = SampleArgs{nullptr}) {
  for (int pass = 0; pass < 2; ++pass) {
    build_fragments(sm);
    clear_parts(sm);
    __syncthreads();
    if constexpr (MixSmem<D, MT, NW, PF>::SH)
      mixture_tiles_sh(md, sm, T0, T1);
    else if constexpr (PF != kPfF32)
      mixture_tiles_bf(md, sm, T0, T1);
    else
      mixture_tiles(md, sm, T0, T1);
    __syncthreads();
    const uint32_t ev = ++seq;
    if constexpr (MT == 1) {
      if (pc != nullptr) {
        merge_pair(sm, md.n_out, *pc, ev, sa);
      } else {
        merge_waves(sm, md.n_out, ev, sa);
      }
    } else {
      merge_waves(sm, md.n_out, ev, sa);
    }
    __syncthreads();
    const bool again = pass == 0 && (force_second || sm.redo[ev & 1] != 0);
    // the next evaluation's flag: last read before this evaluation's barriers
    if (threadIdx.x == 0) sm.redo[(ev + 1) & 1] = 0;
    if (!again) {
      // Anchor of the next step: the largest activation moves smoothly along a
      // trajectory (it drifts steadily once the state leaves the models'
      // support), so extrapolate it linearly from the last two steps; the
      // lanes that merged each (row, output) own its entries.
      constexpr int ROWS = MixSmem<D, MT, NW, PF>::ROWS;
      for (int i = threadIdx.x; i < ROWS * md.n_out; i += NW * 64) {
        const int row = i % ROWS, o = i / ROWS;
        const float M = sm.mref[row][o];
        const float d = force_second ? 0.f : M - sm.mprev[row][o];
        sm.mprev[row][o] = M;
        if (isfinite(d)) sm.mref[row][o] = M + d;
      }
      break;
    }
  }
}

template <int D, int MT, int NW, int PF>
__device__ __forceinline__ void reset_anchors(MixSmem<D, MT, NW, PF> &sm) {
  for (int i = threadIdx.x; i < MixSmem<D, MT, NW, PF>::ROWS * MixSmem<D, MT, NW, PF>::NOUT; i += NW * 64) {
    (&sm.mref[0][0])[i] = 0.0f;
    (&sm.yref[0][0])[i] = 0.0f;
    (&sm.mprev[0][0])[i] = 0.0f;
  }
}

// --------------------------------------------------------------- predict
// 16 MT inputs per workgroup.  Float32 products: two passes, the second with
// the first one's largest activations as anchors and its means as references.
// bf16 pieces (d = 16): the first pass takes the leading piece alone, a sixth of
// the products -- an anchor within 100 units of the largest activation and a
// reference within two standard deviations of the mean are all it has to give --
// and the second all three; a third follows where the reference was out of that
// range, a fourth where the anchor was (inputs far from every model).  Bound: the matrix pipe (42 bf16 products per 16 x 16
// block against 88 float32 ones of twice the length); 100003 inputs, 6 x 256
// models: 0.36 ms, 0.94 ms in two float32 passes of 16-row workgroups.
template <int D, int MT, int NW, int PF>
__global__ void __launch_bounds__(NW * 64) predict_mfma_kernel(MfmaModel md, const float *__restrict__ Z,
                                                               int64_t n_base, int64_t N, float *__restrict__ mean,
                                                               float *__restrict__ var) {
  using SM = MixSmem<D, MT, NW, PF>;
  __shared__ SM sm;
  constexpr int ROWS = SM::ROWS;
  mix_setup(sm);
  reset_anchors(sm);
  const int64_t n0 = n_base + (int64_t)blockIdx.x * ROWS;
  for (int i = threadIdx.x; i < ROWS * (D + 2); i += NW * 64) {
    const int row = i / (D + 2), a = i % (D + 2);
    sm.z[row][a] = a < D ? ((n0 + row < N) ? Z[(n0 + row) * D + a] : 0.0f) : (a == D ? 1.0f : 0.0f);
  }
  __syncthreads();
  SampleArgs sa{nullptr};
  sa.mean = mean + n0 * md.n_out;
  sa.var = var + n0 * md.n_out;
  sa.moment_rows = (int)min<int64_t>(ROWS, N - n0);
  sa.n_out = md.n_out;
  uint32_t seq = 0;
  if constexpr (PF == kPfF32) {
    mixture_step(md, sm, true, 0, md.n_tiles, (const PairCtx *)nullptr, seq, sa);
  } else {
    build_fragments(sm);
    for (int pass = 0; pass < 4; ++pass) {
      clear_parts(sm);
      if (threadIdx.x == 0) sm.redo[0] = sm.redo[1] = 0;
      __syncthreads();
      if constexpr (SM::SH) {
        if (pass == 0)
          mixture_tiles_sh<D, MT, NW, PF, 1>(md, sm, 0, md.n_tiles);
        else
          mixture_tiles_sh<D, MT, NW, PF, SM::NPC, true>(md, sm, 0, md.n_tiles);
      } else {
        if (pass == 0)
          mixture_tiles_bf<D, MT, NW, PF, 1>(md, sm, 0, md.n_tiles);
        else
          mixture_tiles_bf<D, MT, NW, PF, SM::NPC, true>(md, sm, 0, md.n_tiles);
      }
      __syncthreads();
      sa.full = pass > 0;
      merge_waves(sm, md.n_out, 0u, sa);
      __syncthreads();
      if (pass > 0 && sm.redo[0] == 0) break;
      __syncthreads();   // every lane has read the flag
    }
  }
}

template <int D, int MT, int NW, int PF>
static hipError_t predict_mfma_t(const MfmaModel &md, const float *Z, int64_t n_base, int64_t N, float *mean,
                                 float *var, hipStream_t s) {
  const int64_t nb = (N - n_base + 16 * MT - 1) / (16 * MT);
  hipLaunchKernelGGL((predict_mfma_kernel<D, MT, NW, PF>), dim3((unsigned)nb), dim3(NW * 64), 0, s, md, Z, n_base, N,
                     mean, var);
  return hipGetLastError();
}

// pieces: the bf16 form (d = 16).  Whole passes of 128-row workgroups over 256
// compute units first (139 us for 32768 inputs, 6 x 256 models); the rest in the
// tile with the fewest passes times their cost (microseconds per pass for t
// model tiles: 16 rows 2 + 0.22 t, 32 rows 7 + 0.29 t, 128 rows 15 + 0.85 t;
// 16384 inputs: 96 us in 32-row tiles, 139 in 128-row ones, and the float32
// form 160).
hipError_t launch_predict_mfma(const ModelArgs &m, const MfmaLayout &l, const void *base, const void *Z, int64_t N,
                               void *mean, void *var, bool pieces, hipStream_t s) {
  if (N == 0) return hipSuccess;
  const MfmaModel md = mfma_view(l, base);
  const float *z = (const float *)Z;
  float *mn = (float *)mean, *vr = (float *)var;
  if (m.d == 16 && pieces && md.Wb != nullptr) {
    constexpr int64_t kPass = 128 * 256;
    const bool sh = m.n_out <= 6;   // outputs per row the shared tile holds
    const double t = l.n_tiles;
    int64_t n0 = 0;
    hipError_t e = hipSuccess;
    const int64_t rest = sh ? N % kPass : N;
    const double t16 = (double)((rest + 4095) / 4096) * (2 + 0.22 * t), t32 = (double)((rest + 8191) / 8192) * (7 + 0.29 * t);
    const double t128 = sh ? 15 + 0.85 * t : 1e30;
    const bool tail128 = rest > 0 && t128 < t16 && t128 < t32;
    const int64_t n128 = sh ? (tail128 ? N : N - rest) : 0;
    if (n128 > 0) {
      e = predict_mfma_t<16, 8, 8, kPfBf16x3>(md, z, 0, n128, mn, vr, s);
      n0 = n128;
    }
    if (e != hipSuccess || n0 == N) return e;
    return t16 <= t32 ? predict_mfma_t<16, 1, 4, kPfBf16x3>(md, z, n0, N, mn, vr, s)
                      : predict_mfma_t<16, 2, 4, kPfBf16x3>(md, z, n0, N, mn, vr, s);
  }
  if (m.d == 16) return predict_mfma_t<16, 1, 4, kPfF32>(md, z, 0, N, mn, vr, s);
  if (m.d == 6) return predict_mfma_t<6, 1, 4, kPfF32>(md, z, 0, N, mn, vr, s);
  if (m.d == 4) return predict_mfma_t<4, 1, 4, kPfF32>(md, z, 0, N, mn, vr, s);
  return hipErrorInvalidValue;
}

// --------------------------------------------------------------- rollout
template <int DYN>
struct Dims;
template <>
struct Dims<kDynPointMass2D> {
  static constexpr int NX = 4, NU = 2, NO = 2, D = 6;
};
template <>
struct Dims<kDynQuad12> {
  static constexpr int NX = 12, NU = 4, NO = 6, D = 16;
};
template <>
struct Dims<kDynQuadHybrid> {
  static constexpr int NX = 9, NU = 4, NO = 3, D = 4;
};

constexpr int kNoiseChunk = 16;   // steps of noise drawn ahead into LDS

template <int DYN, int MT, int NW, int PF = 0>
struct RollSmem {
  static constexpr int ROWS = 16 * MT;
  // steps per noise chunk, and whether the costs wait for the end of the chunk
  // too: the shared-tile form, whose LDS holds the tile ring, draws four steps
  // ahead (one where the ring fills it: 128 rows of bf16 pieces) and evaluates
  // each step's costs at once, four lanes to a row
  static constexpr bool SH = MixSmem<Dims<DYN>::D, MT, NW, PF>::SH;
  static constexpr int CH = !SH ? kNoiseChunk : PF == kPfBf16x3 && MT == 8 ? 1 : 4;
  MixSmem<Dims<DYN>::D, MT, NW, PF> sm;
  // the state and its compensation (euler_step_comp): up to 0.8 % of a step with a lane
  // per row, nothing measurable with 16, and an eighth of the float32 batch's error
  // after an update
  float xs[ROWS][Dims<DYN>::NX], xlo[ROWS][Dims<DYN>::NX];
  float us_s[CH][ROWS][4];           // applied controls u_nom + sigma eps of the chunk
  float xi_s[CH][ROWS][MixSmem<Dims<DYN>::D, MT, NW, PF>::XIS];
  // x_{t+1} of the chunk's steps, for the costs (the shared-tile form: xs)
  std::conditional_t<SH, char[16], float[CH][ROWS][Dims<DYN>::NX]> xc;
  float obs_s[kMaxObs * 3];
  // the batched kernel's work item: here, so that the kernel has one LDS object
  // (with two the compiler waits for every load to LDS in flight before each
  // LDS read: 16 controllers 42.2 against 34.4 ms)
  int item;
};

// Rollouts s_base .. s_base + spw - 1 of one problem for its whole horizon.
// Every CH steps (RollSmem::CH) all lanes draw the chunk's eps and xi, store the
// applied controls u_nom + sigma eps in LDS (no global read is left on the
// per-step critical section) and evaluate the previous chunk's step costs
// dt*q(x_{t+1}) from the states kept in LDS (the cost feeds nothing on the
// path, so it leaves the per-step critical section too; the shared tile, which
// has no room for them, evaluates each step's).  Per step: rows form z, the waves
// run the model tiles, partial sums are merged and the accelerations sampled, and
// the rows step Euler.  Block-synchronous; rs.sm must have been set up.  With a pair
// context (pc->half = 0 or 1) the workgroup runs its half of the model tiles,
// exchanges sums with its partner, and only half 0 writes costs.
// The steps a rollout tile runs and what it keeps besides the costs (see
// RolloutArgs): the whole horizon from x0 unless the adjoint's checkpointed
// forward asks for a segment or for checkpoints.
struct RollSeg {
  int tb, te, trace_T, ckpt;
  const float *xstart;
  float *ckpt_out;
};
__device__ __forceinline__ RollSeg roll_seg(const RolloutArgs<float> &ra) {
  return RollSeg{ra.t_begin, ra.t_end < 0 ? ra.p.T : ra.t_end, ra.trace_T < 0 ? ra.p.T : ra.trace_T, ra.ckpt,
                 ra.xstart, ra.ckpt_out};
}

template <int DYN, int MT, int NW, int PF>
__device__ void rollout_tile(RollSmem<DYN, MT, NW, PF> &rs, const ProbDev<float> &p,
                             const float *__restrict__ x0, const float *__restrict__ u_nom,
                             uint32_t it, float *__restrict__ cost, const MfmaModel &md,
                             int64_t s_base, int spw, const PairCtx *pc = nullptr, float *tr = nullptr,
                             const RollSeg *sg = nullptr) {
  using DD = Dims<DYN>;
  constexpr int D = DD::D, NX = DD::NX, NU = DD::NU, NO = DD::NO;
  constexpr int ROWS = 16 * MT;
  constexpr int CH = RollSmem<DYN, MT, NW, PF>::CH;
  constexpr bool SH = RollSmem<DYN, MT, NW, PF>::SH;
  MixSmem<D, MT, NW, PF> &sm = rs.sm;
  constexpr int SEGW = NX + 5 * NO;   // trace row: x_t, then 5 values per output (SampleArgs)
  // the shared tile runs whole horizons from x0 and keeps nothing besides the costs
  if constexpr (SH) {
    sg = nullptr;
    tr = nullptr;
  }
  const int tb = sg ? sg->tb : 0, te = sg ? sg->te : p.T;
  const int ck = sg ? sg->ckpt : 0;
  const int nck = ck > 0 ? (p.T + ck - 1) / ck : 0;
  float *ckpt_out = sg ? sg->ckpt_out : nullptr;
  const int64_t tstride = (int64_t)((sg ? sg->trace_T : p.T) + 1) * SEGW;
  float *trace = writer_of(pc) && tr ? tr + s_base * tstride : nullptr;
  const int trows = (int)min<int64_t>(spw, (int64_t)p.K * p.Ms - s_base);
  const int T0 = pc == nullptr || pc->half == 0 ? 0 : md.n_tiles / 2;
  const int T1 = pc == nullptr || pc->half == 1 ? md.n_tiles : md.n_tiles / 2;
  const bool writer = writer_of(pc);
  uint32_t seq = 0;
  __syncthreads();  // the previous tile (persistent use) is done with LDS
  reset_anchors(sm);
  if constexpr (MixSmem<D, MT, NW, PF>::SH && PF == kPfF16x2) {
    // some model of the problem carries powers of two
    if (threadIdx.x == 0) sm.model_scaled = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < md.n_tiles; i += NW * 64)
      if (md.hmeta[(size_t)i * kHfMeta + kHfPlain] == 0.0f) sm.model_scaled = 1;
  }
  const int row = threadIdx.x;
  const int64_t s = s_base + row;
  const bool active = row < spw && s < (int64_t)p.K * p.Ms;
  const uint32_t wc = stream_word(kTagCtrl, p.problem_id, it);
  const uint32_t wd = stream_word(kTagDyn, p.problem_id, it);
  if (row < ROWS) {
    const bool seg = sg && sg->xstart && active;
    const float *xs0 = seg ? sg->xstart + (s * nck + tb / ck) * (2 * NX) : x0;
    for (int a = 0; a < NX; ++a) {
      rs.xs[row][a] = xs0[a];
      rs.xlo[row][a] = seg ? xs0[NX + a] : 0.0f;
    }
    sm.z[row][D] = 1.0f;
    sm.z[row][D + 1] = 0.0f;
  }
  for (int i = threadIdx.x; i < 3 * p.n_obs; i += NW * 64) rs.obs_s[i] = p.obs[i];
  // costs of steps t0 .. t0+n-1 from rs.xc, one (row, step) per lane, runs of
  // consecutive steps per row so the stores coalesce
  auto flush_costs = [&](int t0, int n) {
    if (!writer || cost == nullptr) return;
    if constexpr (SH) {
      // the step's costs from rs.xs, the obstacles of a row over four lanes
      for (int i = threadIdx.x; i < ROWS * 4; i += NW * 64) {
        const int rr = i >> 2, q = i & 3;
        const float c = state_cost_quad<float, DYN>(p, rs.obs_s, rs.xs[rr], q);
        const int64_t ss = s_base + rr;
        if (q == 0 && rr < spw && ss < (int64_t)p.K * p.Ms) cost[ss * p.T + t0] = p.dt * c;
      }
    } else {
    const bool failed = sm.pair_fail != 0;
    for (int i = threadIdx.x; i < ROWS * n; i += NW * 64) {
      const int rr = i / n, cc = i - rr * n;
      const int64_t ss = s_base + rr;
      if (rr >= spw || ss >= (int64_t)p.K * p.Ms) continue;
      float c = p.dt * state_cost<float>(p, rs.obs_s, rs.xc[cc][rr]);
      if constexpr (DYN == kDynQuadHybrid)
        if (p.ctrl_cost) c += rs.xi_s[cc][rr][7];
      cost[ss * p.T + t0 + cc] = failed ? __builtin_nanf("") : c;
    }
    }
  };
  for (int t = tb; t < te; ++t) {
    const int tc = (t - tb) % CH;
    if (SH && t > tb) {
      __syncthreads();  // the step's states are in rs.xs
      flush_costs(t - 1, 1);
    }
    if (tc == 0) {
      if (t > tb && !SH) {
        __syncthreads();  // the chunk's states are in rs.xc
        flush_costs(t - CH, CH);
        // the control terms of the flushed chunk are read from the draw slots
        // the next chunk overwrites
        if (DYN == kDynQuadHybrid && p.ctrl_cost) __syncthreads();
      }
      // draw the next chunk: one lane per (step, row, counter block)
      constexpr int NB = 1 + (NO + 3) / 4;
      for (int i = threadIdx.x; i < CH * ROWS * NB; i += NW * 64) {
        const int blk = i % NB, rr = (i / NB) % ROWS, cc = i / (NB * ROWS);
        const int64_t ss = s_base + rr;
        const bool act = rr < spw && ss < (int64_t)p.K * p.Ms && t + cc < te;
        if (!act) continue;
        // K max(M, 1) < 2^31: the 64-bit division would cost more than the draw
        const uint32_t kk = p.Ms == 1 ? (uint32_t)ss : (uint32_t)ss / (uint32_t)p.Ms;
        const uint32_t mm = (uint32_t)ss - kk * (uint32_t)p.Ms;
        if (blk == 0) {
          float e4[4], pert[NU];
          normals<float, 4>(p.key0, p.key1, wc, kk, 0u, (uint32_t)(t + cc), e4);
#pragma unroll
          for (int a = 0; a < NU; ++a) {
            pert[a] = p.noise_std[a] * e4[a];
            rs.us_s[cc][rr][a] = u_nom[(t + cc) * NU + a] + pert[a];
          }
          // the step's control terms ride in the draw slot the hybrid model leaves unused
          if constexpr (DYN == kDynQuadHybrid)
            if (p.ctrl_cost) rs.xi_s[cc][rr][7] = control_cost<float>(p, u_nom + (t + cc) * NU, pert);
        } else if (p.M > 0) {
          // counter block blk-1 of the sub-rollout's draw: normals 4(blk-1) .. 4(blk-1)+3
          const Philox4 r4 = philox4x32_10((uint32_t)(t + cc), kk, (mm << 4) | (uint32_t)(blk - 1), wd,
                                           p.key0, p.key1);
          float *dst = &rs.xi_s[cc][rr][4 * (blk - 1)];
          float v[4];
          box_muller(r4.v[0], r4.v[1], &v[0], &v[1]);
          box_muller(r4.v[2], r4.v[3], &v[2], &v[3]);
          constexpr int XIS = MixSmem<D, MT, NW, PF>::XIS;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (XIS == 8 || 4 * (blk - 1) + i < XIS) dst[i] = v[i];
        }
      }
      __syncthreads();
    }
    // the applied controls of the row at step t
    auto applied = [&](float (&u)[NU]) {
#pragma unroll
      for (int a = 0; a < NU; ++a) u[a] = rs.us_s[tc][row][a];
    };
    if constexpr (MT > 1) {
      if (row < ROWS) {
        if (active) {
          float u[NU], x[NX], z[D];
          applied(u);
#pragma unroll
          for (int a = 0; a < NX; ++a) x[a] = rs.xs[row][a];
          if (trace) {
#pragma unroll
            for (int a = 0; a < NX; ++a) trace[row * tstride + (int64_t)(t - tb) * SEGW + a] = x[a];
          }
          if (ckpt_out && t % ck == 0) {
            float *dst = ckpt_out + (s * nck + t / ck) * (2 * NX);
#pragma unroll
            for (int a = 0; a < NX; ++a) {
              dst[a] = x[a];
              dst[NX + a] = rs.xlo[row][a];
            }
          }
          lwpr_input<DYN>(x, u, z);
#pragma unroll
          for (int a = 0; a < D; ++a) sm.z[row][a] = z[a];
        } else {
#pragma unroll
          for (int a = 0; a < D; ++a) sm.z[row][a] = 0.0f;
        }
      }
    } else {
      // 16 rows: 16 lanes to each, one component a lane (2048 rollouts x 100 steps of
      // 6 x 256 models 1037 us with a lane per row, 1024 so; 32 rows take two rounds
      // and 1 to 3 % longer)
      for (int i = threadIdx.x; i < ROWS * 16; i += NW * 64) {
        const int rr = i >> 4, l = i & 15;
        const int64_t ss = s_base + rr;
        const bool act = rr < spw && ss < (int64_t)p.K * p.Ms;
        if (l < D) {
          const float z = lwpr_input_at<DYN>(rs.xs[rr], rs.us_s[tc][rr], l);
          sm.z[rr][l] = act ? z : 0.0f;
        }
        if (act && l < NX) {
          if (trace) trace[rr * tstride + (int64_t)(t - tb) * SEGW + l] = rs.xs[rr][l];
          if (ckpt_out && t % ck == 0) {
            float *dst = ckpt_out + (ss * nck + t / ck) * (2 * NX);
            dst[l] = rs.xs[rr][l];
            dst[NX + l] = rs.xlo[rr][l];
          }
        }
      }
    }
    __syncthreads();
    SampleArgs sa{p.M > 0 ? &rs.xi_s[tc][0][0] : nullptr};
    if (trace) {
      sa.trace = trace + (int64_t)(t - tb) * SEGW;
      sa.trace_stride = tstride;
      sa.trace_off = NX;
      sa.trace_rows = trows;
    }
    mixture_step(md, sm, t == tb, T0, T1, pc, seq, sa);
    if constexpr (MT > 1) {
      if (active) {
        float acc[NO], xn[NX], x[NX], lo[NX], u[NU];
#pragma unroll
        for (int o = 0; o < NO; ++o) acc[o] = sm.accel(row, o);
#pragma unroll
        for (int a = 0; a < NX; ++a) {
          x[a] = rs.xs[row][a];
          lo[a] = rs.xlo[row][a];
        }
        applied(u);
        euler_step_comp(DYN, p.dt, x, acc, u, xn, lo);
#pragma unroll
        for (int a = 0; a < NX; ++a) {
          rs.xs[row][a] = xn[a];
          rs.xlo[row][a] = lo[a];
          if constexpr (!SH) rs.xc[tc][row][a] = xn[a];
        }
      }
    } else {
      for (int i = threadIdx.x; i < ROWS * 16; i += NW * 64) {
        const int rr = i >> 4, l = i & 15;
        const bool on = l < NX && rr < spw && s_base + rr < (int64_t)p.K * p.Ms;
        float x = 0.0f, lo = 0.0f;
        if (on) {
          x = rs.xs[rr][l];
          lo = rs.xlo[rr][l];
          euler_lane_comp<DYN>(l, p.dt, rs.xs[rr], rs.us_s[tc][rr], [&](int o) { return sm.accel(rr, o); }, x, lo);
        }
        // a row's lanes are one wave's: their reads are done before their writes
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (on) {
          rs.xs[rr][l] = x;
          rs.xlo[rr][l] = lo;
          rs.xc[tc][rr][l] = x;
        }
      }
    }
  }
  if constexpr (MT == 1) __syncthreads();   // the last states, of other lanes
  if (trace && active) {
#pragma unroll
    for (int a = 0; a < NX; ++a) trace[row * tstride + (int64_t)(te - tb) * SEGW + a] = rs.xs[row][a];
  }
  __syncthreads();
  const int tl = SH ? te - 1 : tb + ((te - tb - 1) / CH) * CH;
  flush_costs(tl, te - tl);
}

// Waves per SIMD the rollout kernels are compiled for: the small-model
// dynamics fit four 4-wave workgroups per compute unit in LDS, so their
// register budget is held to 128 to keep all four resident; the 12-state
// quadrotor's fragments need twice that (two waves per SIMD).
template <int DYN, int MT, int NW>
constexpr int rollout_waves_per_eu() {
  return (DYN != kDynQuad12 && MT == 1 && NW == 4) ? 4 : 1;
}

// One workgroup per tile of `spw` (<= 16*MT) sub-rollouts; PF: the contraction
// in the three-piece bf16 form.
template <int DYN, int MT, int NW, int PF>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(rollout_waves_per_eu<DYN, MT, NW>())))
rollout_mfma_kernel(RolloutArgs<float> ra, MfmaModel md,
                                                               int spw) {
  __shared__ RollSmem<DYN, MT, NW, PF> rs;
  mix_setup(rs.sm);
  const RollSeg sg = roll_seg(ra);
  rollout_tile<DYN, MT, NW, PF>(rs, ra.p, ra.x0, ra.u_nom, *ra.iter, ra.cost, md,
                                (int64_t)blockIdx.x * spw, spw, nullptr, ra.trace, &sg);
}

// Paired form (one 16-row tile per pair of workgroups, for problems with
// fewer tiles than compute units): partners are blocks b and b + 8 of each
// 16-block group, which the round-robin dispatch places on the same XCD, so
// their exchange stays inside one L2.  The grid must be resident at once.
template <int DYN, int NW, int PF>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(rollout_waves_per_eu<DYN, 1, NW>())))
rollout_pair_kernel(RolloutArgs<float> ra, MfmaModel md, int spw,
                                                               int n_groups, uint64_t *__restrict__ xbuf,
                                                               uint32_t spin_limit) {
  __shared__ RollSmem<DYN, 1, NW, PF> rs;
  const int blk = blockIdx.x;
  const int g = (blk / 16) * 8 + (blk % 8);
  if (g >= n_groups) return;  // both halves of an unused pair leave
  const PairCtx pc{xbuf + (size_t)g * kPairWords, (blk / 8) & 1, spin_limit};
  mix_setup(rs.sm);
  rollout_tile<DYN, 1, NW, PF>(rs, ra.p, ra.x0, ra.u_nom, *ra.iter, ra.cost, md, (int64_t)g * spw, spw, &pc,
                               ra.trace);
  // pair_fail is final: the tile's last evaluation ended with a barrier
  if (threadIdx.x == 0 && rs.sm.pair_fail) atomicAdd(&pair_give_ups_total, 1ull);
}

__global__ void read_give_ups_kernel(unsigned long long *out) { out[0] = pair_give_ups_total; }

// Persistent form for many independent problems: every workgroup pulls
// (problem, tile) items from a queue (items are ordered by decreasing work)
// until the queue is empty.  Each item is exactly a plain rollout tile.
template <int DYN, int MT, int NW, int PF>
__global__ void __launch_bounds__(NW * 64) rollout_batched_kernel(const BatchedProblem *__restrict__ probs,
                                                                  const BatchedItem *__restrict__ items,
                                                                  int n_items, int *__restrict__ queue) {
  __shared__ RollSmem<DYN, MT, NW, PF> rs;
  mix_setup(rs.sm);
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) rs.item = atomicAdd(queue, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(rs.item);   // uniform: the item's descriptors stay scalar
    if (item >= n_items) break;
    const BatchedItem it = items[item];
    const BatchedProblem &bp = probs[it.b];
    const ProbDev<float> p = bp.p;
    const MfmaModel md = bp.md;
    rollout_tile<DYN, MT, NW, PF>(rs, p, bp.x0, bp.u_nom, *bp.iter, bp.cost, md, it.s_base, it.spw);
  }
}

// One problem's descriptor and work items of a batched launch.
__global__ void batched_describe_kernel(BatchedProblem bp, BatchedProblem *__restrict__ probs,
                                        BatchedItem *__restrict__ items, int b, int64_t item_off, int64_t n_tiles,
                                        int spw) {
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i0 == 0) probs[b] = bp;
  for (int64_t i = i0; i < n_tiles; i += (int64_t)gridDim.x * blockDim.x)
    items[item_off + i] = BatchedItem{b, spw, i * spw};
}

template <int DYN, int MT, int NW, int PF = 0>
static hipError_t rollout_mfma_t(const RolloutArgs<float> &ra, const MfmaModel &md, int spw,
                                 hipStream_t s) {
  const int64_t n = (int64_t)ra.p.K * ra.p.Ms;
  const int64_t nb = (n + spw - 1) / spw;
  hipLaunchKernelGGL((rollout_mfma_kernel<DYN, MT, NW, PF>), dim3((unsigned)nb), dim3(NW * 64), 0, s, ra,
                     md, spw);
  return hipGetLastError();
}

// A pieces form's plain launch: the shared tile for tiles of 33..128 rows (of
// 64 rows up to 64 on 4 waves, else of 128), else one or two 16-row tiles per
// wave.
template <int PF>
static hipError_t rollout_pieces_t(const RolloutArgs<float> &ra, const MfmaModel &md, int spw, int waves,
                                   hipStream_t s) {
  if (spw > 32 && waves == 8) return rollout_mfma_t<kDynQuad12, 8, 8, PF>(ra, md, spw, s);
  if (spw > 64) return rollout_mfma_t<kDynQuad12, 8, 4, PF>(ra, md, spw, s);
  if (spw > 32) return rollout_mfma_t<kDynQuad12, 4, 4, PF>(ra, md, spw, s);
  if (waves == 8) return rollout_mfma_t<kDynQuad12, 1, 8, PF>(ra, md, spw, s);
  if (spw <= 16) return rollout_mfma_t<kDynQuad12, 1, 4, PF>(ra, md, spw, s);
  return rollout_mfma_t<kDynQuad12, 2, 4, PF>(ra, md, spw, s);
}

hipError_t launch_rollout_mfma(const RolloutArgs<float> &ra, const ModelArgs &m, const MfmaLayout &l,
                               const void *base, int tile_samples, int waves, int pf, hipStream_t s) {
  const MfmaModel md = mfma_view(l, base);
  const int spw = tile_samples;
  if (spw > 32 && (ra.trace || ra.ckpt_out || ra.xstart || ra.t_begin != 0 || ra.t_end >= 0)) return hipErrorInvalidValue;
  if (pf != kPfF32) {
    if (ra.p.dyn != kDynQuad12 || (pf == kPfF16x2 ? md.Wh : md.Wb) == nullptr ||
        (waves == 8 && spw > 16 && spw <= 32) || spw > 128)
      return hipErrorInvalidValue;
    return pf == kPfF16x2 ? rollout_pieces_t<kPfF16x2>(ra, md, spw, waves, s)
                          : rollout_pieces_t<kPfBf16x3>(ra, md, spw, waves, s);
  }
  if (ra.p.dyn == kDynQuad12) {
    if (waves == 8) {
      if (spw <= 16) return rollout_mfma_t<kDynQuad12, 1, 8>(ra, md, spw, s);
      return rollout_mfma_t<kDynQuad12, 2, 8>(ra, md, spw, s);
    }
    if (spw <= 16) return rollout_mfma_t<kDynQuad12, 1, 4>(ra, md, spw, s);
    return rollout_mfma_t<kDynQuad12, 2, 4>(ra, md, spw, s);
  }
  if (ra.p.dyn == kDynQuadHybrid) {
    if (spw <= 16) return rollout_mfma_t<kDynQuadHybrid, 1, 4>(ra, md, spw, s);
    return rollout_mfma_t<kDynQuadHybrid, 2, 4>(ra, md, spw, s);
  }
  if (spw <= 16) return rollout_mfma_t<kDynPointMass2D, 1, 4>(ra, md, spw, s);
  return rollout_mfma_t<kDynPointMass2D, 2, 4>(ra, md, spw, s);
}

size_t pair_ws_bytes(int64_t n_groups) { return align_up((size_t)n_groups * kPairWords * sizeof(uint64_t), 256); }

int pair_grid(int64_t n_groups) { return (int)(16 * ((n_groups + 7) / 8)); }

int pair_blocks_per_cu(int dyn, int waves, int pf) {
  int nb = 0;
  hipError_t e;
  if (dyn == kDynQuad12 && pf == kPfF16x2)
    e = waves == 8 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rollout_pair_kernel<kDynQuad12, 8, kPfF16x2>, 512, 0)
                   : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rollout_pair_kernel<kDynQuad12, 4, kPfF16x2>, 256, 0);
  else if (dyn == kDynQuad12 && pf == kPfBf16x3)
    e = waves == 8 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rollout_pair_kernel<kDynQuad12, 8, kPfBf16x3>, 512, 0)
                   : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rollout_pair_kernel<kDynQuad12, 4, kPfBf16x3>, 256, 0);
  else if (dyn == kDynQuad12 && waves == 8)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rollout_pair_kernel<kDynQuad12, 8, kPfF32>, 512, 0);
  else if (dyn == kDynQuad12)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rollout_pair_kernel<kDynQuad12, 4, kPfF32>, 256, 0);
  else if (dyn == kDynQuadHybrid)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rollout_pair_kernel<kDynQuadHybrid, 4, kPfF32>, 256, 0);
  else
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rollout_pair_kernel<kDynPointMass2D, 4, kPfF32>, 256, 0);
  return e == hipSuccess ? nb : 0;
}

hipError_t launch_rollout_pair(const RolloutArgs<float> &ra, const MfmaLayout &l, const void *base, int spw,
                               int waves, int pf, void *pair_ws, hipStream_t s) {
  const MfmaModel md = mfma_view(l, base);
  if (pf != kPfF32 && (ra.p.dyn != kDynQuad12 || (pf == kPfF16x2 ? md.Wh : md.Wb) == nullptr))
    return hipErrorInvalidValue;
  const int64_t n = (int64_t)ra.p.K * ra.p.Ms;
  const int64_t n_groups = (n + spw - 1) / spw;
  uint64_t *xbuf = (uint64_t *)pair_ws;
  // sequence numbers restart at 1 every launch: clear the previous launch's
  hipError_t e = launch_zero_u32((uint32_t *)xbuf, 2 * n_groups * kPairWords, s);
  if (e != hipSuccess) return e;
  // PI2RH_PAIR_SPIN_LIMIT (testing): polls of one wait before giving up
  uint32_t spin = kSpinLimit;
  if (const char *env = getenv("PI2RH_PAIR_SPIN_LIMIT")) spin = (uint32_t)strtoul(env, nullptr, 10);
  const dim3 grid((unsigned)pair_grid(n_groups));
  if (pf == kPfF16x2) {
    if (waves == 8)
      hipLaunchKernelGGL((rollout_pair_kernel<kDynQuad12, 8, kPfF16x2>), grid, dim3(512), 0, s, ra, md, spw,
                         (int)n_groups, xbuf, spin);
    else
      hipLaunchKernelGGL((rollout_pair_kernel<kDynQuad12, 4, kPfF16x2>), grid, dim3(256), 0, s, ra, md, spw,
                         (int)n_groups, xbuf, spin);
  } else if (pf == kPfBf16x3) {
    if (waves == 8)
      hipLaunchKernelGGL((rollout_pair_kernel<kDynQuad12, 8, kPfBf16x3>), grid, dim3(512), 0, s, ra, md, spw,
                         (int)n_groups, xbuf, spin);
    else
      hipLaunchKernelGGL((rollout_pair_kernel<kDynQuad12, 4, kPfBf16x3>), grid, dim3(256), 0, s, ra, md, spw,
                         (int)n_groups, xbuf, spin);
  } else if (ra.p.dyn == kDynQuad12) {
    if (waves == 8)
      hipLaunchKernelGGL((rollout_pair_kernel<kDynQuad12, 8, kPfF32>), grid, dim3(512), 0, s, ra, md, spw,
                         (int)n_groups, xbuf, spin);
    else
      hipLaunchKernelGGL((rollout_pair_kernel<kDynQuad12, 4, kPfF32>), grid, dim3(256), 0, s, ra, md, spw,
                         (int)n_groups, xbuf, spin);
  } else if (ra.p.dyn == kDynQuadHybrid) {
    hipLaunchKernelGGL((rollout_pair_kernel<kDynQuadHybrid, 4, kPfF32>), grid, dim3(256), 0, s, ra, md, spw,
                       (int)n_groups, xbuf, spin);
  } else {
    hipLaunchKernelGGL((rollout_pair_kernel<kDynPointMass2D, 4, kPfF32>), grid, dim3(256), 0, s, ra, md, spw,
                       (int)n_groups, xbuf, spin);
  }
  return hipGetLastError();
}

hipError_t launch_read_give_ups(uint64_t *out, hipStream_t s) {
  hipLaunchKernelGGL(read_give_ups_kernel, dim3(1), dim3(1), 0, s, (unsigned long long *)out);
  return hipGetLastError();
}

hipError_t launch_batched_describe(const BatchedProblem &bp, BatchedProblem *probs, BatchedItem *items, int b,
                                   int64_t item_off, int64_t n_tiles, int spw, hipStream_t s) {
  const int64_t nb = std::max<int64_t>(1, std::min<int64_t>((n_tiles + 255) / 256, 64));
  hipLaunchKernelGGL(batched_describe_kernel, dim3((unsigned)nb), dim3(256), 0, s, bp, probs, items, b, item_off,
                     n_tiles, spw);
  return hipGetLastError();
}

// A pieces form's batched launch (tile shape as in rollout_pieces_t).
template <int PF>
static void batched_pieces_t(const BatchedProblem *probs, const BatchedItem *items, int n_items, int max_spw,
                             int waves, int grid, int *queue, hipStream_t s) {
  if (max_spw > 32) {
    if (waves == 8)
      hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 8, 8, PF>), dim3(grid), dim3(512), 0, s, probs, items,
                         n_items, queue);
    else if (max_spw > 64)
      hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 8, 4, PF>), dim3(grid), dim3(256), 0, s, probs, items,
                         n_items, queue);
    else
      hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 4, 4, PF>), dim3(grid), dim3(256), 0, s, probs, items,
                         n_items, queue);
  } else if (waves == 8) {
    hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 1, 8, PF>), dim3(grid), dim3(512), 0, s, probs, items,
                       n_items, queue);
  } else if (max_spw <= 16) {
    hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 1, 4, PF>), dim3(grid), dim3(256), 0, s, probs, items,
                       n_items, queue);
  } else {
    hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 2, 4, PF>), dim3(grid), dim3(256), 0, s, probs, items,
                       n_items, queue);
  }
}

hipError_t launch_rollout_batched(const BatchedProblem *probs, const BatchedItem *items, int n_items,
                                  int max_spw, int waves, int pf, int grid, int *queue, hipStream_t s) {
  if (n_items == 0) return hipSuccess;
  if (pf != kPfF32) {
    if ((waves == 8 && max_spw > 16 && max_spw <= 32) || max_spw > 128) return hipErrorInvalidValue;
    if (pf == kPfF16x2)
      batched_pieces_t<kPfF16x2>(probs, items, n_items, max_spw, waves, grid, queue, s);
    else
      batched_pieces_t<kPfBf16x3>(probs, items, n_items, max_spw, waves, grid, queue, s);
  } else if (max_spw <= 16) {
    if (waves == 8)
      hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 1, 8, kPfF32>), dim3(grid), dim3(512), 0, s, probs,
                         items, n_items, queue);
    else
      hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 1, 4, kPfF32>), dim3(grid), dim3(256), 0, s, probs,
                         items, n_items, queue);
  } else {
    hipLaunchKernelGGL((rollout_batched_kernel<kDynQuad12, 2, 4, kPfF32>), dim3(grid), dim3(256), 0, s, probs,
                       items, n_items, queue);
  }
  return hipGetLastError();
}

MfmaModel mfma_model_view(const MfmaLayout &l, const void *base) { return mfma_view(l, base); }

// ------------------------------------------------------ adjoint parameters
// Parameter gradients of the adjoint on the matrix cores.  For a tile of 16
// records (sub-rollout steps of the reverse sweep) and a tile of 16 local
// models of output o:
//  (1) the forward contraction, with the activation anchor and prediction
//      reference the forward used for record r and output o, returns the
//      forward's a_{rj} and y_j - yref bitwise; w_{rj} = 2^(a_{rj} - log2 Z)
//      and e_{rj} = y_j - mu = (y_j - yref) - d1;
//  (2) each lane turns its four (record, model) elements into
//      ybar = w (mubar + 2 vbar e) and qbar = -w (mubar e + vbar (e^2 + sigma_j^2 - var)) / 2;
//  (3) G_j += sum_r qbar_{rj} Phi(z_r), Phi = [z_a z_b (a <= b), z, 1]: the C
//      fragments of (1) serve unchanged as the A operand (rows = models,
//      k = records) of a second contraction against the records' features,
//      which the fragments built for (1) already hold.
// Every workgroup holds a record chunk and 16 model tiles (2 per wave) and
// writes per-chunk sums G_j (NF features) and sum_r ybar_{rj}; the finish pass
// adds the chunks in double and centres them at c_j.  Bound by the matrix cores
// (88 instructions per 16 x 16 tile: 1.13 ms of their time at 163840 records and
// 6 x 256 models): 2.34 ms with 4 waves and three barriers per record tile, 2.03 with
// 8 waves sharing a record tile's fragments, 1.85 with those built a tile ahead.
constexpr int kPrmTilesPerWave = 2, kPrmWaves = 8;

template <int D>
__global__ void __launch_bounds__(kPrmWaves * 64) adj_param_mfma_kernel(MfmaModel md, const float *__restrict__ recs, int RW,
                                                              int64_t R, int nch, float *__restrict__ gpart,
                                                              int accumulate) {
  using G = Geo<D>;
  constexpr int NF = G::NP + D + 1;           // features of Phi
  constexpr int NFB = (NF + 15) / 16;
  constexpr int PWM = NFB * 16 + 1;           // per-model partial: G (padded), sum ybar
  constexpr int KQS = G::FQS / 4, GQS = G::FQS % 4;
  constexpr int KYS = G::FYS / 4, GYS = G::FYS % 4;
  // record tile n uses sm[n % 2] and st[n % 3]
  __shared__ MixSmem<D, 1, kPrmWaves> sm[2];
  __shared__ float st[3][16][kMaxOut][7];     // d1, var, log2 Z, m, yref, mubar, vbar per record and output
  // the wave index is uniform: its tiles' indices and offsets stay scalar
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ch = blockIdx.y;
  const int64_t r0 = R * ch / nch, r1 = R * (ch + 1) / nch;
  const int n_out = md.n_out;
  mix_setup(sm[0]);
  mix_setup(sm[1]);
  for (int i = threadIdx.x; i < 32; i += kPrmWaves * 64) {
    sm[i >> 4].z[i & 15][D] = 1.0f;
    sm[i >> 4].z[i & 15][D + 1] = 0.0f;
  }
  int tile[kPrmTilesPerWave], tout[kPrmTilesPerWave];
#pragma unroll
  for (int q = 0; q < kPrmTilesPerWave; ++q) {
    tile[q] = (blockIdx.x * kPrmWaves + wave) * kPrmTilesPerWave + q;
    int oo = 0;
    for (int i = 1; i < n_out; ++i) oo += (md.tile_off[i] <= tile[q]) ? 1 : 0;
    tout[q] = oo;
  }
  f32x4 acc[kPrmTilesPerWave][NFB];
  float ysum[kPrmTilesPerWave];
#pragma unroll
  for (int q = 0; q < kPrmTilesPerWave; ++q) {
    ysum[q] = 0.f;
#pragma unroll
    for (int fb = 0; fb < NFB; ++fb) acc[q][fb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // the wave's model tiles are fixed: W of the first one is requested ahead of
  // each record tile, the second one's right after the first contraction
  const __amdgpu_buffer_rsrc_t wrs = buffer_rsrc(md.W, md.n_tiles * G::KB4 * 1024);
  const __amdgpu_buffer_rsrc_t srs = buffer_rsrc(md.sig2, md.n_tiles * 16 * 4);
  auto loadW = [&](f32x4 (&Wd)[G::KB4], int q) {
    const int tq = min(tile[q], md.n_tiles - 1);
#pragma unroll
    for (int k = 0; k < G::KB4; ++k) Wd[k] = buffer_f32x4(wrs, lane * 16, (tq * G::KB4 + k) * 1024);
  };
  // A record tile's inputs (z and the five statistics per output of 16
  // records) pass through registers: the next tile's are requested while the
  // current one is contracted, so their memory latency is hidden.
  constexpr int NZI = (16 * D + kPrmWaves * 64 - 1) / (kPrmWaves * 64), NSI = (16 * kMaxOut * 7 + kPrmWaves * 64 - 1) / (kPrmWaves * 64);
  float zr[NZI], sr[NSI];
  auto fetch = [&](int64_t rb) {
    const int nr = (int)min((int64_t)16, r1 - rb);
#pragma unroll
    for (int k = 0; k < NZI; ++k) {
      const int i = threadIdx.x + kPrmWaves * 64 * k;
      const int row = i / D, a = i - row * D;
      zr[k] = (i < 16 * D && row < nr) ? recs[(rb + row) * RW + a] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < NSI; ++k) {
      const int i = threadIdx.x + kPrmWaves * 64 * k;
      const int row = i / (n_out * 7), rem = i - row * (n_out * 7);
      const int o = rem / 7, c = rem - o * 7;
      // rows past the chunk carry mubar = vbar = 0, so they add nothing
      sr[k] = (i < 16 * n_out * 7 && row < nr) ? recs[(rb + row) * RW + D + 7 * o + c] : 0.0f;
    }
  };
  f32x4 B[G::KB4];
  loadW(B, 0);
  auto store = [&](int zbuf, int sbuf) {
#pragma unroll
    for (int k = 0; k < NZI; ++k) {
      const int i = threadIdx.x + kPrmWaves * 64 * k;
      if (i < 16 * D) sm[zbuf].z[i / D][i % D] = zr[k];
    }
#pragma unroll
    for (int k = 0; k < NSI; ++k) {
      const int i = threadIdx.x + kPrmWaves * 64 * k;
      if (i < 16 * n_out * 7) {
        const int row = i / (n_out * 7), rem = i - row * (n_out * 7);
        st[sbuf][row][rem / 7][rem % 7] = sr[k];
      }
    }
  };
  // One barrier per record tile n: behind it the waves store tile n + 2's inputs,
  // request tile n + 3's, build tile n + 1's fragments and contract tile n, so
  // building overlaps the other waves' contractions.  (Tile n's statistics are read
  // until the next barrier, hence their third buffer.)
  if (r0 < r1) fetch(r0);
  store(0, 0);
  if (r0 + 16 < r1) fetch(r0 + 16);
  __syncthreads();
  build_fragments(sm[0]);
  store(1, 1);
  if (r0 + 32 < r1) fetch(r0 + 32);
  int cur = 0, sc = 0;
  for (int64_t rb = r0; rb < r1; rb += 16, cur ^= 1, sc = sc == 2 ? 0 : sc + 1) {
    __syncthreads();
    store(cur, sc == 0 ? 2 : sc - 1);
    if (rb + 48 < r1) fetch(rb + 48);
    if (rb + 16 < r1) build_fragments(sm[cur ^ 1]);
    const float *Af = (const float *)&sm[cur].A[0][0][0];
    const auto &sn = st[sc];
    f32x4 A[G::KB4];
#pragma unroll
    for (int q = 0; q < G::KB4; ++q) {
      const float4 v = sm[cur].A[0][q][lane];
      A[q] = f32x4{v.x, v.y, v.z, v.w};
    }
    // Phi(record 4k + i)[16 fb + lane%16] for the second contraction's B
    // operand (k = lane/16), read once per record tile from the anchor-free
    // fragments in LDS
    float phi[NFB][4];
#pragma unroll
    for (int fb = 0; fb < NFB; ++fb) {
      const int f = 16 * fb + (lane & 15);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * (lane >> 4) + i;
        phi[fb][i] = f < NF ? Af[((f >> 4) * 64 + 16 * (f & 3) + r) * 4 + ((f & 15) >> 2)] : 0.0f;
      }
    }
#pragma unroll
    for (int q = 0; q < kPrmTilesPerWave; ++q) {
      if (tile[q] >= md.n_tiles) continue;   // uniform over the wave
      const int o = tout[q];
      const int row = lane & 15;
      // the forward's anchors (activation anchor m, prediction reference yref)
      if ((lane >> 4) == GQS) A[KQS / 4][KQS % 4] = -sn[row][o][3];
      if ((lane >> 4) == GYS) A[KYS / 4][KYS % 4] = -sn[row][o][4];
      const float s2 = buffer_f32(srs, (lane & 15) * 4, tile[q] * 64);
      __builtin_amdgcn_sched_barrier(0);
      f32x4 qa = {0.f, 0.f, 0.f, 0.f}, qb = qa, ya = qa;
#pragma unroll
      for (int kb = 0; kb < G::KQB; ++kb) {
        if (kb & 1)
          qb = __builtin_amdgcn_mfma_f32_16x16x4f32(A[kb / 4][kb % 4], B[kb / 4][kb % 4], qb, 0, 0, 0);
        else
          qa = __builtin_amdgcn_mfma_f32_16x16x4f32(A[kb / 4][kb % 4], B[kb / 4][kb % 4], qa, 0, 0, 0);
      }
#pragma unroll
      for (int kb = G::KQB; kb < G::KB; ++kb)
        ya = __builtin_amdgcn_mfma_f32_16x16x4f32(A[kb / 4][kb % 4], B[kb / 4][kb % 4], ya, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      // the next tile this wave contracts: its second tile, else (next record
      // tile) its first
      loadW(B, (q + 1 < kPrmTilesPerWave && tile[q + 1] < md.n_tiles) ? q + 1 : 0);
      __builtin_amdgcn_sched_barrier(0);
      float qbar[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rr = 4 * (lane >> 4) + i;
        // normalised weight 2^(a - log2 Z) <= 1 (the bare v_exp_f32, whose
        // results below 2^-126 flush to 0, loses nothing); e = y - mu
        const float w = __builtin_amdgcn_exp2f((qa[i] + qb[i]) - sn[rr][o][2]), e = ya[i] - sn[rr][o][0];
        const float var = sn[rr][o][1], mub = sn[rr][o][5], vb = sn[rr][o][6];
        ysum[q] += w * (mub + 2.0f * vb * e);
        qbar[i] = -0.5f * w * (mub * e + vb * (e * e + s2 - var));
      }
      // G[model][feature] += sum_r qbar[r][model] Phi(z_r)[feature]: instance i
      // takes records 4k + i at k = lane/16
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int fb = 0; fb < NFB; ++fb)
          acc[q][fb] = __builtin_amdgcn_mfma_f32_16x16x4f32(qbar[i], phi[fb][i], acc[q][fb], 0, 0, 0);
      // restore the anchor slots for the next tile (they were set for output o)
      if ((lane >> 4) == GQS) A[KQS / 4][KQS % 4] = 0.0f;
      if ((lane >> 4) == GYS) A[KYS / 4][KYS % 4] = 0.0f;
    }
  }
  // per-chunk partials: acc[q][fb][j] = G[model 4 (lane/16) + j][feature 16 fb + lane%16]
#pragma unroll
  for (int q = 0; q < kPrmTilesPerWave; ++q) {
    if (tile[q] >= md.n_tiles) continue;
    float *dst = gpart + ((size_t)ch * md.n_tiles + tile[q]) * 16 * PWM;
#pragma unroll
    for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float &g = dst[(4 * (lane >> 4) + j) * PWM + 16 * fb + (lane & 15)];
        g = accumulate ? g + acc[q][fb][j] : acc[q][fb][j];
      }
    float y = ysum[q];
    y += __shfl_xor(y, 16);
    y += __shfl_xor(y, 32);
    if (lane < 16) {
      float &g = dst[lane * PWM + NFB * 16];
      g = accumulate ? g + y : y;
    }
  }
}

// ------------------------------------------------------ adjoint reverse sweep
// The reverse sweep needs, per (sample, step),
//   zbar = sum_j qbar_j ((D_j + D_j^T) z + h_j) + ybar_j b_j,   h_j = -(D_j + D_j^T) c_j,
// with qbar, ybar from the weights and residuals of Eq. (1) as in the
// parameter pass.  On the matrix cores: the forward contraction with the
// operands swapped (the model tile as the A operand, the samples' features as
// B: the folded tiles and the built fragments have exactly those register
// layouts) leaves, per lane, four models of one sample -- which is the A
// operand layout of the second contraction over models (rows = samples,
// k = models) against per-model parameters P = [packed D + D^T, h] (for qbar)
// and b (for ybar), stored by adj_rfold_kernel in B operand order:
//   [tile][block fb][lane][i] = param(model 4 (lane/16) + i)[16 fb + lane%16].
template <int D>
struct RevGeo {
  static constexpr int NP = D * (D + 1) / 2;
  static constexpr int NQ = NP + D;              // packed D + D^T, then h
  static constexpr int NFBQ = (NQ + 15) / 16;
  static constexpr int NFB = NFBQ + 1;           // + the b block
};

__global__ void __launch_bounds__(256) adj_rfold_kernel(ModelArgs m, MfmaLayout l, const float *__restrict__ rec,
                                                        int RS, int nfbq, float *__restrict__ dst) {
  const int tile = blockIdx.x, d = m.d, np = d * (d + 1) / 2;
  int o = 0;
  while (o + 1 < m.n_out && tile >= l.tile_off[o + 1]) ++o;
  const int jfirst = m.L_off[o] + (tile - l.tile_off[o]) * 16;
  const int n = (nfbq + 1) * 64 * 4;
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    const int i = e & 3, lane = (e >> 2) & 63, fb = e >> 8;
    const int j = jfirst + 4 * (lane >> 4) + i;
    const int f = 16 * fb + (lane & 15);
    float v = 0.0f;
    if (j < m.L_off[o + 1]) {
      const float *r = rec + (size_t)j * RS;   // [c | packed theta | b | beta0 | sigma^2]
      // entry (a, b) of D + D^T from the packed theta (theta_aa = D_aa)
      auto P = [&](int a, int b) {
        const int lo = a < b ? a : b, hi = a < b ? b : a;
        const float t = r[d + lo * d - lo * (lo - 1) / 2 + (hi - lo)];
        return a == b ? 2.0f * t : t;
      };
      if (fb < nfbq) {
        if (f < np) {
          int a = 0, rem = f;
          while (rem >= d - a) {
            rem -= d - a;
            ++a;
          }
          v = P(a, a + rem);
        } else if (f < np + d) {
          const int a = f - np;
          double h = 0.0;
          for (int b = 0; b < d; ++b) h -= (double)P(a, b) * (double)r[b];
          v = (float)h;
        }
      } else if ((lane & 15) < d) {
        v = r[d + np + (lane & 15)];
      }
    }
    dst[(size_t)tile * n + e] = v;
  }
}

struct RevArgs {
  ProbDev<float> p;
  const float *u_nom;
  const uint32_t *iter;
  MfmaModel md;
  const float4 *P;        // adj_rfold_kernel output
  const float *trace;     // [S][trace_T+1][NX + 3 NO], rows from step tb
  float *recs;            // [S][te-tb][D + 5 NO + NU]
  float *xbar_io;         // [S][NX]: the state adjoint between segments
  int tb, te, trace_T;
};

template <int DYN>
__global__ void __launch_bounds__(256) adj_reverse_mfma_kernel(RevArgs ra) {
  using DD = Dims<DYN>;
  constexpr int D = DD::D, NX = DD::NX, NU = DD::NU, NO = DD::NO;
  using G = Geo<D>;
  using RG = RevGeo<D>;
  constexpr int SEGW = NX + 5 * NO, RW = D + 7 * NO + NU;
  constexpr int NPOS = DYN == kDynPointMass2D ? 2 : 3;
  constexpr int KQS = G::FQS / 4, GQS = G::FQS % 4;
  constexpr int KYS = G::FYS / 4, GYS = G::FYS % 4;
  constexpr int PSTR = RG::NFB * 16;
  __shared__ MixSmem<D, 1, 4> sm;
  __shared__ float xbar[16][NX];
  __shared__ float stt[16][kMaxOut][7];          // d1, var, log2 Z, m, yref, mubar, vbar
  // per-wave sums of the second contraction; before it, the step's draws in
  // part[0][sample]: control, then accelerations (two workgroups fit a unit's LDS)
  __shared__ float part[4][16][PSTR];
  __shared__ float zb[16][D];
  __shared__ float obs_s[kMaxObs * 3];
  const ProbDev<float> &p = ra.p;
  const MfmaModel &md = ra.md;
  // the wave index is uniform: its tile range and offsets stay scalar
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // outside the contractions 16 lanes share a sample (four samples per wave):
  // lane l holds component l of the state, of its adjoint and of z (8192 samples x
  // 20 steps, 6 x 256 models: 1.86 ms with a lane per sample, 1.74 so)
  const int row = threadIdx.x >> 4, l = threadIdx.x & 15;
  const int64_t S = (int64_t)p.K * p.Ms, s = (int64_t)blockIdx.x * 16 + row;
  const bool active = s < S;
  const uint32_t k = active ? (uint32_t)s / (uint32_t)p.Ms : 0u, mm = active ? (uint32_t)s - k * (uint32_t)p.Ms : 0u;
  const uint32_t it = *ra.iter;
  const uint32_t wc = stream_word(kTagCtrl, p.problem_id, it), wd = stream_word(kTagDyn, p.problem_id, it);
  mix_setup(sm);
  for (int i = threadIdx.x; i < 3 * p.n_obs; i += 256) obs_s[i] = p.obs[i];
  const int tb = ra.tb, te = ra.te;
  if (l == 0) {
    sm.z[row][D] = 1.0f;
    sm.z[row][D + 1] = 0.0f;
  }
  // the adjoint of x_te: zero at the horizon's end, else what the later
  // segment's sweep left
  if (l < NX) xbar[row][l] = (te < p.T && active) ? ra.xbar_io[s * NX + l] : 0.0f;
  const int t0w = (int)((int64_t)wave * md.n_tiles / 4), t1w = (int)((int64_t)(wave + 1) * md.n_tiles / 4);
  // trace rows count from step tb; row t's values l, l + 16, .. of the sample are
  // requested one step ahead, and its state is row t - 1's next state
  const float *tr = ra.trace + (active ? s : 0) * (int64_t)(ra.trace_T + 1) * SEGW - (int64_t)tb * SEGW;
  constexpr int NSV = (SEGW + 15) / 16;
  float sv[NSV];
  auto fetch = [&](int t) {
#pragma unroll
    for (int c = 0; c < NSV; ++c) sv[c] = l + 16 * c < SEGW ? tr[(int64_t)t * SEGW + l + 16 * c] : 0.0f;
  };
  float x1 = l < NX ? tr[(int64_t)te * SEGW + l] : 0.0f;   // component l of x_{t+1}
  fetch(te - 1);
  __syncthreads();
  for (int t = te - 1; t >= tb; --t) {
    // (1) per sample: cost gradient at x_{t+1}, the draws of step t, z_t and the
    //     adjoints of the sampled accelerations
    {
      const float px = __shfl(x1, 0, 16), py = __shfl(x1, 1, 16);
      float gx = 0.0f, gy = 0.0f;
      if (p.obs_kind == kObsSmooth) {   // the indicator has zero derivative almost everywhere
        for (int i = l; i < p.n_obs; i += 16) {
          const float dx = px - obs_s[3 * i], dy = py - obs_s[3 * i + 1];
          const float e = -2.0f * p.obs_decay * p.obs_penalty * exp_(-p.obs_decay * (dx * dx + dy * dy));
          gx += dx * e;
          gy += dy * e;
        }
        auto add = [](float a, float b) { return a + b; };
        gx = lanes_reduce<16>(gx, add);
        gy = lanes_reduce<16>(gy, add);
      }
      if (l < NX) {
        float g = 0.0f;
        if (l < NPOS)
          g = 2 * p.w_pos[l] * (x1 - p.goal[l]) + (l == 0 ? gx : l == 1 ? gy : 0.0f);
        else if (l < 2 * NPOS)
          g = 2 * p.w_vel * x1;
        else if (DYN == kDynQuad12 && l < 9)
          g = 2 * p.w_ang * x1;
        xbar[row][l] += p.dt * g;
      }
      // lane 0 draws the control noise, lanes 1 and 2 the accelerations'
      const Philox4 r4 = philox4x32_10((uint32_t)t, k, l == 0 ? 0u : (mm << 4) | (uint32_t)(l - 1), l == 0 ? wc : wd,
                                       p.key0, p.key1);
      float e4[4];
      box_muller(r4.v[0], r4.v[1], &e4[0], &e4[1]);
      box_muller(r4.v[2], r4.v[3], &e4[2], &e4[3]);
      if (l <= (NO + 3) / 4)
#pragma unroll
        for (int i = 0; i < 4; ++i) part[0][row][4 * l + i] = e4[i];
#pragma unroll
      for (int c = 0; c < NSV; ++c) {
        const int i = l + 16 * c - NX;
        if (i >= 0 && i < 5 * NO) stt[row][i / 5][i % 5] = active ? sv[c] : (i % 5 == 1 ? 1.0f : 0.0f);
      }
      x1 = sv[0];   // component l of x_t
    }
    // a sample's lanes are one wave's: its LDS values are in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (l < D) {
      const int a = max(l - NX, 0);
      const float u = ra.u_nom[t * NU + min(a, NU - 1)] + p.noise_std[min(a, NU - 1)] * part[0][row][min(a, NU - 1)];
      sm.z[row][l] = !active ? 0.0f : l < NX ? x1 : u;
    }
    if (l < NO) {
      const int i = l < NPOS ? NPOS + l : 6 + l;
      const float ab = active ? p.dt * xbar[row][i] : 0.0f, v = stt[row][l][1];
      stt[row][l][5] = ab;
      stt[row][l][6] = (p.M > 0 && v > 0.f) ? ab * part[0][row][4 + l] / (2.0f * sqrtf(v)) : 0.0f;
    }
    fetch(max(t - 1, tb));
    __syncthreads();
    build_fragments(sm);
    __syncthreads();
    // (2) this wave's model tiles: both contractions
    f32x4 Z[G::KB4];
#pragma unroll
    for (int q = 0; q < G::KB4; ++q) {
      const float4 v = sm.A[0][q][lane];
      Z[q] = f32x4{v.x, v.y, v.z, v.w};
    }
    f32x4 accq[RG::NFBQ], accy = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int fb = 0; fb < RG::NFBQ; ++fb) accq[fb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int smp = lane & 15;   // this lane's sample in the swapped contraction
    int ocur = -1;
    // Loads run one stage ahead: the parameters P of a tile are requested
    // before its first contraction, the next tile's W right after it, so both
    // arrive while the matrix cores work (indices are clamped, not skipped,
    // so every wait counts a fixed number of loads).
    const __amdgpu_buffer_rsrc_t wrs = buffer_rsrc(md.W, md.n_tiles * G::KB4 * 1024);
    const __amdgpu_buffer_rsrc_t prs = buffer_rsrc(ra.P, md.n_tiles * RG::NFB * 1024);
    const __amdgpu_buffer_rsrc_t srs = buffer_rsrc(md.sig2, md.n_tiles * 16 * 4);
    auto loadW = [&](f32x4 (&Wd)[G::KB4], int tile) {
#pragma unroll
      for (int q = 0; q < G::KB4; ++q) Wd[q] = buffer_f32x4(wrs, lane * 16, (tile * G::KB4 + q) * 1024);
    };
    auto loadP = [&](f32x4 (&Pd)[RG::NFB], int tile) {
#pragma unroll
      for (int fb = 0; fb < RG::NFB; ++fb) Pd[fb] = buffer_f32x4(prs, lane * 16, (tile * RG::NFB + fb) * 1024);
    };
    f32x4 W[G::KB4], P[RG::NFB];
    if (t0w < t1w) loadW(W, t0w);
    for (int tile = t0w; tile < t1w; ++tile) {
      int o = 0;
#pragma unroll
      for (int i = 1; i < kMaxOut; ++i) o += (i < md.n_out && md.tile_off[i] <= tile) ? 1 : 0;
      if (o != ocur) {
        // the forward's anchors: every activation and prediction difference
        // comes out bitwise as the forward's final pass had them
        ocur = o;
        if ((lane >> 4) == GQS) Z[KQS / 4][KQS % 4] = -stt[smp][o][3];
        if ((lane >> 4) == GYS) Z[KYS / 4][KYS % 4] = -stt[smp][o][4];
      }
      const float d1 = stt[smp][o][0], var = stt[smp][o][1], l2z = stt[smp][o][2];
      const float mub = stt[smp][o][5], vb = stt[smp][o][6];
      // sigma^2 of the lane's four models 4 (lane/16) + i, one 16-byte read
      const f32x4 s2v = buffer_f32x4(srs, 16 * (lane >> 4), tile * 64);
      loadP(P, tile);
      __builtin_amdgcn_sched_barrier(0);
      f32x4 qa = {0.f, 0.f, 0.f, 0.f}, qb = qa, ya = qa;
#pragma unroll
      for (int kb = 0; kb < G::KQB; ++kb) {
        if (kb & 1)
          qb = __builtin_amdgcn_mfma_f32_16x16x4f32(W[kb / 4][kb % 4], Z[kb / 4][kb % 4], qb, 0, 0, 0);
        else
          qa = __builtin_amdgcn_mfma_f32_16x16x4f32(W[kb / 4][kb % 4], Z[kb / 4][kb % 4], qa, 0, 0, 0);
      }
#pragma unroll
      for (int kb = G::KQB; kb < G::KB; ++kb)
        ya = __builtin_amdgcn_mfma_f32_16x16x4f32(W[kb / 4][kb % 4], Z[kb / 4][kb % 4], ya, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      loadW(W, min(tile + 1, t1w - 1));
      __builtin_amdgcn_sched_barrier(0);
      float qbar[4], ybar[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float s2 = s2v[i];
        // normalised weight 2^(a - log2 Z) <= 1: the bare v_exp_f32, whose
        // results below 2^-126 flush to 0, loses nothing; e = y - mu
        const float w = __builtin_amdgcn_exp2f((qa[i] + qb[i]) - l2z), e = ya[i] - d1;
        ybar[i] = w * (mub + 2.0f * vb * e);
        qbar[i] = -0.5f * w * (mub * e + vb * (e * e + s2 - var));
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int fb = 0; fb < RG::NFBQ; ++fb) accq[fb] = __builtin_amdgcn_mfma_f32_16x16x4f32(qbar[i], P[fb][i], accq[fb], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) accy = __builtin_amdgcn_mfma_f32_16x16x4f32(ybar[i], P[RG::NFBQ][i], accy, 0, 0, 0);
    }
    // (3) per-wave sums to LDS: acc[fb][j] = sum[sample 4 (lane/16) + j][16 fb + lane%16]
#pragma unroll
    for (int fb = 0; fb < RG::NFBQ; ++fb)
#pragma unroll
      for (int j = 0; j < 4; ++j) part[wave][4 * (lane >> 4) + j][16 * fb + (lane & 15)] = accq[fb][j];
#pragma unroll
    for (int j = 0; j < 4; ++j) part[wave][4 * (lane >> 4) + j][16 * RG::NFBQ + (lane & 15)] = accy[j];
    __syncthreads();
    // (4) zbar[s][a] = sum_b M[a][b] z_b + h part + b part (waves added in order)
    {
      const int sr = threadIdx.x >> 4, a = threadIdx.x & 15;
      if (a < D) {
        float acc = 0.f;
        for (int b = 0; b < D; ++b) {
          const int lo = a < b ? a : b, hi = a < b ? b : a;
          const int pk = lo * D - lo * (lo - 1) / 2 + (hi - lo);
          const float M = ((part[0][sr][pk] + part[1][sr][pk]) + part[2][sr][pk]) + part[3][sr][pk];
          acc = fmaf(M, sm.z[sr][b], acc);
        }
        const int ih = RG::NP + a, iy = 16 * RG::NFBQ + a;
        acc += ((part[0][sr][ih] + part[1][sr][ih]) + part[2][sr][ih]) + part[3][sr][ih];
        acc += ((part[0][sr][iy] + part[1][sr][iy]) + part[2][sr][iy]) + part[3][sr][iy];
        zb[sr][a] = acc;
      }
    }
    __syncthreads();
    // (5) per sample: Euler transpose, the record of (s, t)
    {
      float xp = 0.0f;
      if (l < NX) {
        xp = xbar[row][l];
        if ((l >= NPOS && l < 2 * NPOS) || (DYN == kDynQuad12 && l >= 9)) xp += p.dt * xbar[row][l - (l < 9 ? NPOS : 3)];
        xp += zb[row][l];
      }
      __builtin_amdgcn_wave_barrier();   // every lane has read the old values
      if (l < NX) xbar[row][l] = xp;
      float *rec = ra.recs + (s * (te - tb) + (t - tb)) * RW;
      if (active)
        for (int i = l; i < RW; i += 16)
          rec[i] = i < D ? sm.z[row][i] : i < D + 7 * NO ? stt[row][(i - D) / 7][(i - D) % 7] : zb[row][NX + i - D - 7 * NO];
    }
    __syncthreads();
  }
  // the adjoint of x_tb for the earlier segment
  if (tb > 0 && active && l < NX) ra.xbar_io[s * NX + l] = xbar[row][l];
}

size_t adj_rfold_bytes(const MfmaLayout &l) {
  const int np = l.d * (l.d + 1) / 2, nfbq = (np + l.d + 15) / 16;
  return align_up((size_t)l.n_tiles * (nfbq + 1) * 64 * 4 * sizeof(float), 256);
}

hipError_t launch_adj_rfold(const ModelArgs &m, const MfmaLayout &l, const void *rec, int RS, void *rfold,
                            hipStream_t s) {
  const int np = l.d * (l.d + 1) / 2, nfbq = (np + l.d + 15) / 16;
  hipLaunchKernelGGL(adj_rfold_kernel, dim3(l.n_tiles), dim3(256), 0, s, m, l, (const float *)rec, RS, nfbq,
                     (float *)rfold);
  return hipGetLastError();
}

hipError_t launch_adj_reverse_mfma(const ProbDev<float> &p, const float *u_nom, const uint32_t *iter,
                                   const MfmaLayout &l, const void *base, const void *rfold, const float *trace,
                                   int trace_T, int tb, int te, float *xbar_io, float *recs, hipStream_t s) {
  RevArgs ra;
  ra.p = p;
  ra.u_nom = u_nom;
  ra.iter = iter;
  ra.md = mfma_view(l, base);
  ra.P = (const float4 *)rfold;
  ra.trace = trace;
  ra.recs = recs;
  ra.xbar_io = xbar_io;
  ra.tb = tb;
  ra.te = te;
  ra.trace_T = trace_T;
  const int64_t S = (int64_t)p.K * p.Ms;
  const dim3 grid((unsigned)((S + 15) / 16));
  if (p.dyn == kDynQuad12)
    hipLaunchKernelGGL(adj_reverse_mfma_kernel<kDynQuad12>, grid, dim3(256), 0, s, ra);
  else if (p.dyn == kDynPointMass2D)
    hipLaunchKernelGGL(adj_reverse_mfma_kernel<kDynPointMass2D>, grid, dim3(256), 0, s, ra);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

int adj_param_mfma_width(int d) {
  const int nf = d * (d + 1) / 2 + d + 1;
  return ((nf + 15) / 16) * 16 + 1;
}

hipError_t launch_adj_param_mfma(const MfmaLayout &l, const void *base, const float *recs, int RW, int64_t R,
                                 int nch, float *gpart, bool accumulate, hipStream_t s) {
  const MfmaModel md = mfma_view(l, base);
  const dim3 grid((unsigned)((md.n_tiles + kPrmWaves * kPrmTilesPerWave - 1) / (kPrmWaves * kPrmTilesPerWave)), (unsigned)nch);
  if (l.d == 16)
    hipLaunchKernelGGL(adj_param_mfma_kernel<16>, grid, dim3(kPrmWaves * 64), 0, s, md, recs, RW, R, nch, gpart,
                       (int)accumulate);
  else if (l.d == 6)
    hipLaunchKernelGGL(adj_param_mfma_kernel<6>, grid, dim3(kPrmWaves * 64), 0, s, md, recs, RW, R, nch, gpart,
                       (int)accumulate);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pi2rh
