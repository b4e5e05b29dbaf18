// Surrogate networks of the QED step and their training, on gfx950 matrix cores.
//
//   net A  (log10 chi, logit u) -> r,  logit(xi) = r + ln chi + 3 ln u
//   net B  log10 chi -> (ln h_rad - ln chi, ln h_pair + 8/(3 chi) - ln chi)
//
// Three hidden layers of width 64 with SiLU.  The two 64x64 layers run on
// bf16 matrix cores (v_mfma_f32_16x16x32_bf16; v_mfma_f32_16x16x16_bf16 where the
// contraction runs over a tile's 16 samples) with every
// operand split into bf16 hi + lo parts and
// the three products hi*hi + hi*lo + lo*hi accumulated in float32 (about 16
// significant bits; one bf16 product alone would leave ~3e-3 relative error,
// too coarse for the 1e-3 rate target).  Input and output layers (1-2 inputs,
// 1-2 outputs) are float32 vector code.
//
// A forward call evaluates a tile of 16 samples.  Lane l holds features
// mt*16 + 4*(l/16) + v (mt, v = 0..3) of sample l%16 both as the D result and as
// the B operand of the next layer, so activations stay in registers between
// layers; waves that own 64 samples make four calls.  Training (forward, backward,
// weight gradients, Adam) splits a tile over four waves and uses the same products;
// training data are drawn from the float64 master tables.
#include <hip/hip_runtime.h>
#include <math.h>

#include "internal.h"
#include "lookup.h"
#include "qed_device.h"
#include "mlp_device.h"

namespace qed {
namespace {
using namespace mlp;

// ------------------------------------------------------------- inputs/targets

// Training sample g of net A: chi at a table row, logit u uniform in
// [-Tmax, Tmax]; target from the float64 master inverse CDF of that row.
__device__ void sample_A(uint64_t g, uint32_t seed, const double *S64, float &x0, float &x1, float &yt) {
  const uint4 r = philox4x32_10(make_uint4((uint32_t)g, (uint32_t)(g >> 32), kTrainPurpose << 24, 0u),
                                make_uint2(seed, 0xA5A5A5A5u));
  const int row = (int)(r.x >> 24);                                     // 0..255
  const double t = -kTmax + 2.0 * kTmax * unit<double>(r.y);
  const double chi = exp(log(kRadChiMin) + row * ((log(kRadChiMax) - log(kRadChiMin)) / (kRadNChi - 1)));
  const double tlo = log(kRadULo) - log1p(-kRadULo), thi = log(kRadUHi) - log1p(-kRadUHi);
  const double dtn = (thi - tlo) / (kNU - 1);
  const double y = (t - tlo) / dtn;
  int j = (int)floor(y);
  j = j < 0 ? 0 : (j > kNU - 2 ? kNU - 2 : j);
  const double f = y - j;
  const double s = (1.0 - f) * S64[row * kNU + j] + f * S64[row * kNU + j + 1];
  const double lnu = -log1p(exp(-t));
  x0 = xin(chi);
  x1 = (float)(t / kTmax);
  yt = (float)((s - log(chi) - 3.0 * lnu - kAShift) / kAScale);
}

// Training sample g of net B: log10 chi uniform in [-3, 2]; targets from the
// float64 master rate tables (pair output masked below chi = 1e-2).
__device__ void sample_B(uint64_t g, uint32_t seed, const double *lnh, const double *L, const TabRange &rg,
                         float &x0, float yt[2], float m[2]) {
  const uint4 r = philox4x32_10(make_uint4((uint32_t)g, (uint32_t)(g >> 32), (kTrainPurpose << 24) | 1u, 0u),
                                make_uint2(seed, 0x5A5A5A5Au));
  const double lx = -3.0 + 5.0 * unit<double>(r.x);
  const double chi = pow(10.0, lx);
  x0 = xin(chi);
  yt[0] = (float)((log(h_rad<double>(chi, lnh, rg)) - log(chi) - kBShift0) / kBScale0);
  if (chi >= kPairChiMin) {
    const double x = (log(chi) - rg.pair_lnlo) * rg.pair_rate_inv;
    int i = (int)floor(x);
    i = i < 0 ? 0 : (i > kPairNRate - 2 ? kPairNRate - 2 : i);
    const double f = x - i;
    yt[1] = (float)(((1.0 - f) * L[i] + f * L[i + 1] - log(chi) - kBShift1) / kBScale1);
    m[1] = 1.f;
  } else {
    yt[1] = 0.f;
    m[1] = 0.f;
  }
  m[0] = 1.f;
}

// ------------------------------------------------------------------ training
struct TrainArgs {
  const float *theta;
  float *grad;
  const double *S64, *lnh, *L;
  const float *ext_x, *ext_t, *ext_m;   // optional external batch (gradient checks)
  int64_t nbatch;
  uint64_t sample0;
  uint32_t seed;
  TabRange rg;             // the default table range (the nets' domain)
};

// A workgroup's four waves work on a tile of 16 samples, wave w on rows 16 w ..
// 16 w + 15 of every layer.  A lane holds features 16 w + 4 (lane / 16) + v (v =
// 0..3) of sample lane % 16.  The waves' weights stay in registers, split, in the
// order of the A operand (K = 32, the order of swz32; the backward products'
// transposes too), the gradients are summed in registers over the tiles and reach
// memory once per workgroup; activations and deltas pass between the waves through
// LDS: in the order of the B operand (ExLds::x) for the next layer, and by feature
// (ExLds::t) for the weight gradients, whose contraction runs over the samples.
// What bounds it: at the training batch of 4096 (256 tiles) the latency of a tile's
// chain of four 64x64 products with a barrier each (2.2 us) and the workgroups'
// atomics on the same 8600 floats (0.04 us per workgroup).  Gradients of both nets
// at 4096 samples: 208 -> 37 us against one wave per tile, LDS atomics for every
// gradient element and the weights staged by each workgroup; at 100000 153 us.
constexpr int kTrainThreads = 256;

struct alignas(16) ExLds {
  uint32_t x[2][4][64][4];        // [buffer][wave][lane]: four values, hi then lo
  __bf16 t[3][2][H][16];          // a1 (two buffers by tile parity), a2: [hi / lo][feature][sample]
  __bf16 d[4][2][16][16];         // per wave: delta [hi / lo][row][sample]
  float y[4][2][16];              // per wave: partial outputs
};

// Rows r0 + lane % 16 of a 64x64 layer (or of its transpose) in the order of the
// K = 32 A operand, split.
struct WFrag {
  b8 h[2], l[2];
};
template <bool T>
__device__ __forceinline__ void load_frag(const float *W, int r0, WFrag &f) {
  const int lane = threadIdx.x & 63, r = r0 + (lane & 15), c0 = 4 * (lane >> 4);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int c = 32 * ks + 16 * (s >> 2) + c0 + (s & 3);
      const float x = T ? W[c * H + r] : W[r * H + c];
      const __bf16 h = (__bf16)x;
      f.h[ks][s] = h;
      f.l[ks][s] = (__bf16)(x - (float)h);
    }
}

// c + (rows of the layer) a, with a in ExLds::x order.
__device__ __forceinline__ f4 product(const WFrag &w, const uint32_t (*x)[64][4], f4 c) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const uint4 p = *reinterpret_cast<const uint4 *>(x[2 * ks][lane]);
    const uint4 q = *reinterpret_cast<const uint4 *>(x[2 * ks + 1][lane]);
    const b8 bh = __builtin_bit_cast(b8, make_uint4(p.x, p.y, q.x, q.y));
    const b8 bl = __builtin_bit_cast(b8, make_uint4(p.z, p.w, q.z, q.w));
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.h[ks], bh, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.h[ks], bl, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.l[ks], bh, c, 0, 0, 0);
  }
  return c;
}

// Publishes the lane's four values in both orders; t: rows of this wave.
__device__ __forceinline__ void publish(const float v[4], uint32_t x[4], __bf16 (*th)[16], __bf16 (*tl)[16]) {
  s4 h, l;
  split4(v, h, l);
  const uint2 uh = __builtin_bit_cast(uint2, h), ul = __builtin_bit_cast(uint2, l);
  *reinterpret_cast<uint4 *>(x) = make_uint4(uh.x, uh.y, ul.x, ul.y);
  const int lane = threadIdx.x & 63, f0 = 4 * (lane >> 4), j = lane & 15;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    th[f0 + k][j] = __builtin_bit_cast(__bf16, (short)h[k]);
    tl[f0 + k][j] = __builtin_bit_cast(__bf16, (short)l[k]);
  }
}

// Orders this wave's LDS writes before its later LDS reads (and vice versa).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// acc[kt] += delta a^T: this wave's 16 rows of delta, 64 features of a.
__device__ __forceinline__ void weight_grad(const __bf16 (*d)[16][16], const __bf16 (*t)[H][16], f4 acc[4]) {
  const int lane = threadIdx.x & 63, i = lane & 15, k0 = 4 * (lane >> 4);
  const s4 dh = *reinterpret_cast<const s4 *>(&d[0][i][k0]), dl = *reinterpret_cast<const s4 *>(&d[1][i][k0]);
#pragma unroll
  for (int kt = 0; kt < 4; ++kt) {
    const s4 ah = *reinterpret_cast<const s4 *>(&t[0][kt * 16 + i][k0]);
    const s4 al = *reinterpret_cast<const s4 *>(&t[1][kt * 16 + i][k0]);
    acc[kt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(dh, ah, acc[kt], 0, 0, 0);
    acc[kt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(dh, al, acc[kt], 0, 0, 0);
    acc[kt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(dl, ah, acc[kt], 0, 0, 0);
  }
}

// Sum over the 16 lanes of a row (the samples of a feature).
__device__ __forceinline__ float row_sum(float v) {
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Net = 0: net A, 1: net B.
template <int Net>
__global__ __launch_bounds__(kTrainThreads) void k_train(TrainArgs a) {
  constexpr Layout L = Net == 0 ? kA : kB;
  constexpr int NI = L.nin, NO = L.nout;
  __shared__ ExLds S;
  __shared__ float sum_s[L.n];
  const int lane = threadIdx.x & 63, j = lane & 15, w = threadIdx.x >> 6;
  const int r0 = 16 * w, f0 = r0 + 4 * (lane >> 4);      // the wave's first row, the lane's first feature
  WFrag w2, w3, w2t, w3t;
  load_frag<false>(a.theta + L.W2, r0, w2);
  load_frag<false>(a.theta + L.W3, r0, w3);
  load_frag<true>(a.theta + L.W2, r0, w2t);
  load_frag<true>(a.theta + L.W3, r0, w3t);
  float W1[4][NI], W4[NO][4], b1[4], b2[4], b3[4], b4[NO];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    b1[v] = a.theta[L.b1 + f0 + v]; b2[v] = a.theta[L.b2 + f0 + v]; b3[v] = a.theta[L.b3 + f0 + v];
#pragma unroll
    for (int c = 0; c < NI; ++c) W1[v][c] = a.theta[L.W1 + (f0 + v) * NI + c];
#pragma unroll
    for (int o = 0; o < NO; ++o) W4[o][v] = a.theta[L.W4 + o * H + f0 + v];
  }
#pragma unroll
  for (int o = 0; o < NO; ++o) b4[o] = a.theta[L.b4 + o];
  f4 gW2[4], gW3[4];
  float gW1[4][NI], gW4[NO][4], gb1[4], gb2[4], gb3[4], gb4[NO];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    gW2[v] = gW3[v] = f4{0.f, 0.f, 0.f, 0.f};
    gb1[v] = gb2[v] = gb3[v] = 0.f;
#pragma unroll
    for (int c = 0; c < NI; ++c) gW1[v][c] = 0.f;
#pragma unroll
    for (int o = 0; o < NO; ++o) gW4[o][v] = 0.f;
  }
#pragma unroll
  for (int o = 0; o < NO; ++o) gb4[o] = 0.f;
  const int64_t ntile = (a.nbatch + 15) / 16;
  const float inv_n = 1.0f / (float)a.nbatch;
  const int64_t stride = gridDim.x;
  int par = 0;
  // four of the workgroup's tiles at a time: lane 16 q + j draws sample j of the q-th
  for (int64_t tile0 = blockIdx.x; tile0 < ntile; tile0 += 4 * stride) {
    const int64_t smp = (tile0 + (lane >> 4) * stride) * 16 + j;
    float x0s = 0.f, x1s = 0.f, ts[2] = {0.f, 0.f}, ms[2] = {0.f, 0.f};
    if (smp < a.nbatch) {
      if (a.ext_x) {
        x0s = a.ext_x[smp * NI];
        if (NI > 1) x1s = a.ext_x[smp * NI + 1];
#pragma unroll
        for (int o = 0; o < NO; ++o) { ts[o] = a.ext_t[smp * NO + o]; ms[o] = a.ext_m ? a.ext_m[smp * NO + o] : 1.f; }
      } else if (Net == 0) {
        sample_A(a.sample0 + smp, a.seed, a.S64, x0s, x1s, ts[0]);
        ms[0] = 1.f;
      } else {
        sample_B(a.sample0 + smp, a.seed, a.lnh, a.L, a.rg, x0s, ts, ms);
      }
    }
#pragma unroll 1
    for (int q = 0; q < 4 && tile0 + q * stride < ntile; ++q) {
      const int src = 16 * q + j;
      const float x0 = __shfl(x0s, src, 64), x1 = NI > 1 ? __shfl(x1s, src, 64) : 0.f;
      float yt[NO], m[NO];
#pragma unroll
      for (int o = 0; o < NO; ++o) { yt[o] = __shfl(ts[o], src, 64); m[o] = __shfl(ms[o], src, 64); }
      auto &a1t = S.t[par];
      auto &a2t = S.t[2];
      par ^= 1;
      // forward; s1, s2, s3: derivatives of the activations
      float act[4], s1[4], s2[4], s3[4];
      auto activate = [&](float z, float &val, float &der) {
        const float g = sigm(z);
        val = z * g;
        der = g * (1.0f + z * (1.0f - g));
      };
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float z = b1[v] + W1[v][0] * x0;
        if (NI > 1) z += W1[v][NI - 1] * x1;
        activate(z, act[v], s1[v]);
      }
      publish(act, S.x[0][w][lane], &a1t[0][r0], &a1t[1][r0]);
      __syncthreads();
      f4 z = product(w2, S.x[0], f4{b2[0], b2[1], b2[2], b2[3]});
#pragma unroll
      for (int v = 0; v < 4; ++v) activate(z[v], act[v], s2[v]);
      publish(act, S.x[1][w][lane], &a2t[0][r0], &a2t[1][r0]);
      __syncthreads();
      z = product(w3, S.x[1], f4{b3[0], b3[1], b3[2], b3[3]});
#pragma unroll
      for (int v = 0; v < 4; ++v) activate(z[v], act[v], s3[v]);
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        float p = 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) p += W4[o][v] * act[v];
        p += __shfl_xor(p, 16, 64);
        p += __shfl_xor(p, 32, 64);
        if (lane < 16) S.y[w][o][j] = p;
      }
      __syncthreads();
      // output layer
      float dy[NO], d[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        const float y = ((S.y[0][o][j] + S.y[1][o][j]) + (S.y[2][o][j] + S.y[3][o][j])) + b4[o];
        dy[o] = 2.f * (y - yt[o]) * m[o] * inv_n;
        gb4[o] += dy[o];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          gW4[o][v] += dy[o] * act[v];
          d[v] += W4[o][v] * dy[o];
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) { d[v] *= s3[v]; gb3[v] += d[v]; }
      publish(d, S.x[0][w][lane], S.d[w][0], S.d[w][1]);
      __syncthreads();
      weight_grad(S.d[w], a2t, gW3);
      z = product(w3t, S.x[0], f4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
      for (int v = 0; v < 4; ++v) { d[v] = z[v] * s2[v]; gb2[v] += d[v]; }
      wave_lds_sync();
      publish(d, S.x[1][w][lane], S.d[w][0], S.d[w][1]);
      __syncthreads();
      weight_grad(S.d[w], a1t, gW2);
      z = product(w2t, S.x[1], f4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float dd = z[v] * s1[v];
        gb1[v] += dd;
        gW1[v][0] += dd * x0;
        if (NI > 1) gW1[v][NI - 1] += dd * x1;
      }
    }
  }
  // sums over the samples of a feature, then over the workgroups
  auto flush = [&](auto add) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        add(L.W2 + (f0 + v) * H + kt * 16 + j, gW2[kt][v]);
        add(L.W3 + (f0 + v) * H + kt * 16 + j, gW3[kt][v]);
      }
    if (j == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        add(L.b1 + f0 + v, gb1[v]);
        add(L.b2 + f0 + v, gb2[v]);
        add(L.b3 + f0 + v, gb3[v]);
#pragma unroll
        for (int c = 0; c < NI; ++c) add(L.W1 + (f0 + v) * NI + c, gW1[v][c]);
#pragma unroll
        for (int o = 0; o < NO; ++o) add(L.W4 + o * H + f0 + v, gW4[o][v]);
      }
    }
    if (w == 0 && lane == 0) {
#pragma unroll
      for (int o = 0; o < NO; ++o) add(L.b4 + o, gb4[o]);
    }
  };
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    gb1[v] = row_sum(gb1[v]); gb2[v] = row_sum(gb2[v]); gb3[v] = row_sum(gb3[v]);
#pragma unroll
    for (int c = 0; c < NI; ++c) gW1[v][c] = row_sum(gW1[v][c]);
#pragma unroll
    for (int o = 0; o < NO; ++o) gW4[o][v] = row_sum(gW4[o][v]);
  }
#pragma unroll
  for (int o = 0; o < NO; ++o) gb4[o] = row_sum(gb4[o]);
  flush([&](int i, float v) { sum_s[i] = v; });
  __syncthreads();
  // each workgroup starts at a place of its own: all at the same one, their
  // atomics queue up behind each other on one line after the next (83 us for both
  // nets at 4096 samples in 128 workgroups instead of 49)
  const int at = (int)((int64_t)blockIdx.x * L.n / gridDim.x) & ~63;
  for (int k = threadIdx.x; k < L.n; k += kTrainThreads) {
    const int i = k + at < L.n ? k + at : k + at - L.n;
    atomicAdd(&a.grad[i], sum_s[i]);
  }
}

// (a kernel, not a memset, so that a caller may capture it)
__global__ void k_zero(float *p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

__global__ void k_adam(float *theta, float *grad, float *m, float *v, int n, float lr, float b1t, float b2t) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float g = grad[i];
  const float mm = 0.9f * m[i] + 0.1f * g;
  const float vv = 0.999f * v[i] + 0.001f * g * g;
  m[i] = mm;
  v[i] = vv;
  theta[i] -= lr * (mm / (1.f - b1t)) / (sqrtf(vv / (1.f - b2t)) + 1e-8f);
  grad[i] = 0.f;
}

// PyTorch-style initial weights: U(-1/sqrt(fan_in), 1/sqrt(fan_in)).
__global__ void k_init(float *theta, int net, uint32_t seed) {
  const Layout L = net == 0 ? kA : kB;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= L.n) return;
  const int fan = (i < L.W2) ? L.nin : H;
  const uint4 r = philox4x32_10(make_uint4((uint32_t)i, (uint32_t)net, kInitPurpose << 24, 0u), make_uint2(seed, 0u));
  theta[i] = (float)((2.0 * unit<double>(r.x) - 1.0) / sqrt((double)fan));
}

// --------------------------------------------------------------- inference
struct InferArgs {
  const float *thA, *thB;
  const double *chi, *gamma;
  const uint64_t *id;
  int64_t n;
  uint32_t seed;
  uint64_t step;
  const int64_t *d_step;
  const float *lnh32, *L32, *s0sc, *chk;
  const uint16_t *q16;
  float *lnw, *xi, *lnwp;
  float tol;
  unsigned long long *fallback;     // [0] xi fallbacks, [1] rate fallbacks
  TabRange rg;                      // the default table range (the nets' domain)
};

struct InferLds {
  NetLdsI A, B;
  float chk[kRadNChi * (2 + 2 * kChkN)];
};

// Bound by the instructions of the activations (48 exponentials and reciprocals a lane
// per net and tile).  Three waves per SIMD: 1e7 samples 1.96 (two) -> 1.76 ms; four
// spill (1.77), two tiles per read of the weights gain less (1.81).  A small call spreads
// its waves over all workgroups: 1e3 samples 34 -> 26 us, 5e5 114 -> 92.
constexpr int kInferThreads = 768;

__global__ __launch_bounds__(kInferThreads) void k_infer(InferArgs a) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  InferLds &S = *reinterpret_cast<InferLds *>(lds_raw);
  stage_net_infer(a.thA, kA, &S.A);
  stage_net_infer(a.thB, kB, &S.B);
  for (int k = threadIdx.x; k < kRadNChi * (2 + 2 * kChkN); k += blockDim.x) S.chk[k] = a.chk[k];
  __syncthreads();
  const RowQ16 tab{a.q16, a.s0sc};
  const int lane = threadIdx.x & 63;
  const int64_t ntile = (a.n + 63) / 64;     // 64 samples per wave, one per lane
  const int wpb = blockDim.x >> 6;
  uint32_t nfx = 0, nfr = 0;
  // (wave-major, so that few tiles spread over all the workgroups)
  for (int64_t tile = (int64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x; tile < ntile;
       tile += (int64_t)gridDim.x * wpb) {
    reload_barrier();
    const int64_t i = tile * 64 + lane;
    const bool valid = i < a.n;
    const double chi = valid ? a.chi[i] : 1.0;
    const double gam = valid ? a.gamma[i] : 1.0;
    const uint64_t id = valid ? a.id[i] : 0;
    const uint4 r = stream4<true>(id, a.seed, a.d_step ? (uint64_t)*a.d_step : a.step, kLeptonEvent, 0u);
    const float u = unit<float>(r.x), urow = unit<float>(r.z);
    const float t = logf(u) - log1pf(-u);
    const bool in_chi = chi >= kRadChiMin && chi <= kRadChiMax;
    const float x0 = xin(in_chi ? chi : 1.0), x1 = (float)(t / kTmax);
    // the wave's 64 samples go through each net as four 16-sample tiles; lane
    // q*16 + j keeps the outputs of sample j of tile q, its own
    float yB0 = 0.f, yB1 = 0.f, yA = 0.f;
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      reload_barrier();
      float y[2];
      forward_inf(S.B, 1, 2, __shfl(x0, q * 16 + (lane & 15), 64), 0.f, y);    // rates (net B)
      if ((lane >> 4) == q) { yB0 = y[0]; yB1 = y[1]; }
    }
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      reload_barrier();
      float y[2];
      forward_inf(S.A, 2, 1, __shfl(x0, q * 16 + (lane & 15), 64), __shfl(x1, q * 16 + (lane & 15), 64), y);
      if ((lane >> 4) == q) yA = y[0];                                          // xi (net A)
    }
    const float lchi = logf((float)chi);
    float lh = kBShift0 + kBScale0 * yB0 + lchi;
    const float env = logf(1.001f * (float)kHc1 * (float)chi);
    bool rate_ok = in_chi && isfinite(lh) && lh <= env;
    if (!rate_ok) lh = logf(h_rad<float>((float)chi, a.lnh32, a.rg));
    float lhp;
    if (chi < kPairChiMin || gam < 2.0) lhp = -INFINITY;
    else if (chi <= kPairChiMax && isfinite(yB1)) lhp = kBShift1 + kBScale1 * yB1 + lchi - 8.0f / (3.0f * (float)chi);
    else lhp = logf(h_pair<float>((float)chi, a.L32, a.rg));
    // xi with residual check against the Hermite CDF table
    const bool in_u = fabsf(t) <= (float)kTmax;
    float s_hat = kAShift + kAScale * yA + lchi + 3.0f * (-log1pf(__expf(-t)));
    bool xi_ok = in_chi && in_u && isfinite(s_hat);
    float xi, om;
    if (xi_ok) {
      const float x = (lchi - (float)a.rg.rad_lnlo) * (float)a.rg.rad_inv;
      int ii = (int)floorf(x);
      ii = ii < 0 ? 0 : (ii > kRadNChi - 2 ? kRadNChi - 2 : ii);
      const float w = x - ii;
      const float P = (1.f - w) * check_cdf(S.chk, ii, s_hat) + w * check_cdf(S.chk, ii + 1, s_hat);
      xi_ok = fabsf(P - u) <= a.tol;
    }
    if (xi_ok) {
      xi = 1.f / (1.f + __expf(-s_hat));
      om = 1.f / (1.f + __expf(s_hat));
    } else {
      sample_rad<float>(tab, (float)chi, u, urow, xi, om, a.rg);
    }
    if (valid) {
      const double lng = log_rate_unit() - ln_any(gam);   // ln W = ln h + lng
      a.lnw[i] = (float)((double)lh + lng);
      a.xi[i] = xi;
      if (a.lnwp) a.lnwp[i] = isfinite(lhp) ? (float)((double)lhp + lng) : -INFINITY;
      nfx += !xi_ok;
      nfr += !rate_ok;
    }
  }
  // per-wave totals of fallbacks
  for (int o = 32; o > 0; o >>= 1) { nfx += __shfl_xor(nfx, o, 64); nfr += __shfl_xor(nfr, o, 64); }
  if (lane == 0) {
    unsigned long long *f = a.fallback + (blockIdx.x % kCounterSlots) * cNumCounters;
    if (nfx) atomicAdd(&f[0], (unsigned long long)nfx);
    if (nfr) atomicAdd(&f[1], (unsigned long long)nfr);
  }
}

// raw forward for tests: y = net(x) for n samples (normalised inputs/outputs)
__global__ __launch_bounds__(256) void k_forward_raw(const float *theta, int net, const float *x, int64_t n, float *y) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  NetLdsI &S = *reinterpret_cast<NetLdsI *>(lds_raw);
  const Layout L = net == 0 ? kA : kB;
  stage_net_infer(theta, L, &S);
  __syncthreads();
  const int lane = threadIdx.x & 63, j = lane & 15;
  const int64_t ntile = (n + 15) / 16;
  for (int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); tile < ntile; tile += (int64_t)gridDim.x * 4) {
    reload_barrier();
    const int64_t i = tile * 16 + j;
    const bool valid = i < n;
    const float x0 = valid ? x[i * L.nin] : 0.f;
    const float x1 = (valid && L.nin > 1) ? x[i * L.nin + 1] : 0.f;
    float yy[2];
    forward_inf(S, L.nin, L.nout, x0, x1, yy);
    if (valid && (lane >> 4) == 0)
      for (int o = 0; o < L.nout; ++o) y[i * L.nout + o] = yy[o];
  }
}

}  // namespace

int mlp_params(int net) { return net == 0 ? kA.n : kB.n; }

hipError_t launch_mlp_init(float *theta, int net, uint32_t seed, hipStream_t st) {
  const int n = mlp_params(net);
  hipLaunchKernelGGL(k_init, dim3((n + 255) / 256), dim3(256), 0, st, theta, net, seed);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(int net, const float *theta, float *grad, const double *S64, const double *lnh,
                           const double *L, const float *ext_x, const float *ext_t, const float *ext_m,
                           int64_t nbatch, uint64_t sample0, uint32_t seed, hipStream_t st) {
  TrainArgs a{theta, grad, S64, lnh, L, ext_x, ext_t, ext_m, nbatch, sample0, seed,
              make_range(kRadChiMax, kPairChiMax)};
  const int64_t tiles = (nbatch + 15) / 16;
  // a workgroup costs 0.04 us of atomics, a tile 2.2 us of its workgroup's time:
  // about sqrt(55 tiles) workgroups are the shortest, fewer where whole turns allow it,
  // up to the chip's 256 compute units.  The minimum is flat: 4096 samples take 25 us
  // a net in 86 workgroups (these), 119 or 128, with 256 a quarter more.
  int64_t blocks = (int64_t)ceil(sqrt(55.0 * (double)tiles));
  if (blocks > 256) blocks = 256;
  if (blocks > tiles) blocks = tiles;
  const int64_t turns = (tiles + blocks - 1) / blocks;
  blocks = (tiles + turns - 1) / turns;
  if (net == 0) hipLaunchKernelGGL(k_train<0>, dim3((unsigned)blocks), dim3(kTrainThreads), 0, st, a);
  else hipLaunchKernelGGL(k_train<1>, dim3((unsigned)blocks), dim3(kTrainThreads), 0, st, a);
  return hipGetLastError();
}

// Dynamic LDS above the default limit, for the kernels of this file; called
// once per context, with the context's device current.
hipError_t mlp_set_attributes() {
  hipError_t e =
      hipFuncSetAttribute((const void *)k_forward_raw, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)sizeof(NetLdsI));
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void *)k_infer, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(InferLds));
  return e;
}

hipError_t launch_zero(float *p, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_zero, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

hipError_t launch_adam(float *theta, float *grad, float *m, float *v, int net, float lr, float b1t, float b2t,
                       hipStream_t st) {
  const int n = mlp_params(net);
  hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, st, theta, grad, m, v, n, lr, b1t, b2t);
  return hipGetLastError();
}

hipError_t launch_mlp_forward(const float *theta, int net, const float *x, int64_t n, float *y, hipStream_t st) {
  int64_t blocks = ((n + 15) / 16 + 3) / 4;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_forward_raw, dim3((unsigned)blocks), dim3(256), sizeof(NetLdsI), st, theta, net, x, n, y);
  return hipGetLastError();
}

hipError_t launch_mlp_sample(qed_ctx *c, const double *chi, const double *gamma, const uint64_t *id, int64_t n,
                             int64_t step, float *lnw, float *xi, float *lnwp, float tol, hipStream_t st) {
  InferArgs a{c->mlp_theta[0], c->mlp_theta[1], chi, gamma, id, n, c->params.seed, (uint64_t)step,
              step < 0 ? c->d_step : nullptr,
              c->rad_lnh32, c->pair_L32, c->rad_s0sc, c->rad_chk, c->rad_q16, lnw, xi, lnwp, tol,
              c->d_counters + cMlpFallbackXi, make_range(kRadChiMax, kPairChiMax)};
  int64_t blocks = (n + 63) / 64;
  if (blocks > c->n_cu) blocks = c->n_cu;      // one workgroup per CU (LDS-bound)
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_infer, dim3((unsigned)blocks), dim3(kInferThreads), sizeof(InferLds), st, a);
  return hipGetLastError();
}

}  // namespace qed
