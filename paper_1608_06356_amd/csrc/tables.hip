// Table builder: total rates and inverse CDFs of the photon spectrum (Eq. 1,
// Eq. 4 or Eq. 5) and of the pair spectrum (Eq. 6), by float64 quadrature on
// the GPU.
//
// K_nu(x) = int_0^inf exp(-x cosh t) cosh(nu t) dt and its tail integral
// int_x^inf K_nu = int_0^inf exp(-x cosh t) cosh(nu t) / cosh t dt (DLMF 10.32.9)
// by the trapezoid rule with step min(0.1, 0.35/sqrt(x)) up to cosh t = 1 + 40/x.
// Every spectrum is made of a few functions of one variable (K_{1/3}, K_{2/3}, the
// tail integrals, Eq. 4's J_1..J_3), so these are integrated once at the Chebyshev
// nodes of short intervals of ln x and the rows interpolate them.
// Per chi row: density in s = logit(xi) on 1024 uniform intervals, 3-point
// Gauss-Legendre per interval, cumulative sum, infrared tail below the grid
// (photons), quantiles at 256 nodes uniform in logit(u) from the cubic Hermite
// interpolant of the cumulative spectrum (52 bisections per node).
#include <hip/hip_runtime.h>
#include <math.h>

#include "internal.h"
#include "qed_device.h"

namespace qed {
namespace {

constexpr double kInvSqrt3Pi = 0.18377629847393068;   // 1 / (sqrt3 pi)
constexpr double kGamma23 = 1.3541179394264004;        // Gamma(2/3)
enum Kind { kFormulaI = 1, kFormulaII = 2, kPair = 3, kClassical = 4 };

// ---------------------------------------------- functions of one variable
// f(x) exp(c x) (c = 1 for the Bessel functions, 2 for the J) as Chebyshev
// series on intervals of 1/8 in ln x, x from below the smallest argument of any
// row (3.3e-16, Eq. 4 at xi = 1e-15 chi) to above the largest (8 / (3 chi) + 45
// at chi = 1e-2, Eq. 6).  The scaled functions are analytic in ln x in a strip
// of half-width pi, about 50 interval half-widths, so the terms fall by about
// 100 each and ten of them reach the float64 rounding (the rows agree with the
// integration at every point to 3e-16 in ln h).
constexpr int kTerms = 10;
constexpr double kYLo = -35.75, kYStep = 0.125;
constexpr int kIntervals = 333;                        // up to ln x = 5.875
enum Fun { fK13 = 0, fK23, fI13, fI53, fJ1, fJ2, fJ3, kFuns };
struct FunTab {
  double c[kIntervals][kFuns][kTerms];
};
static_assert(sizeof(FunTab) / sizeof(double) == kTabWork, "size of the context's table scratch");

__device__ __forceinline__ int interval(double y, double &tau) {
  const double p = (y - kYLo) * (1.0 / kYStep);
  int i = (int)floor(p);
  i = i < 0 ? 0 : (i > kIntervals - 1 ? kIntervals - 1 : i);
  tau = 2.0 * (p - i) - 1.0;
  return i;
}

// Clenshaw sum
__device__ __forceinline__ double series(const double *c, double tau) {
  const double t2 = 2.0 * tau;
  double b1 = 0.0, b2 = 0.0;
#pragma unroll
  for (int k = kTerms - 1; k > 0; --k) {
    const double b = fma(t2, b1, c[k]) - b2;
    b2 = b1;
    b1 = b;
  }
  return fma(tau, b1, c[0]) - b2;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// cos(pi m / 20)
constexpr int kCosN = 4 * kTerms;
__constant__ const double kCos[kCosN] = {
    1.0, 0.98768834059513772619, 0.95105651629515357212, 0.89100652418836786236, 0.80901699437494742410,
    0.70710678118654752440, 0.58778525229247312917, 0.45399049973954679156, 0.30901699437494742410,
    0.15643446504023086901, 0.0, -0.15643446504023086901, -0.30901699437494742410, -0.45399049973954679156,
    -0.58778525229247312917, -0.70710678118654752440, -0.80901699437494742410, -0.89100652418836786236,
    -0.95105651629515357212, -0.98768834059513772619, -1.0, -0.98768834059513772619, -0.95105651629515357212,
    -0.89100652418836786236, -0.80901699437494742410, -0.70710678118654752440, -0.58778525229247312917,
    -0.45399049973954679156, -0.30901699437494742410, -0.15643446504023086901, 0.0, 0.15643446504023086901,
    0.30901699437494742410, 0.45399049973954679156, 0.58778525229247312917, 0.70710678118654752440,
    0.80901699437494742410, 0.89100652418836786236, 0.95105651629515357212, 0.98768834059513772619};
static_assert(kTerms == 10, "kCos holds the angles of ten nodes");

// ln x of Chebyshev node j of interval i
__device__ __forceinline__ double node_y(int i, int j) {
  return kYLo + kYStep * (i + 0.5 + 0.5 * kCos[2 * j + 1]);
}

// Coefficients of N functions from their values at the interval's nodes
template <int N>
__device__ __forceinline__ void chebyshev(FunTab *tab, int i, int fun0, const double (*v)[N]) {
  if (threadIdx.x < N * kTerms) {
    const int f = threadIdx.x / kTerms, k = threadIdx.x % kTerms;
    double s = 0.0;
    for (int j = 0; j < kTerms; ++j) s += v[j][f] * kCos[k * (2 * j + 1) % kCosN];
    tab->c[i][fun0 + f][k] = s * ((k ? 2.0 : 1.0) / kTerms);
  }
}

// One workgroup per interval, one wave per node, the trapezoid nodes over the
// lanes.  exp(-x (cosh t - 1)) with cosh t - 1 = 2 sinh^2(t/2); cosh(2t/3) from
// cosh(t/3).  I53 (the classical spectrum's tail integral) on request.
template <bool I53>
__global__ __launch_bounds__(64 * kTerms) void k_bessel(FunTab *tab) {
  constexpr int N = I53 ? 4 : 3;
  __shared__ double v[kTerms][N];
  const int i = blockIdx.x, j = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double x = exp(node_y(i, j));
  const double h = fmin(0.1, 0.35 / sqrt(x));
  const int n = (int)ceil(acosh(1.0 + 40.0 / x) / h);
  double k13 = 0.0, k23 = 0.0, i13 = 0.0, i53 = 0.0;
  for (int q = lane; q <= n; q += 64) {
    const double t = q * h, sh = sinh(0.5 * t), c1 = 2.0 * sh * sh, ch = 1.0 + c1;
    const double e = exp(-x * c1) * (q ? 1.0 : 0.5);
    const double c13 = cosh((1.0 / 3.0) * t), a = e * c13;
    k13 += a;
    k23 += e * (2.0 * c13 * c13 - 1.0);
    i13 += a / ch;
    if (I53) i53 += e * cosh((5.0 / 3.0) * t) / ch;
  }
  k13 = wave_sum_f64(k13); k23 = wave_sum_f64(k23); i13 = wave_sum_f64(i13);
  if (I53) i53 = wave_sum_f64(i53);
  if (lane == 0) {
    v[j][0] = h * k13; v[j][1] = h * k23; v[j][2] = h * i13;
    if (I53) v[j][N - 1] = h * i53;
  }
  __syncthreads();
  chebyshev<N>(tab, i, fK13, v);
}

// J_1..J_3 of Eq. (4) after u = sigma cosh^3(theta): trapezoid in theta with step
// min(0.08, 0.3/sqrt(sigma)) up to sigma cosh^3 = sigma + 22.5.  Scaled by
// exp(2 sigma).
__global__ __launch_bounds__(64 * kTerms) void k_jfun(FunTab *tab) {
  __shared__ double v[kTerms][3];
  const int i = blockIdx.x, j = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double ly = node_y(i, j), sigma = exp(ly);
  const double h = fmin(0.08, 0.3 / sqrt(sigma));
  const int n = (int)ceil(acosh(cbrt(1.0 + 22.5 / sigma)) / h);
  double a = 0.0, b = 0.0, c = 0.0;
  for (int q = lane; q <= n; q += 64) {
    const double th = q * h, sh = sinh(th), hs = sinh(0.5 * th), c1 = 2.0 * hs * hs, ch = 1.0 + c1;
    // x = sigma cosh^3; x - sigma = sigma (cosh - 1)(cosh^2 + cosh + 1)
    const double dx = sigma * c1 * (ch * ch + ch + 1.0);
    double tau;
    const int m = interval(ly + 3.0 * log(ch), tau);
    const double e = exp(-dx), k13 = e * series(tab->c[m][fK13], tau), k23 = e * series(tab->c[m][fK23], tau);
    const double w = q ? 1.0 : 0.5, c3 = w * ch * ch * ch, c5 = c3 * ch * ch;
    a += c5 * k23 * k23;
    b += c3 * sh * sh * k13 * k13;
    c += c5 * k13 * k13;
  }
  a = wave_sum_f64(a); b = wave_sum_f64(b); c = wave_sum_f64(c);
  if (lane == 0) { v[j][0] = h * a; v[j][1] = h * b; v[j][2] = h * c; }
  __syncthreads();
  chebyshev<3>(tab, i, fJ1, v);
}

// Density in s: S(xi, chi) xi (1 - xi), S normalised so dW/dxi = alpha E_S S / gamma.
// With e = exp(s): xi = e / (1 + e), 1 - xi = 1 / (1 + e), 1 / xi = 1 + 1 / e.  The
// spectrum's variable is k e (Eqs. 1, 4), k xi (Eq. 5) or k / (xi (1 - xi)) (Eq. 6),
// k = arg_scale(chi), lk = ln k.
template <int K>
__device__ __forceinline__ double arg_scale(double chi) {
  return (K == kFormulaII ? 1.0 / 3.0 : 2.0 / 3.0) / chi;
}
template <int K>
__device__ __forceinline__ double density(const FunTab *tab, double s, double k, double lk) {
  const double e = exp(s), ope = 1.0 + e, om = 1.0 / ope, xi = e * om;
  double S, tau;
  if constexpr (K == kFormulaI) {                               // Eq. (1)
    const auto &c = tab->c[interval(lk + s, tau)];
    S = kInvSqrt3Pi * ((om + ope) * series(c[fK23], tau) - series(c[fI13], tau)) * exp(-k * e);
  } else if constexpr (K == kFormulaII) {                       // Eq. (4)
    const auto &c = tab->c[interval(lk + s, tau)];
    const double f1 = 1.0 + ope * ope, f2 = 2.0 * ope, f3 = e * e;      // xi / (1 - xi) = e
    S = xi * k * (1.0 / (kPi * kPi)) *
        (f1 * series(c[fJ1], tau) + f2 * series(c[fJ2], tau) + f3 * series(c[fJ3], tau)) * exp(-2.0 * k * e);
  } else if constexpr (K == kClassical) {                       // Eq. (5), z = 2 xi / (3 chi)
    const double z = k * xi;
    const auto &c = tab->c[interval(log(z), tau)];
    S = 1.7320508075688772 / (3.0 * kPi) * series(c[fI53], tau) * exp(-z);
  } else {                                                      // Eq. (6), "+" sign
    const double r = ope * ope / e, d = k * r;                  // r = 1 / (xi (1 - xi)) = 1 / xi + 1 / (1 - xi)
    const auto &c = tab->c[interval(log(d), tau)];
    S = kInvSqrt3Pi * ((r - 2.0) * series(c[fK23], tau) + series(c[fI13], tau)) * exp(-d);
  }
  return S * xi * om;
}

__device__ __forceinline__ double hermite(double tau, double p0, double p1, double d0, double d1,
                                          double ds) {
  const double t2 = tau * tau, t3 = t2 * tau;
  return (2 * t3 - 3 * t2 + 1) * p0 + (t3 - 2 * t2 + tau) * ds * d0 + (-2 * t3 + 3 * t2) * p1 +
         (t3 - t2) * ds * d1;
}

__device__ __forceinline__ double chi_node(int i, int n, double lo, double hi) {
  return exp(log(lo) + i * ((log(hi) - log(lo)) / (n - 1)));
}

struct TabOut {
  const FunTab *tab;
  double *rad_lnh, *rad_S, *pair_L, *pair_S;
  float *rad_lnh32, *rad_s0sc, *pair_L32, *pair_s0sc;
  uint16_t *rad_q16, *pair_q16;
  float *chk;
  double rad_hi, pair_hi;
  double rad_tlo, rad_dt, pair_tlo, pair_dt;
};

constexpr int kRowM = 1024, kRowThreads = 256;

// Row of 256 quantiles (thread k: quantile k) with its 16-bit copy; F the
// cumulative spectrum in units of its total, rho the density in the same units.
template <bool Rad>
__device__ __forceinline__ void write_quantiles(const TabOut &o, int row, const double *P, const double *rho,
                                                double slo, double shi, double ds, double *ends) {
  const int k = threadIdx.x;
  const double t = Rad ? o.rad_tlo + k * o.rad_dt : o.pair_tlo + k * o.pair_dt;
  const double u = 1.0 / (1.0 + exp(-t));
  double s;
  if (u <= P[0]) {
    if (Rad) {
      const double xi_lo = 1.0 / (1.0 + exp(-slo));
      const double r = u / P[0], xi = xi_lo * (r * r * r);
      s = log(xi) - log1p(-xi);
    } else {
      s = slo;
    }
  } else if (u >= P[kRowM]) {
    s = shi;
  } else {
    // largest m with P[m] <= u
    int lo = 0, hi = kRowM;           // P[lo] <= u < P[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (P[mid] <= u) lo = mid; else hi = mid;
    }
    const int m = lo;
    const double p0 = P[m], p1 = P[m + 1], d0 = rho[m], d1 = rho[m + 1];
    double a = 0.0, b = 1.0;
    for (int it = 0; it < 52; ++it) {
      const double mid = 0.5 * (a + b);
      if (hermite(mid, p0, p1, d0, d1, ds) < u) a = mid; else b = mid;
    }
    s = (slo + m * ds) + 0.5 * (a + b) * ds;
  }
  (Rad ? o.rad_S : o.pair_S)[row * kNU + k] = s;
  // 16-bit copy: q = round((s - s_0) / step)
  if (k == 0) ends[0] = s;
  if (k == kNU - 1) ends[1] = s;
  __syncthreads();
  const double s0 = ends[0], step = (ends[1] - s0) / 65535.0;
  double v = rint((s - s0) / step);
  v = fmin(fmax(v, 0.0), 65535.0);
  (Rad ? o.rad_q16 : o.pair_q16)[row * kNU + k] = (uint16_t)v;
  float *sc = Rad ? o.rad_s0sc : o.pair_s0sc;
  if (k == 0) { sc[2 * row] = (float)s0; sc[2 * row + 1] = (float)step; }
}

// One workgroup per row: 256 photon rows, then 512 pair rates, then 256 pair
// CDF rows.  Densities, cumulative sum, quantiles and the float32 and 16-bit
// copies stay in the workgroup (16 KB of LDS); its time is the
// reads of the series (a wave's points lie in about twenty intervals): 45 us for
// the 4 million densities, beside 22 us for the Bessel functions and 16 for the J.
// Building and reading back the tables of Eq. (4) takes 0.21 ms, half of it the
// copies; integrating the functions anew at every point took 363 ms (Eq. (1): 4.4).
template <int Formula>
__global__ __launch_bounds__(kRowThreads) void k_rows(TabOut o) {
  static_assert(kRowThreads == kNU && kRowM == 4 * kRowThreads, "a thread sums four intervals and makes one quantile");
  __shared__ double F[kRowM + 1], rho[kRowM + 1], part[kRowThreads / 64], ends[2];
  const int tid = threadIdx.x;
  const bool rad = blockIdx.x < kRadNChi;
  const bool rate = !rad && blockIdx.x < kRadNChi + kPairNRate;
  const int row = rad ? blockIdx.x : (rate ? blockIdx.x - kRadNChi : blockIdx.x - kRadNChi - kPairNRate);
  const double chi = rad ? chi_node(row, kRadNChi, kRadChiMin, o.rad_hi)
                         : chi_node(row, rate ? kPairNRate : kPairNCdf, kPairChiMin, o.pair_hi);
  double xi_lo, s_hi, tail;
  if (rad) {
    xi_lo = kRadXiLoOverChi * chi;
    s_hi = log(1.5 * kRadDHi * chi);
    tail = kInvSqrt3Pi * 3.0 * kGamma23 * pow(3.0 * chi, 2.0 / 3.0) * pow(xi_lo, 1.0 / 3.0);
  } else {
    const double q = 2.0 / (8.0 + 3.0 * chi * kPairDD);
    xi_lo = 2.0 * q / (1.0 + sqrt(1.0 - 4.0 * q));
    s_hi = 0.0;
    tail = 0.0;
  }
  const double s_lo = log(xi_lo) - log1p(-xi_lo), ds = (s_hi - s_lo) / kRowM;
  const double k = rad ? arg_scale<Formula>(chi) : arg_scale<kPair>(chi), lk = log(k);
  auto dens = [&](double s) {
    return rad ? density<Formula>(o.tab, s, k, lk) : density<kPair>(o.tab, s, k, lk);
  };
  // interval sums into F[m + 1], node densities into rho[m]
  const double g = 0.5 * sqrt(0.6);
#pragma unroll 1
  for (int q = 0; q < 3; ++q) {
#pragma unroll 1
    for (int m = tid; m < kRowM; m += kRowThreads) {
      const double d = dens((s_lo + m * ds) + ds * (0.5 + (q - 1) * g)) * (q == 1 ? 8.0 / 18.0 : 5.0 / 18.0);
      F[m + 1] = q ? F[m + 1] + d : d;
    }
  }
  if (!rate) {
#pragma unroll 1
    for (int m = tid; m <= kRowM; m += kRowThreads) rho[m] = dens(s_lo + m * ds);
  }
  __syncthreads();
  // cumulative sum: four intervals per thread, then the threads of a wave, then the waves
  double v[4], sum = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) { sum += ds * F[4 * tid + k + 1]; v[k] = sum; }
  double incl = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double t = __shfl_up(incl, d, 64);
    if ((tid & 63) >= d) incl += t;
  }
  if ((tid & 63) == 63) part[tid >> 6] = incl;
  __syncthreads();
  double base = tail, total = tail;
#pragma unroll
  for (int w = 0; w < kRowThreads / 64; ++w) {
    if (w < (tid >> 6)) base += part[w];
    total += part[w];
  }
  if (rate) {
    if (tid == 0) {
      const double L = log(2.0 * total) + 8.0 / (3.0 * chi);
      o.pair_L[row] = L;
      o.pair_L32[row] = (float)L;
    }
    return;
  }
  base += __shfl_up(incl, 1, 64) * ((tid & 63) ? 1.0 : 0.0);
#pragma unroll
  for (int k = 0; k < 4; ++k) F[4 * tid + k + 1] = (base + v[k]) / total;
  if (tid == 0) F[0] = tail / total;
  if (tid == kRowThreads - 1) F[kRowM] = 1.0;
  for (int m = tid; m <= kRowM; m += kRowThreads) rho[m] /= total;
  if (rad && tid == 0) {
    const double lnh = log(total);
    o.rad_lnh[row] = lnh;
    o.rad_lnh32[row] = (float)lnh;
  }
  __syncthreads();
  if (rad && tid < 40) {
    // residual-check row of the surrogate: P and dP/ds at 40 nodes uniform in s
    // over the fine grid, from the fine cubic Hermite interpolant
    constexpr int NC = 40;
    const double dsc = (s_hi - s_lo) / (NC - 1);
    const double sc = s_lo + tid * dsc;
    int m = (int)floor((sc - s_lo) / ds);
    m = m < 0 ? 0 : (m > kRowM - 1 ? kRowM - 1 : m);
    const double tau = (sc - (s_lo + m * ds)) / ds;
    const double p0 = F[m], p1 = F[m + 1], r0 = rho[m], r1 = rho[m + 1];
    const double t2 = tau * tau;
    const double P = hermite(tau, p0, p1, r0, r1, ds);
    const double dP = ((6 * t2 - 6 * tau) * p0 + (3 * t2 - 4 * tau + 1) * ds * r0 + (-6 * t2 + 6 * tau) * p1 +
                       (3 * t2 - 2 * tau) * ds * r1) / ds;
    float *r = o.chk + row * (2 + 2 * NC);
    if (tid == 0) { r[0] = (float)s_lo; r[1] = (float)dsc; }
    r[2 + 2 * tid] = (float)P;
    r[3 + 2 * tid] = (float)dP;
  }
  if (rad) write_quantiles<true>(o, row, F, rho, s_lo, s_hi, ds, ends);
  else write_quantiles<false>(o, row, F, rho, s_lo, s_hi, ds, ends);
}

}  // namespace

hipError_t launch_build_tables(qed_ctx *c, int formula, TabRange rg, hipStream_t st) {
  FunTab *tab = reinterpret_cast<FunTab *>(c->tab_work);
  TabOut o;
  o.tab = tab;
  o.rad_lnh = c->rad_lnh64; o.rad_S = c->rad_S64; o.pair_L = c->pair_L64; o.pair_S = c->pair_S64;
  o.rad_lnh32 = c->rad_lnh32; o.rad_s0sc = c->rad_s0sc; o.pair_L32 = c->pair_L32; o.pair_s0sc = c->pair_s0sc;
  o.rad_q16 = c->rad_q16; o.pair_q16 = c->pair_q16;
  o.chk = c->rad_chk;
  o.rad_hi = rg.rad_hi; o.pair_hi = rg.pair_hi;
  const double rtlo = log(kRadULo) - log1p(-kRadULo), rthi = log(kRadUHi) - log1p(-kRadUHi);
  const double ptlo = log(kPairULo) - log1p(-kPairULo), pthi = log(kPairUHi) - log1p(-kPairUHi);
  o.rad_tlo = rtlo; o.rad_dt = (rthi - rtlo) / (kNU - 1);
  o.pair_tlo = ptlo; o.pair_dt = (pthi - ptlo) / (kNU - 1);
  if (formula == QED_FORMULA_CLASSICAL)
    hipLaunchKernelGGL(k_bessel<true>, dim3(kIntervals), dim3(64 * kTerms), 0, st, tab);
  else
    hipLaunchKernelGGL(k_bessel<false>, dim3(kIntervals), dim3(64 * kTerms), 0, st, tab);
  const dim3 rows(kRadNChi + kPairNRate + kPairNCdf);
  if (formula == QED_FORMULA_II) {
    // sigma only reaches 20 (Eq. 4 at the upper end of the rows)
    const int n = (int)((log(20.0) - kYLo) / kYStep) + 2;
    hipLaunchKernelGGL(k_jfun, dim3(n), dim3(64 * kTerms), 0, st, tab);
    hipLaunchKernelGGL(k_rows<kFormulaII>, rows, dim3(kRowThreads), 0, st, o);
  } else if (formula == QED_FORMULA_CLASSICAL) {
    hipLaunchKernelGGL(k_rows<kClassical>, rows, dim3(kRowThreads), 0, st, o);
  } else {
    hipLaunchKernelGGL(k_rows<kFormulaI>, rows, dim3(kRowThreads), 0, st, o);
  }
  return hipGetLastError();
}

}  // namespace qed
