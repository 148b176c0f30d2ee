// simr_bk.hpp -- Broadie and Kaya's exact simulation of one Heston step, in FP64 device code.
//
//   V_t | v_u   = c X, X noncentral chi-square (4 kappa theta / xi^2 degrees of freedom,
//                 noncentrality v_u e^{-kappa dt} / c, c = xi^2 (1 - e^{-kappa dt}) / (4 kappa)),
//                 drawn by inverting its Poisson-mixture CDF at the uniform of word 2;
//   I | v_u, V_t  the integrated variance, drawn by inverting at the uniform of word 3 the CDF
//                 that the trapezoid rule gives from the conditional characteristic function
//                 (the Bessel-bridge law of the CIR process);
//   x_t = x_u + r dt - I / 2 + rho (V_t - v_u - kappa theta dt + kappa I) / xi
//         + sqrt((1 - rho^2) I) Z2.
// xi = 0: the deterministic CIR mean and its exact integral (rho taken as 0).  The FP32 path
// state is widened to FP64 for the step and rounded back.  The series for the Bessel function
// keeps full accuracy while its argument stays moderate (few large steps: the scheme's use as
// an accuracy reference); roots are found to ~1e-13 relative.
//
// Bound by FP64 issue of the characteristic function.  The variance draw stays one path per
// lane; the integrated-variance draw takes the wave's 64 paths one after another and spreads a
// path's M frequencies (80 to 4,096, by the option) over the lanes: each value is computed once
// and kept for the root search, where every lane had recomputed all M of its own path in each of
// its ~8 iterations and the wave waited for its largest M.  One step of 65,536 paths took 416 ms
// that way and takes 6.8 ms so, the same FP32 states bit for bit.
#pragma once

#include <hip/hip_runtime.h>

namespace simr {
namespace bk {

struct cplx {
  double re, im;
};
__device__ __forceinline__ cplx cx(double re, double im = 0.0) { return cplx{re, im}; }
__device__ __forceinline__ cplx operator+(cplx a, cplx b) { return cx(a.re + b.re, a.im + b.im); }
__device__ __forceinline__ cplx operator-(cplx a, cplx b) { return cx(a.re - b.re, a.im - b.im); }
__device__ __forceinline__ cplx operator*(cplx a, cplx b) {
  return cx(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
__device__ __forceinline__ cplx operator*(double s, cplx a) { return cx(s * a.re, s * a.im); }
__device__ __forceinline__ cplx cdiv(cplx a, cplx b) {  // scaled to avoid overflow
  const double s = fmax(fabs(b.re), fabs(b.im));
  const double br = b.re / s, bi = b.im / s;
  const double d = br * br + bi * bi;
  return cx((a.re * br + a.im * bi) / (s * d), (a.im * br - a.re * bi) / (s * d));
}
__device__ __forceinline__ double cabs_(cplx a) { return hypot(a.re, a.im); }
__device__ __forceinline__ cplx cexp_(cplx a) {
  const double m = exp(a.re);
  double s, c;
  sincos(a.im, &s, &c);
  return cx(m * c, m * s);
}
__device__ __forceinline__ cplx clog_(cplx a) { return cx(log(cabs_(a)), atan2(a.im, a.re)); }
__device__ __forceinline__ cplx csqrt_(cplx a) {  // principal branch (non-negative real part)
  const double m = cabs_(a);
  const double re = sqrt(0.5 * (m + a.re));
  const double im = sqrt(fmax(0.5 * (m - a.re), 0.0));
  return cx(re, a.im < 0.0 ? -im : im);
}

// Regularised lower incomplete gamma P(a, x).  Below x = a + 1 the power series
//   P = x^a e^{-x} / Gamma(a + 1) * sum_k x^k / ((a + 1)(a + 2)...(a + k)).
// Above it P = 1 - Q, with the upper function Q = x^a e^{-x} / (Gamma(a) g) and g the continued
// fraction g = b_0 + a_1/(b_1 + a_2/(b_2 + ...)), b_j = x + 2j + 1 - a, a_j = -j (j - a)
// (Legendre's fraction for the upper incomplete gamma function, in its even contraction).  g is
// evaluated front to back by the modified Lentz algorithm (W. J. Lentz, Applied Optics 15, 1976;
// I. J. Thompson and A. R. Barnett, J. Comput. Phys. 64, 1986): f_j = f_{j-1} C_j D_j with
// C_j = b_j + a_j / C_{j-1} and D_j = 1 / (b_j + a_j D_{j-1}), starting from f_0 = C_0 = b_0,
// D_0 = 0, any zero denominator replaced by a tiny number, until C_j D_j is 1 to rounding.
__device__ inline double inc_gamma_p(double a, double x) {
  if (!(x > 0.0)) return 0.0;
  const double log_pref = a * log(x) - x - lgamma(a);  // ln(x^a e^{-x} / Gamma(a))
  if (x < a + 1.0) {
    double ratio = 1.0, total = 1.0;  // k = 0 term of the sum; the 1/a goes into the prefactor
    for (int k = 1; k < 20000; ++k) {  // a + k > x after at most ~x terms; bounded regardless
      ratio *= x / (a + (double)k);
      total += ratio;
      if (ratio < total * 1e-17) break;
    }
    return total * exp(log_pref) / a;
  }
  constexpr double kTiny = 1e-300;
  const double b0 = x + 1.0 - a;
  double f = fabs(b0) < kTiny ? kTiny : b0;
  double C = f, D = 0.0;
  for (int j = 1; j < 20000; ++j) {
    const double aj = -(double)j * ((double)j - a);
    const double bj = b0 + 2.0 * (double)j;
    D = bj + aj * D;
    D = 1.0 / (fabs(D) < kTiny ? kTiny : D);
    C = bj + aj / C;
    if (fabs(C) < kTiny) C = kTiny;
    const double step = C * D;
    f *= step;
    if (fabs(step - 1.0) < 1e-16) break;
  }
  return 1.0 - exp(log_pref) / f;
}

// CDF F and density f at v of c X, X noncentral chi-square(df, lam): Poisson(m = lam / 2) weights w_j
// over central chi-squares, the mixture truncated 12 standard deviations either side.  With
// a_j = df / 2 + j, y = v / (2 c) and G_j = y^{a_j} e^{-y} / Gamma(a_j + 1), P(a, y) = P(a + 1, y) +
// y^a e^{-y} / Gamma(a + 1) gives P(a_j, y) = P(a_top, y) + sum_{i >= j} G_i, so
//   F = P(a_top, y) sum_j w_j + sum_i G_i (w_lo + ... + w_i),   f = sum_j w_j G_j a_j / y / (2 c),
// sums of positive terms with w_{j+1} = w_j m / (j + 1) and G_{j+1} = G_j y / a_{j+1}: one incomplete
// gamma function per evaluation, where one per Poisson term had been the cost of this draw.
__device__ inline void ncx2_cdf_pdf(double v, double c, double df, double lam, double& F, double& f) {
  const double y = v / (2.0 * c);
  const double m = 0.5 * lam;
  int jlo = 0, jhi = 0;
  double w = 1.0;
  if (m > 0.0) {
    const double sd = sqrt(m);
    jlo = (int)fmax(0.0, floor(m - 12.0 * sd - 10.0));
    jhi = (int)ceil(m + 12.0 * sd + 10.0);
    w = exp(-m + (double)jlo * log(m) - lgamma((double)jlo + 1.0));
  }
  F = 0.0;
  f = 0.0;
  if (!(y > 0.0)) return;
  double a = 0.5 * df + (double)jlo;
  double G = exp(a * log(y) - y - lgamma(a + 1.0));
  double W = 0.0, s = 0.0, sp = 0.0;
  for (int j = jlo; j <= jhi; ++j) {
    W += w;
    s += G * W;
    sp += w * G * a;
    w *= m / (double)(j + 1);
    a += 1.0;
    G *= y / a;
  }
  F = W * inc_gamma_p(a, y) + s;
  f = sp / y / (2.0 * c);
}

// A Newton step of this relative size is the last: the iteration converges quadratically, so the
// root it leads to is off by its square.
constexpr double kLastStep = 1e-9;

// The exact variance draw: safeguarded Newton on F(e^y) = u in y = ln V.
__device__ inline double variance(double v, double kappa, double theta, double xi, double dt, double u) {
  const double E = exp(-kappa * dt);
  if (!(xi > 0.0)) return theta + (v - theta) * E;
  const double c = xi * xi * (1.0 - E) / (4.0 * kappa);
  const double df = 4.0 * kappa * theta / (xi * xi);
  const double lam = v * E / c;
  const double mean = c * (df + lam), sd = c * sqrt(2.0 * (df + 2.0 * lam));
  double lo = log(1e-300), hi = log(mean + 40.0 * sd), y = log(mean);
  for (int it = 0; it < 200; ++it) {
    const double x = exp(y);
    double F, f;
    ncx2_cdf_pdf(x, c, df, lam, F, f);
    if (F < u) lo = y; else hi = y;
    double yn = y - (F - u) / (f * x);
    const bool newton = f * x > 0.0 && yn > lo && yn < hi;
    if (!newton) yn = 0.5 * (lo + hi);
    if ((newton && fabs(yn - y) <= kLastStep) || hi - lo <= 1e-14) return exp(yn);
    y = yn;
  }
  return exp(y);
}

// ln S(z), S(z) = sum_k (z^2/4)^k / (k! Gamma(k + nu + 1)) (I_nu(z) = (z/2)^nu S(z)), the terms
// scaled by e^{-|z|}.
__device__ inline cplx log_bessel_series(cplx z, double nu) {
  const double az = cabs_(z);
  const cplx q = 0.25 * (z * z);
  cplx t = cx(exp(-az - lgamma(nu + 1.0))), s = t;
  const int kmax = (int)fmin(4.0 * az, 1e6) + 2000;  // bounded also for non-finite input
  for (int k = 1; k < kmax; ++k) {
    const double ik = 1.0 / ((double)k * ((double)k + nu));
    t = cx((t.re * q.re - t.im * q.im) * ik, (t.re * q.im + t.im * q.re) * ik);
    s = s + t;
    const double at = fabs(t.re) + fabs(t.im);  // within sqrt(2) of |t|
    if (((double)k > az && at < 1e-18 * (fabs(s.re) + fabs(s.im))) || !(at == at)) break;
  }
  return cx(az) + clog_(s);
}

// ln E[exp(i a I) | v_u, v_t]: with g = sqrt(kappa^2 - 2 xi^2 i a) and the ratio
// r = z(g) / z(kappa) = (g / kappa) e^{-(g - kappa) dt / 2} (1 - e^{-kappa dt}) / (1 - e^{-g dt})
// (its logarithm summed from principal logarithms of factors with positive real part, so the
// phase is continuous in a):  ln r + (v_u + v_t) / xi^2 [kappa coth-term - g coth-term]
// + nu ln r + ln S(z0 r) - ln S(z0).
struct CfConst {
  double kappa, xi, dt, nu, ek, ckap, z0, ls0, vs;
};

__device__ inline cplx log_cf(const CfConst& k, double a) {
  const cplx g = csqrt_(cx(k.kappa * k.kappa, -2.0 * k.xi * k.xi * a));
  const cplx eg = cexp_(cx(-g.re * k.dt, -g.im * k.dt));
  const cplx one_m_eg = cx(1.0 - eg.re, -eg.im);
  const cplx lr = clog_(cx(g.re / k.kappa, g.im / k.kappa)) - cx(0.5 * (g.re - k.kappa) * k.dt, 0.5 * g.im * k.dt) +
                  cx(log(1.0 - k.ek)) - clog_(one_m_eg);
  const cplx coth_g = cdiv(g * cx(1.0 + eg.re, eg.im), one_m_eg);
  cplx l = (1.0 + k.nu) * lr + (k.vs / (k.xi * k.xi)) * (cx(k.ckap) - coth_g);
  if (k.z0 > 0.0) l = l + log_bessel_series(k.z0 * cexp_(lr), k.nu) - cx(k.ls0);
  return l;
}

// The lanes that share a path's frequencies: the whole wave, all lanes active.
struct WaveLanes {
  static constexpr int kLanes = 64;
  static __device__ __forceinline__ int lane() { return (int)(threadIdx.x & 63u); }
  static __device__ __forceinline__ uint64_t ballot(bool b) { return __ballot(b); }
  static __device__ __forceinline__ double from(double x, int l) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
  }
  static __device__ __forceinline__ double sum(double x) {  // a fixed butterfly: the same bits in every lane
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
  }
};

// The integrated-variance draw of every lane's path: Newton (safeguarded by bisection on [0, u_e])
// on the trapezoid CDF F(x) = h x / pi + (2 / pi) sum_{j=1..M} sin(h j x) / j Re phi(h j), period
// 2 pi / h = 2 u_e, u_e = mu + 20 sd from the characteristic function near 0, M where
// |phi(h j)| / j < pi 1e-13 / 2 (at most kMaxFreq).  Called by whole waves with one option's constants;
// the constants of each path's law are formed by its own lane, then the paths go one after
// another, lane i taking the frequencies j = i + 1 + kLanes b: the sines and cosines of a lane's
// terms follow each other by the rotation through kLanes h x.
constexpr int kMaxFreq = 4096;

template <class Lanes>
__device__ inline double integrated_variance(double vu, double vt, double kappa, double theta, double xi,
                                             double dt, double u) {
  if (!(xi > 0.0)) return theta * dt + (vu - theta) * (1.0 - exp(-kappa * dt)) / kappa;
  CfConst k;
  k.kappa = kappa;
  k.xi = xi;
  k.dt = dt;
  k.nu = 2.0 * kappa * theta / (xi * xi) - 1.0;
  k.ek = exp(-kappa * dt);
  k.ckap = kappa * (1.0 + k.ek) / (1.0 - k.ek);
  k.vs = vu + vt;
  k.z0 = (vu > 0.0 && vt > 0.0) ? sqrt(vu * vt) * 4.0 * kappa * exp(-0.5 * kappa * dt) / (xi * xi * (1.0 - k.ek))
                                : 0.0;
  k.ls0 = k.z0 > 0.0 ? log_bessel_series(cx(k.z0), k.nu).re : 0.0;
  const double guess = 0.5 * (vu + vt) * dt + 1e-12;
  const double ea = 1e-4 / guess;
  const cplx p = cexp_(log_cf(k, ea));
  const double mu = p.im / ea;
  const double m2 = 2.0 * (1.0 - p.re) / (ea * ea);
  const double sd = sqrt(fmax(m2 - mu * mu, 1e-6 * mu * mu));
  const bool usable = mu > 0.0 && sd < 1e300;
  double drawn = guess;  // no usable moments: the trapezoid value
  const double ue_own = mu + 20.0 * sd;
  const uint64_t todo = Lanes::ballot(usable);
  constexpr int kBlocks = kMaxFreq / Lanes::kLanes;
  double re[kBlocks], rej[kBlocks];  // Re phi(h j) and Re phi(h j) / j of the lane's frequencies
  const int lane = Lanes::lane();
  for (int l = 0; l < Lanes::kLanes; ++l) {
    if (!((todo >> l) & 1u)) continue;
    CfConst kl = k;  // the constants of lane l's path
    kl.vs = Lanes::from(k.vs, l);
    kl.z0 = Lanes::from(k.z0, l);
    kl.ls0 = Lanes::from(k.ls0, l);
    const double ue = Lanes::from(ue_own, l), mul = Lanes::from(mu, l), ul = Lanes::from(u, l);
    const double h = M_PI / ue;
    int nb = 0;
    for (bool done = false; !done && nb < kBlocks; ++nb) {
      const double j = (double)(nb * Lanes::kLanes + lane + 1);
      const cplx lp = log_cf(kl, h * j);
      const double mag = exp(lp.re);
      const uint64_t small = Lanes::ballot(mag / j < M_PI * 1e-13 / 2.0);
      done = small != 0;
      const bool past = done && lane > __builtin_ctzll(small);  // beyond M
      re[nb] = past ? 0.0 : mag * cos(lp.im);
      rej[nb] = re[nb] / j;
    }
    double lo = 0.0, hi = ue, x = mul;
    for (int it = 0; it < 100; ++it) {  // bisection alone reaches 1e-14 mu in about 50 steps
      double s, c, sr, cr;
      sincos((double)(lane + 1) * (h * x), &s, &c);
      sincos((double)Lanes::kLanes * (h * x), &sr, &cr);
      double F = 0.0, f = 0.0;
      for (int b = 0; b < nb; ++b) {
        F += s * rej[b];
        f += c * re[b];
        const double sn = s * cr + c * sr;
        c = c * cr - s * sr;
        s = sn;
      }
      F = h * x / M_PI + 2.0 / M_PI * Lanes::sum(F);
      f = h / M_PI + 2.0 * h / M_PI * Lanes::sum(f);
      if (F < ul) lo = x; else hi = x;
      double xn = x - (F - ul) / f;
      const bool newton = f > 0.0 && xn > lo && xn < hi;
      if (!newton) xn = 0.5 * (lo + hi);
      const bool last = (newton && fabs(xn - x) <= kLastStep * mul) || hi - lo <= 1e-14 * mul;
      x = xn;
      if (last) break;
    }
    if (lane == l) drawn = x;
  }
  return drawn;
}

}  // namespace bk
}  // namespace simr
