// Device pieces of the neutrino response shared by the exact and the surrogate kernels
// (FP64, one workgroup of NT threads per (k-bin, box): RT = 256 when there are few
// (bin, box) pairs to spread over the chip, one wave when there are many).
#pragma once
#include "pm_nu_internal.hpp"

namespace pmnu {

constexpr int RT = 256;

// Rational fit of the free-streaming kernel I(x), the paper's Appendix C eq. (fit).
// x^4.1811 is taken as x^4 2^(0.1811 log2 x): FP64 to a few ulp, and cheaper than pow,
// whose extra-precision logarithm the small fractional exponent does not need.
__device__ __forceinline__ double i_fit_l2(double x, double l2x) {   // l2x = log2 x
  const double x2 = x * x, x4 = x2 * x2;
  const double num = 1.0 + 0.0168 * x2 + 0.0407 * x4;
  const double xp = x > 0.0 ? x4 * exp2(0.1811 * l2x) : 0.0;
  const double den = 1.0 + 2.1734 * x2 + 1.6787 * xp + 0.1467 * x4 * x4;
  return num / den;
}
__device__ __forceinline__ double i_fit(double x) {
  return i_fit_l2(x, x > 0.0 ? log2(x) : 0.0);
}

// 1 / d by Newton's method from the hardware's estimate, for 1e-300 < d < 1e300 (5 instructions;
// a division, which also serves the ends of the range, is 11).
__device__ __forceinline__ double rcp_newton(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  return fma(r, fma(-d, r, 1.0), r);
}

// The exact kernel of Appendix C, I(x) = 4/(3 zeta(3)) sum_{n>=1} (-1)^{n+1} f(n),
// f(n) = n/(n^2+x^2)^2 = Im (n - ix)^{-2} / (2x): the terms n < N = 13 one by one, the rest by
// the Euler-Boole summation formula (Borwein, Calkin and Manna, Amer. Math. Monthly 116 (2009)
// 387), sum_{m>=0} (-1)^m f(N+m) ~ 1/2 sum_k E_k(0)/k! f^(k)(N), whose terms
// f^(k)(N) = (-1)^k (k+1)!/2 b_{k+2}, b_j = Im (N - ix)^{-j} / x, it takes up to k = 23.
//   - Terms n, n+1 (D, E their n^2 + x^2) are one fraction,
//     [n (2n+1)^2 + D (2n (2n+1) - D)] / (D E)^2, which takes the cancellation between them out
//     in the polynomial; two such pairs share a reciprocal.
//   - f(N)/2 = N q / 2, q = 1/(N^2 + x^2)^2, goes in as q / 2 and one q with each pair: for
//     large x a pair is -1/x^4 and the whole sum 1/(4 x^4), so the partial sums stay small.
//   - b_{j+2} = p b_j - q b_{j-2} with p = 2 Re (N - ix)^{-2}: Clenshaw's summation over the
//     odd j, two operations a term.
// Relative error, rounding and the first term left out: below 2e-14 (the seven fractions and the
// tail cancel by a factor of up to 15; the largest of ten million x up to 1e4 was 1.7e-14, and
// 1.4e-13 of a sum of 32 accelerated terms with a division each).
// Bound by FP64 arithmetic: the response of 16 boxes x 128 bins, 300 nodes of 8 sub-nodes, three
// masses (14.7 M values of I) 294 -> 91 us.
constexpr int kSeriesN = 13, kSeriesTail = 12;
// E_k(0) (-1)^k (k+1) / 4 = (2^{k+1} - 1) B_{k+1} / 2 for k = 1, 3, ..., 23
constexpr double kSeriesTailC[kSeriesTail] = {
    0.25,       -0.25,        0.75,       -4.25,         38.75,          -518.25,
    9556.75,    -232392.25,   7205154.75, -277413226.25, 12985820432.75, -726287760620.25};

__device__ __forceinline__ double i_series(double x) {
  constexpr double C = 4.0 / (3.0 * 1.2020569031595942);
  constexpr double N = kSeriesN;
  const double x2 = x * x;
  // beyond the range of the products below the sum is its leading term 1 / (4 x^4)
  if (x2 > 1e70) return 0.25 * C / x2 / x2;
  const double r = rcp_newton(N * N + x2), q = r * r, p = 2.0 * (N * N - x2) * q;
  double y1 = 0.0, y2 = 0.0;
#pragma unroll
  for (int i = kSeriesTail - 1; i >= 0; --i) {
    const double y = fma(p, y1, fma(-q, y2, kSeriesTailC[i]));
    y2 = y1;
    y1 = y;
  }
  const double b3 = q * r * (3.0 * N * N - x2);
  double s = fma(y1, b3, fma(-q * y2, r, 0.5 * q));
#pragma unroll
  for (int i = kSeriesN - 2; i >= 3; i -= 4) {      // the pairs from i and i - 2: small terms first
    const double n = i, m = i - 2;
    const double d1 = n * n + x2, e1 = (n + 1.0) * (n + 1.0) + x2;
    const double d2 = m * m + x2, e2 = (m + 1.0) * (m + 1.0) + x2;
    const double p1 = d1 * e1, p2 = d2 * e2;
    const double rr = rcp_newton(p1 * p2), r1 = rr * p2, r2 = rr * p1;
    const double a1 = fma(d1, 2.0 * n * (2.0 * n + 1.0) - d1, n * (2.0 * n + 1.0) * (2.0 * n + 1.0));
    const double a2 = fma(d2, 2.0 * m * (2.0 * m + 1.0) - d2, m * (2.0 * m + 1.0) * (2.0 * m + 1.0));
    s = fma(a1, r1 * r1, s + q);
    s = fma(a2, r2 * r2, s + q);
  }
  return C * s;
}

template <bool SERIES>
__device__ __forceinline__ double i_kernel(double x) {
  if constexpr (SERIES) return i_series(x);
  else return i_fit(x);
}
// the same with log2 x known (the fit then needs no logarithm; the series ignores it)
template <bool SERIES>
__device__ __forceinline__ double i_kernel_l2(double x, double l2x) {
  if constexpr (SERIES) return i_series(x);
  else return i_fit_l2(x, l2x);
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum over the workgroup (NT threads); every thread gets the result.
template <int NT = RT>
__device__ __forceinline__ double block_sum_d(double v, double* red) {
  v = wave_sum_d(v);
  if constexpr (NT == 64) return v;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) s += red[w];
  return s;
}

// Two sums over the workgroup at once; every thread gets both.
template <int NT = RT>
__device__ __forceinline__ double2 block_sum_d2(double2 v, double* red) {
  v.x = wave_sum_d(v.x);
  v.y = wave_sum_d(v.y);
  if constexpr (NT == 64) return v;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) {
    red[2 * wave] = v.x;
    red[2 * wave + 1] = v.y;
  }
  __syncthreads();
  double2 s = make_double2(0.0, 0.0);
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    s.x += red[2 * w];
    s.y += red[2 * w + 1];
  }
  return s;
}

// Three sums over the workgroup at once; every thread gets them. red: 3 * NT / 64 doubles.
template <int NT>
__device__ __forceinline__ double3 block_sum_d3(double3 v, double* red) {
  v.x = wave_sum_d(v.x);
  v.y = wave_sum_d(v.y);
  v.z = wave_sum_d(v.z);
  if constexpr (NT == 64) return v;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    red[3 * wave] = v.x;
    red[3 * wave + 1] = v.y;
    red[3 * wave + 2] = v.z;
  }
  __syncthreads();
  double3 s = make_double3(0.0, 0.0, 0.0);
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    s.x += red[3 * w];
    s.y += red[3 * w + 1];
    s.z += red[3 * w + 2];
  }
  return s;
}

// sum over the per-workgroup partial mode sums of bin b ([box][bin][workgroup]):
// sum w |delta_k|^2
template <int NT = RT>
__device__ __forceinline__ double bin_mode_sum(const double* partial, int n_partial, int nbins,
                                               int box, int b, double* red) {
  // Each thread reads per = ceil(n_partial / NT) values at i = tid + NT u (coalesced for
  // every u), in as few rounds of at most U loads in flight as cover them, split evenly, so
  // that no round is a nearly empty one that would cost a memory latency of its own.
  constexpr int U = 16;
  const double* pp = partial + (static_cast<size_t>(box) * nbins + b) * n_partial;
  const int per = (n_partial + NT - 1) / NT;
  const int rounds = (per + U - 1) / U;
  const int chunk = rounds > 0 ? (per + rounds - 1) / rounds : 0;
  double s = 0.0;
  for (int u0 = 0; u0 < per; u0 += chunk) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = threadIdx.x + (u0 + u) * NT;
      v[u] = (u < chunk && i < n_partial) ? pp[i] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s += v[u];
  }
  return block_sum_d<NT>(s, red);
}

// eq. (P-final) for one bin: the initial-condition term plus the trapezoid sum over the
// sub-nodes, iterated `iterations` times on the current node (every thread gets it). With
// several species (mass hierarchy) each free-streams with its own kernel and the result is
// their mean weighted by m_s / M_nu; the source term is the common P_M^{1/2} history, so
// the quadrature uses the weighted sum of the kernels. ic_pnu: [kMaxSpecies][nbins] initial
// amplitudes of this box.
//
// The sum is linear in the unknown current node A_n = (1 - f_nu) P_cdm^{1/2} + f_nu P_nu^{1/2}
// (it enters only the last stored interval), so one pass gathers the part from the stored
// nodes and the coefficient of A_n; each iteration of Appendix B is then a scalar update
// and the kernel is evaluated once whatever the number of iterations. The initial-condition
// term is evaluated by the first wave only and enters the sum through thread 0. Each
// thread takes ceil(nq / NT) sub-nodes q = tid + NT u, in as few rounds of at most U
// whose loads go out together as cover them.
// exact_sums: this thread's share of the known part (x) and of the coefficient of A_n (y).
template <int NSP, bool SERIES, int NT>   // species: 1 (equal masses) or kMaxSpecies
__device__ __forceinline__ double2 exact_sums(const RespBox& bx, double k, const double* ic_pnu,
                                              double ic_theta, const double* hpm, int nbins,
                                              int b, const double* ds, const double* l2ds,
                                              const double* w, int q_sub) {
  const double inv_q = 1.0 / q_sub;
  // log2(k T/m_s) of each species: with log2(ds) per sub-node (host FP64) it gives the
  // fit's log2 x without a logarithm per sub-node
  double l2k[NSP];
#pragma unroll
  for (int sp = 0; sp < NSP; ++sp)
    l2k[sp] = (SERIES || !(sp < bx.n_sp) || !(k * bx.tm_sp[sp] > 0.0)) ? 0.0
                                                                       : log2(k * bx.tm_sp[sp]);
  double known = 0.0, coef = 0.0;
  if (threadIdx.x < 64) {                    // wave-uniform
    double ic = 0.0;
#pragma unroll
    for (int sp = 0; sp < NSP; ++sp)         // constant bound: the arrays stay in registers
      if (sp < bx.n_sp)
        ic += bx.w_sp[sp] * i_kernel<SERIES>(k * bx.tm_sp[sp] * bx.ds_ic) *
              ic_pnu[sp * nbins + b];
    ic *= 1.0 - bx.ds_ic * bx.a_i * ic_theta;
    if (threadIdx.x == 0) known = ic;
  }
  constexpr int U = 4;
  const int per = (bx.nq + NT - 1) / NT;
  const int rounds = (per + U - 1) / U;
  const int chunk = rounds > 0 ? (per + rounds - 1) / rounds : 0;
  for (int u0 = 0; u0 < per; u0 += chunk) {
    double d[U], l2d[U], wq[U], a0[U], a1[U];
    bool c0[U], c1[U];                       // the bracketing node is the current one
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = threadIdx.x + (u0 + u) * NT;
      const int j = q / q_sub;
      const bool in = u < chunk && q < bx.nq;
      d[u] = in ? ds[q] : 0.0;
      l2d[u] = (in && !SERIES) ? l2ds[q] : 0.0;
      wq[u] = in ? w[q] : 0.0;
      c0[u] = !(j < bx.n_cur);
      c1[u] = !(j + 1 < bx.n_cur);
      a0[u] = (in && !c0[u]) ? hpm[static_cast<size_t>(j) * nbins + b] : 0.0;
      a1[u] = (in && !c1[u]) ? hpm[static_cast<size_t>(j + 1) * nbins + b] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = threadIdx.x + (u0 + u) * NT;
      if (u >= chunk || q >= bx.nq) continue;
      const int j = q / q_sub, r = q - j * q_sub;
      const double t = r * inv_q;
      // amplitude = (1 - t) A_j + t A_{j+1}, with A_n split off
      const double amp = (r != 0) ? (1.0 - t) * a0[u] + t * a1[u] : a0[u];
      const double cur = (c0[u] ? (r != 0 ? 1.0 - t : 1.0) : 0.0) +
                         ((r != 0 && c1[u]) ? t : 0.0);
      double kern = 0.0;
#pragma unroll
      for (int sp = 0; sp < NSP; ++sp)
        if (sp < bx.n_sp)
          kern += bx.w_sp[sp] * i_kernel_l2<SERIES>(k * bx.tm_sp[sp] * d[u], l2k[sp] + l2d[u]);
      const double g = wq[u] * kern * d[u];
      known += g * amp;
      coef += g * cur;
    }
  }
  return make_double2(known, coef);
}
// the iterations of Appendix B from the workgroup's sums
__device__ __forceinline__ double exact_iterate(const RespBox& bx, double2 sums, double pcdm_half,
                                                double pnu_prev, int iterations) {
  double pnu_guess = pnu_prev, pnu = 0.0;
  for (int it = 0; it < iterations; ++it) {
    const double a_cur = (1.0 - bx.f_nu) * pcdm_half + bx.f_nu * pnu_guess;
    pnu = sums.x + sums.y * a_cur;
    pnu_guess = pnu;
  }
  return pnu;
}

// red: 2 * NT / 64 doubles
template <int NSP, bool SERIES, int NT>
__device__ __forceinline__ double exact_pnu_n(const RespBox& bx, double k, double pcdm_half,
                                              double pnu_prev, const double* ic_pnu,
                                              double ic_theta, const double* hpm, int nbins,
                                              int b, const double* ds, const double* l2ds,
                                              const double* w, int q_sub, int iterations,
                                              double* red) {
  const double2 part = exact_sums<NSP, SERIES, NT>(bx, k, ic_pnu, ic_theta, hpm, nbins, b, ds,
                                                   l2ds, w, q_sub);
  return exact_iterate(bx, block_sum_d2<NT>(part, red), pcdm_half, pnu_prev, iterations);
}

template <int NT = RT>
__device__ __forceinline__ double exact_pnu(const RespBox& bx, double k, double pcdm_half,
                                            double pnu_prev, const double* ic_pnu,
                                            double ic_theta, const double* hpm, int nbins,
                                            int b, const double* ds, const double* l2ds,
                                            const double* w, int q_sub, int iterations,
                                            double* red) {
  if (bx.n_sp <= 0) return 0.0;          // no massive neutrinos: the term drops out
#define PMNU_EXACT_PNU(NSP, SERIES)                                                        \
  exact_pnu_n<NSP, SERIES, NT>(bx, k, pcdm_half, pnu_prev, ic_pnu, ic_theta, hpm, nbins, b, ds, \
                               l2ds, w, q_sub, iterations, red)
  if (bx.series) {
    if (bx.n_sp == 1) return PMNU_EXACT_PNU(1, true);
    return PMNU_EXACT_PNU(kMaxSpecies, true);
  }
  if (bx.n_sp == 1) return PMNU_EXACT_PNU(1, false);
  return PMNU_EXACT_PNU(kMaxSpecies, false);
#undef PMNU_EXACT_PNU
}

}  // namespace pmnu
