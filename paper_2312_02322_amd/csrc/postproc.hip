// Cross-section post-processing (paper Section III): the microscopic-reversibility
// diagnostic of Eq. 19, the symmetrised cross sections of Eq. 20 and rate
// coefficients from them by Maxwell-Boltzmann averaging over a cubic spline
// through the computed collision energies.
//
// Rates, with beta = k_B T, g the level degeneracy and U the symmetrised
// translational energy (mean of initial and final kinetic energies):
//   k_{i->f} = (1/g_i) sqrt(8/(pi mu)) beta^(-3/2) exp(-(E_f - E_i)/(2 beta))
//              * int s(U) U exp(-U/beta) dU,
// s = natural cubic spline through (U_e, sigma~_e) on [U_1, U_n], a linear ramp
// from zero at the threshold |E_f - E_i|/2 up to U_1, sigma~(U_n) beyond U_n.
// The Boltzmann factor is taken relative to the threshold so that nothing
// overflows.  On every interval s(U) U is a polynomial of degree four, so the
// integral is a sum of moments of e^{-t} in closed form (see xs_rate_kernel); the
// constant tail beyond U_n likewise.
#include "internal.h"

#include <math.h>

#include <algorithm>

namespace mqct {

namespace {

__global__ void xs_sym_kernel(int nE, int L, const double* __restrict__ g,
                              const double* __restrict__ sigma, double* __restrict__ sym,
                              double* __restrict__ ratio) {
  const int64_t LL = (int64_t)L * L;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)nE * LL) return;
  const int64_t e = idx / LL;
  const int i = (int)((idx - e * LL) / L), f = (int)(idx - e * LL - (int64_t)i * L);
  const double lhs = g[i] * sigma[idx];
  const double rhs = g[f] * sigma[e * LL + (int64_t)f * L + i];
  if (sym) sym[idx] = 0.5 * (lhs + rhs);
  if (ratio) ratio[idx] = rhs != 0.0 ? lhs / rhs : __builtin_nan("");
}

constexpr int XS_NE_MAX = 64;
constexpr int RATE_BLOCK = 128;
constexpr int RATE_TC = 4;        // temperatures per thread
constexpr int SER_N = 32;         // terms of the moment series (z <= SER_Z)
constexpr double SER_Z = 5.0;

// mu_m = int_0^z t^m e^{-t} dt, m = 0..4, e = e^{-z}.  Short pieces: the series
//   mu_4 = z^5 e^{-z} sum_q z^q / (5 6 ... (5 + q)),
// whose terms are all positive, then mu_{m-1} = (mu_m + z^m e^{-z}) / m downward,
// also without cancellation.  Long ones: mu_0 = 1 - e^{-z} and upward.
__device__ __forceinline__ void rate_moments(double z, double e, const double* __restrict__ rcp,
                                             double (&mu)[5]) {
  z = fmin(z, 1e4);       // e is 0 from 746 on; z^4 stays finite
  const double z2 = z * z, z3 = z2 * z, z4 = z2 * z2;
  if (z <= SER_Z) {
    double s = 1.0;
    const int n = z <= 0.5 ? 12 : SER_N;
    for (int q = n; q >= 1; --q) s = fma(z * rcp[q], s, 1.0);
    mu[4] = z4 * z * e * 0.2 * s;
    mu[3] = (mu[4] + z4 * e) * 0.25;
    mu[2] = (mu[3] + z3 * e) * (1.0 / 3.0);
    mu[1] = (mu[2] + z2 * e) * 0.5;
    mu[0] = mu[1] + z * e;
  } else {
    mu[0] = 1.0 - e;
    mu[1] = mu[0] - z * e;
    mu[2] = 2.0 * mu[1] - z2 * e;
    mu[3] = 3.0 * mu[2] - z3 * e;
    mu[4] = 4.0 * mu[3] - z4 * e;
  }
}

// One thread per (i, f) and RATE_TC temperatures.  On each interval of the
// energies s(U) U is a quartic in U, so its integral against the Boltzmann factor
// is five moments of e^{-t}: one exponential per interval and temperature, where
// 8-point quadrature on pieces of 2 beta took about 240.  The second derivatives
// sit in LDS ([nE][threads], conflict free; the elimination factors depend on the
// energies only and are formed once per workgroup), so nothing spills to scratch.
// FP64 ALU bound.  1032 levels, 10 energies, 20 temperatures: 15.4 ms before,
// 0.80 ms after (inputs and outputs take 0.05 ms at the copy rate).
__global__ void __launch_bounds__(RATE_BLOCK)
xs_rate_kernel(int nE, int L, int nT, const double* __restrict__ Ug, const double* __restrict__ E,
               const double* __restrict__ g, const double* __restrict__ sym, double mu,
               const double* __restrict__ beta, double* __restrict__ k) {
  extern __shared__ double sh[];
  double* m2 = sh;                          // [nE][RATE_BLOCK]
  double* U = m2 + nE * RATE_BLOCK;         // [nE]
  double* fw = U + nE;                      // [nE] elimination multipliers
  double* fd = fw + nE;                     // [nE] reduced diagonal
  double* rcp = fd + nE;                    // [SER_N + 1] 1 / (5 + q)
  double* bt = rcp + SER_N + 1;             // [RATE_TC] beta
  double* bc = bt + RATE_TC;                // [RATE_TC] sqrt(8 / (pi mu)) beta^{-3/2}
  const int t0 = blockIdx.y * RATE_TC, nt = min(RATE_TC, nT - t0);
  for (int e = threadIdx.x; e < nE; e += RATE_BLOCK) U[e] = Ug[e];
  for (int q = threadIdx.x; q <= SER_N; q += RATE_BLOCK) rcp[q] = 1.0 / (5.0 + q);
  if ((int)threadIdx.x < RATE_TC) {
    const double b = beta[t0 + min((int)threadIdx.x, nt - 1)];
    bt[threadIdx.x] = b;
    bc[threadIdx.x] = sqrt(8.0 / (M_PI * mu)) * pow(b, -1.5);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double dprev = 0.0;
    for (int e = 1; e < nE - 1; ++e) {
      const double h0 = U[e] - U[e - 1], h1 = U[e + 1] - U[e];
      double d = (h0 + h1) / 3.0, w = 0.0;
      if (e > 1) {
        w = h0 / 6.0 / dprev;
        d -= w * (h0 / 6.0);
      }
      fw[e] = w;
      fd[e] = d;
      dprev = d;
    }
  }
  __syncthreads();
  const int64_t LL = (int64_t)L * L;
  const int64_t p = (int64_t)blockIdx.x * RATE_BLOCK + threadIdx.x;
  if (p >= LL) return;
  const int i = (int)(p / L), f = (int)(p - (int64_t)i * L);
  const double dE = E[f] - E[i];
  const double th = fabs(dE) * 0.5;
  const double* y = sym + p;
  // natural-spline second derivatives of sigma~_{if}(U_e) (Thomas elimination)
  double* c2 = m2 + threadIdx.x;
  c2[0] = 0.0;
  c2[(nE - 1) * RATE_BLOCK] = 0.0;
  {
    double rprev = 0.0;
    double yl = y[0], yc = y[LL];
    for (int e = 1; e < nE - 1; ++e) {
      const double yr = y[(e + 1) * LL];
      const double r = (yr - yc) / (U[e + 1] - U[e]) - (yc - yl) / (U[e] - U[e - 1]) -
                       fw[e] * rprev;
      c2[e * RATE_BLOCK] = r;
      rprev = r;
      yl = yc;
      yc = yr;
    }
    double next = 0.0;
    for (int e = nE - 2; e >= 1; --e) {
      next = (c2[e * RATE_BLOCK] - (U[e + 1] - U[e]) / 6.0 * next) / fd[e];
      c2[e * RATE_BLOCK] = next;
    }
  }
  double tot[RATE_TC], ex[RATE_TC];   // integrals, e^{-(a - th)/b} at the piece's start a
#pragma unroll
  for (int q = 0; q < RATE_TC; ++q) {
    tot[q] = 0.0;
    ex[q] = 1.0;
  }
  // [th, U_0] (the ramp), then the intervals of the spline; a piece below the
  // threshold is empty
  double yl = 0.0, ml = 0.0;
  for (int e = -1; e < nE - 1; ++e) {
    const double yr = y[(e + 1) * LL];
    const double mr = e < 0 ? 0.0 : c2[(e + 1) * RATE_BLOCK];
    const double lo = e < 0 ? th : U[e], hi = U[e + 1];
    const double a = fmax(lo, th), len = hi - a;
    if (len > 0.0) {
      // s(a + x) = s0 + s1 x + s2 x^2 + s3 x^3
      double s0, s1, s2, s3;
      if (e < 0) {
        s0 = 0.0; s1 = yr / len; s2 = 0.0; s3 = 0.0;
      } else {
        const double h = hi - lo;
        s3 = (mr - ml) / (6.0 * h);
        s2 = 0.5 * ml;
        s1 = (yr - yl) / h - h * (2.0 * ml + mr) / 6.0;
        s0 = yl;
        const double x = a - lo;       // shift to a (past the threshold)
        if (x > 0.0) {
          s0 = fma(x, fma(x, fma(x, s3, s2), s1), s0);
          s1 = fma(x, fma(x, 3.0 * s3, 2.0 * s2), s1);
          s2 = fma(3.0 * x, s3, s2);
        }
      }
      // s(U) U, U = a + x
      const double q0 = s0 * a, q1 = fma(s1, a, s0), q2 = fma(s2, a, s1), q3 = fma(s3, a, s2);
#pragma unroll
      for (int q = 0; q < RATE_TC; ++q) {
        const double b = bt[q], z = len / b;
        if (ex[q] == 0.0) continue;    // past the range of the exponential
        const double ez = exp(-z);
        double m[5];
        rate_moments(z, ez, rcp, m);
        const double v = fma(b, fma(b, fma(b, fma(b, s3 * m[4], q3 * m[3]), q2 * m[2]), q1 * m[1]),
                             q0 * m[0]);
        tot[q] = fma(ex[q] * b, v, tot[q]);
        ex[q] *= ez;
      }
    }
    yl = yr;
    ml = mr;
  }
  // the constant sigma~(U_n) beyond the last energy (or the threshold above it)
  const double Un = fmax(U[nE - 1], th);
#pragma unroll
  for (int q = 0; q < RATE_TC; ++q) {
    if (q >= nt) break;
    const double b = bt[q];
    const double total = ex[q] > 0.0 ? fma(ex[q] * b, yl * (Un + b), tot[q]) : tot[q];
    k[(int64_t)(t0 + q) * LL + p] = bc[q] * exp(-(th + 0.5 * dE) / b) * total / g[i];
  }
}

}  // namespace

hipError_t launch_xs_symmetrize(int nE, int L, const double* g, const double* sigma, double* sym,
                                double* ratio, hipStream_t s) {
  const int64_t n = (int64_t)nE * L * L;
  xs_sym_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(nE, L, g, sigma, sym, ratio);
  return hipGetLastError();
}

hipError_t launch_xs_rates(int nE, int L, int nT, const double* U, const double* E,
                           const double* g, const double* sym, double mu, const double* beta,
                           double* k, hipStream_t s) {
  if (nE < 2 || nE > XS_NE_MAX) return hipErrorInvalidValue;
  const int64_t n = (int64_t)L * L;
  const size_t lds = ((size_t)nE * (RATE_BLOCK + 3) + SER_N + 1 + 2 * RATE_TC) * sizeof(double);
  const void* fn = (const void*)xs_rate_kernel;
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  // grid.y: at most 65535 groups of RATE_TC temperatures per launch
  const int64_t tmax = 65535 * RATE_TC;
  for (int64_t t = 0; t < nT; t += tmax) {
    const int m = (int)std::min<int64_t>(nT - t, tmax);
    xs_rate_kernel<<<dim3((unsigned)((n + RATE_BLOCK - 1) / RATE_BLOCK),
                          (unsigned)((m + RATE_TC - 1) / RATE_TC)),
                     RATE_BLOCK, lds, s>>>(nE, L, m, U, E, g, sym, mu, beta + t, k + t * n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace mqct
