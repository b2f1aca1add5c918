// Chebyshev expansion of the orbital propagator exp(-i A dt) (Sec. II.C,
// Eq. exponential_integrator): the coefficients of the series in the shifted
// and scaled operator (A - c) / r, shared by the step kernels of every model
// kind (device code).
#pragma once

#include "iesh_internal.hpp"

namespace iesh {

static_assert(kMaxCheb <= 64, "one term to a lane");

// Value of a uniform lane of a double.
__device__ inline double read_lane(double v, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, lane), hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Bessel J_k(rho) of lane k <= K (0 beyond), by Miller's downward recurrence
// normalised with J_0 + 2 sum_{k>=1} J_{2k} = 1; called by a whole wave.  The
// quotients 2 k / rho of the recurrence are formed by the lanes beforehand: with
// one thread dividing in every term, a step's solves at n = 21 took 42 us, 30
// with this, the loads of a step requested together and one barrier to a sum.
// The start lies 32 above K and rho, where J is below 1e-8 of J_K, and its error the square of that.
__device__ inline double bessel_lane(int K, double rho) {
  const int lane = threadIdx.x & 63;
  if (rho < 1e-300) return lane == 0 ? 1.0 : 0.0;
  const int base = (K > (int)rho ? K : (int)rho);
  int m = base + 32;
  m += (m & 1);
  double J = 0.0, jp1 = 0.0, jk = 1e-280, norm = 0.0, quot = 0.0;
  for (int k = m; k > 0; --k) {
    const int l = (k - 1) & 63;
    if (k == m || l == 63) quot = 2.0 * (k - l + lane) / rho;  // of the 64 terms around k
    const double jm1 = read_lane(quot, l) * jk - jp1;  // J_{k-1}
    jp1 = jk;
    jk = jm1;
    if (fabs(jk) > 1e250) {
      jk *= 1e-250;
      jp1 *= 1e-250;
      norm *= 1e-250;
      J *= 1e-250;
    }
    const int km1 = k - 1;
    if (km1 == lane && km1 <= K) J = jk;
    if (km1 > 0 && (km1 & 1) == 0) norm += 2.0 * jk;
  }
  norm += jk;  // J_0
  return J * (1.0 / norm);
}

// Number of Chebyshev terms so that the tail sum_{k>K} 2|J_k(rho)| < tol,
// bounding |J_k(rho)| by (rho/2)^k / k!; lane k of the calling wave tests K = k.
__device__ inline int cheb_terms(double rho, double tol) {
  const int k = threadIdx.x & 63;
  const double h = 0.5 * rho;
  double next = h / (k + 1);  // of the product up to the lane: the bound of |J_{k+1}|
  for (int sh = 1; sh < 64; sh <<= 1) {
    const double o = __shfl_up(next, sh);
    if (k >= sh) next *= o;
  }
  const bool ok = k < kMaxCheb - 1 && k + 2 > h && 2.0 * next / (1.0 - h / (k + 2)) < tol;
  const unsigned long long mask = __ballot(ok);
  if (!mask) return -1;
  const int K = __builtin_ctzll(mask);
  return K > 0 ? K : 1;
}

// Chebyshev block of one trajectory for a propagator over dte whose
// Hermitian matrix has its spectrum in [lo, hi] (Gershgorin bounds): centre,
// 1/radius, number of terms K and the coefficients
//   c_k = e^{-i c dte} (2 - delta_k0) (-i)^k J_k(r dte).
// Counts the terms in the work counters, the context's and (cls_work, may be
// null) the class's (count_step: also one trajectory-step).  Called by a whole
// wave, a coefficient to a lane; returns K, or -1 when the series would need
// more than kMaxCheb terms.
__device__ inline int write_cheb(double* cb, double lo, double hi, double dte, int precision,
                                 Counters* cnt, bool count_step, int64_t* cls_work) {
  const double cc = 0.5 * (lo + hi);
  const double rr = fmax(0.5 * (hi - lo), 1e-300);
  const double rho = rr * dte;
  // truncation: the tail bound stays under about two units of FP64 rounding,
  // or a quarter of one unit of FP32 rounding (2^-26) for the FP32 series
  const int K = cheb_terms(rho, precision == IESH_FP64 ? 2e-16 : 0x1p-26);
  if (K < 0) return -1;
  const int k = threadIdx.x & 63;
  const double J = bessel_lane(K, rho);
  double sn, cs;
  sincos(cc * dte, &sn, &cs);
  // e^{-i c dt} * (2 - delta_k0) * (-i)^k * J_k
  if (k <= K) {
    const double a = (k ? 2.0 : 1.0) * J;
    double ar, ai;  // (-i)^k * a
    switch (k & 3) {
      case 0: ar = a; ai = 0.0; break;
      case 1: ar = 0.0; ai = -a; break;
      case 2: ar = -a; ai = 0.0; break;
      default: ar = 0.0; ai = a; break;
    }
    cb[CHEB_COEF + 2 * k] = cs * ar + sn * ai;
    cb[CHEB_COEF + 2 * k + 1] = cs * ai - sn * ar;
  }
  if (k != 0) return K;
  cb[CHEB_C] = cc;
  cb[CHEB_INVR] = 1.0 / rr;
  cb[CHEB_K] = (double)K;
  cb[CHEB_RHO] = rho;
  // work counters (integer sums: independent of the order of the adds)
  atomicAdd((unsigned long long*)&cnt->sum_cheb, (unsigned long long)K);
  if (count_step) atomicAdd((unsigned long long*)&cnt->traj_steps, 1ull);
  atomicMax((unsigned long long*)&cnt->max_cheb, (unsigned long long)K);
  if (cls_work) {  // the same two sums for the trajectory's class
    atomicAdd((unsigned long long*)&cls_work[0], (unsigned long long)K);
    if (count_step) atomicAdd((unsigned long long*)&cls_work[1], 1ull);
  }
  return K;
}

}  // namespace iesh
