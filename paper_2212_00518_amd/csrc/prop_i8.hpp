// Propagation in FP64 with the products on the 8-bit integer matrix
// instructions (the arrowhead classes).
//
// The series and its recurrence are those of the FP64 kernel (k_prop.hip),
//   b_k = c_k X + 2 At b_{k+1} - b_{k+2},
// with b in FP64.  Only the product B b_{k+1} is taken apart (Ootomo, Ozaki and
// Yokota, DGEMM on integer matrix multiplication unit, 2024): B and b, scaled
// by powers of two, become 55-bit fixed-point numbers of seven signed 8-bit
// digits; products of digits are summed exactly in 32-bit integers, one sum
// per level (the sum of the two digits' places), and the levels meet in FP64.
//
// The coefficients fall off fast and b_k with them, so a product of late terms
// needs few digits: with the bound beta on |b_{k+1}| and the scale of B, the
// levels that reach 2^-60 of a unit orbital (kBits) are kept, 8 of them for
// the last terms of the recurrence and 1 or 2 for the first.  Against the same
// recurrence in 64-bit extended precision the error is that of FP64 products
// (rms 7e-18 to 3e-17 per element and step; with 2^-55 it would be up to
// twice that).  That holds while the largest product stays below a quarter of
// a unit orbital (2^-7 for thermal trajectories at dt = 20): over 1040 emulated
// steps the two errors' mean ratio was 1.002 up to there, 1.011 at 1/4 to 1/2,
// 1.04 to 1, 1.09 to 2 and 1.2 to 4, where the 55 bits of B and b show.  Beyond
// kMostProduct (fast trajectories, long steps) a trajectory's products are left
// to the FP64 instructions (k_prop_queue).  At M = 200 a product takes 16 pairs
// of digits on average, and the integer instructions do 64 for the time of one
// FP64 product.
//
// A work-group of W waves takes NCT tiles of 16 columns (8 orbitals as
// [Re of 8 | Im of 8]); wave w has the row tiles w, w + W, ..  The digits of b
// pass through LDS (two buffers, one barrier a term) in the operand's order:
// row tile 4 kb + t, lane group g and accumulator row r are byte 4 t + r of
// lane 16 g + column.  The digits of B come from memory in that order, each
// reloaded as soon as its last use is issued.
//
// At M = 200 the matrix instructions are busy for a third of the time and the
// vector ones (digits, levels, recurrence: 235 to a tile and term) for another;
// the registers allow two waves to a SIMD, and the barrier keeps those of one
// work-group in step.
// One FP64 propagation of saturating batches, ms, FP64 instructions / this:
// 2048 trajectories of M = 200 9.3 / 6.5, 512 of M = 120 0.56 / 0.36, 256 of
// M = 320 4.9 / 2.4; of 16 trajectories of M = 100 0.098 / 0.046.
#pragma once

#include <type_traits>

#include "iesh_internal.hpp"

namespace iesh {
namespace prop_i8 {

typedef int i4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int kDigits = 7;
constexpr int kBits = 60;
constexpr double kMostProduct = 0.25;

// Exponent of the scale of numbers of modulus at most v: divided by it they stay
// below 1.9.
__device__ inline int scale_exponent(double v) {
  int ex = 0;
  return frexp(v, &ex) < 0.94 ? ex - 1 : ex;
}

// Whether the digits hold a series' products: bounds 2 B b_1 / r by the scale of
// B and sum_m m |c_m| = 2 sum_m m |J_m(rho)|, which is at most 2 rho (0.5 + 0.33
// sqrt(rho)) over the lengths a series may have (evaluated on rho = 1e-4 .. 36),
// both parts of c_m together.  r is a lower bound of the radius, rho an upper
// one of the length.
__device__ inline bool holds(double bscale, double r, double rho) {
  return 2.0 * bscale * 2.8284271247461903 * rho * (0.5 + 0.33 * sqrt(rho)) <= kMostProduct * r;
}

__host__ __device__ constexpr int kblocks(int n_pad) { return (n_pad + 63) / 64; }
__host__ __device__ constexpr size_t b_doubles(int n_pad) { return (size_t)n_pad / 16 * kblocks(n_pad) * kDigits * 128; }

// Digits of four numbers below 1.9 in modulus, by place: byte r of w[a] is
// digit a of v[r], v = sum_a w[a] 2^(-6 - 8 a) to within 2^-54.
template <int S = kDigits>
__device__ inline void split_digits(const double (&v)[4], unsigned (&w)[kDigits]) {
  constexpr double kMagic = 0x1.8p52;  // leaves the integer in the low word
  unsigned hi[4], lo[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double t = fma(v[r], 0x1p22, kMagic);
    if constexpr (S <= 3) {  // to within 2^-23, for digits 0 .. 2
      hi[r] = (unsigned)__builtin_bit_cast(unsigned long long, t) + 0x8080u;
      continue;
    }
    const double rest = fma(v[r], 0x1p22, -(t - kMagic));
    const double u = fma(rest, 4294967294.0, kMagic);
    const unsigned h = (unsigned)__builtin_bit_cast(unsigned long long, t);
    const unsigned l = (unsigned)__builtin_bit_cast(unsigned long long, u);
    // adding 0x80 to every byte but the top one turns them into digits + 0x80
    lo[r] = l + 0x80808080u;
    hi[r] = h + 0x8080u + (unsigned)((int)l >> 31) + (lo[r] < l ? 1u : 0u);
  }
  auto two = [](const unsigned (&x)[4], unsigned sel, unsigned& first, unsigned& second) {
    const unsigned p = __builtin_amdgcn_perm(x[1], x[0], sel), q = __builtin_amdgcn_perm(x[3], x[2], sel);
    first = __builtin_amdgcn_perm(q, p, 0x05040100u);
    second = __builtin_amdgcn_perm(q, p, 0x07060302u);
  };
  unsigned unused;
  two(hi, 0x06020602u, w[0], unused);
  two(hi, 0x04000501u, w[1], w[2]);
  if constexpr (S > 3) {
    two(lo, 0x06020703u, w[3], w[4]);
    two(lo, 0x04000501u, w[5], w[6]);
  }
#pragma unroll
  for (int a = 1; a < (S > 3 ? kDigits : 3); ++a) w[a] ^= 0x80808080u;
}

__device__ inline double swap8(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, 0x128, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), 0x128, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// y[ct] = B b of one row tile in units of the two scales (2^-12 left out):
// all pairs of digits with places a + b < LV.  `half`: the last k-block has at
// most 32 rows, which take half the bytes and half the time.
template <int LV, int NCT>
__device__ __forceinline__ void product(const unsigned char* Arow, const unsigned char* dig, int KB, bool half,
                                        int lane, double (&y)[NCT][4]) {
  constexpr int S = LV < kDigits ? LV : kDigits;
  i4 acc[NCT][LV];
  const i4* A = reinterpret_cast<const i4*>(Arow) + lane;  // [kb][digit][64]
  i4 av[S];
#pragma unroll
  for (int a = 0; a < S; ++a) av[a] = A[a * 64];
  const int last = half ? KB - 1 : KB;
  auto step = [&](int kb, auto first) {
    const i4* An = A + (size_t)(kb + 1 < KB ? kb + 1 : kb) * kDigits * 64;
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const i4* D = reinterpret_cast<const i4*>(dig) + (size_t)(ct * kDigits * KB + kb) * 64 + lane;
      i4 bv[S];
#pragma unroll
      for (int b = 0; b < S; ++b) bv[b] = D[(size_t)b * KB * 64];
#pragma unroll
      for (int a = 0; a < S; ++a) {
#pragma unroll
        for (int b = 0; b < S; ++b)
          if (a + b < LV) {
            const bool fresh = decltype(first)::value && (a == 0 || (b == S - 1 && a + b >= S));
            acc[ct][a + b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[a], bv[b], fresh ? i4{0, 0, 0, 0} : acc[ct][a + b], 0, 0, 0);
          }
        if (ct == NCT - 1) av[a] = An[a * 64];
      }
    }
  };
  if (last > 0) {
    step(0, std::true_type{});
    for (int kb = 1; kb < last; ++kb) step(kb, std::false_type{});
  } else {  // never from seven row tiles on; without it the compiler spills 63 registers for 38
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int l = 0; l < LV; ++l) acc[ct][l] = i4{0, 0, 0, 0};
  }
  if (half) {
    typedef long long i8x8;
    auto low = [](const i4& v) { return __builtin_bit_cast(i8x8, __builtin_shufflevector(v, v, 0, 1)); };
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const i8x8* D = reinterpret_cast<const i8x8*>(reinterpret_cast<const i4*>(dig) + (size_t)(ct * kDigits * KB + last) * 64 + lane);
      i8x8 bv[S];
#pragma unroll
      for (int b = 0; b < S; ++b) bv[b] = D[(size_t)b * KB * 128];
#pragma unroll
      for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < S; ++b)
          if (a + b < LV) acc[ct][a + b] = __builtin_amdgcn_mfma_i32_16x16x32_i8(low(av[a]), bv[b], acc[ct][a + b], 0, 0, 0);
    }
  }
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double s = (double)acc[ct][LV - 1][r];
#pragma unroll
      for (int l = LV - 2; l >= 0; --l) s = fma(s, 0x1p-8, (double)acc[ct][l][r]);
      y[ct][r] = s;
    }
}

template <int W, int NR, int NCT>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_prop_i8(ClassDev c) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n_pad = c.md.n_pad, RT = n_pad >> 4, KB = kblocks(n_pad), N = c.md.N;
  const bool half = (RT & 3) == 1 || (RT & 3) == 2;
  const int buf_bytes = NCT * kDigits * KB * 1024;  // one buffer of digits
  double* lam = reinterpret_cast<double*>(smem + 2 * buf_bytes);
  // blocks b, b + 8, ... share an XCD: a trajectory's work-groups share B in its L2
  const int b = blockIdx.x, local = b >> 3;
  const int slab = local % c.i8_slabs, t = (local / c.i8_slabs) * 8 + (b & 7);
  if (t >= c.n_live) return;
  if (t >= live_slots(c) || (c.status[t] & kFreezeMask)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, col = lane & 15;
  const bool is_re = col < 8;
  const double* cb = c.cheb + (size_t)t * kChebStride;
  const int K = (int)cb[CHEB_K];
  const double invr = cb[CHEB_INVR], cc = cb[CHEB_C], bscale = cb[CHEB_BSCALE];
  for (int i = tid; i < n_pad; i += 64 * W) lam[i] = c.lam_mid[(size_t)t * n_pad + i] - cc;

  // X: rows 16 rt + 4 g + r of the lane's column; a lane reads two complex
  // rows, the lane of the orbital's other part has the two others
  double X[NR][NCT][4], nrm[NCT];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    nrm[ct] = 0.0;
    const int o = (slab * NCT + ct) * 8 + (lane & 7);
    const double* Cg = c.C64 + ((size_t)t * N + (o < N ? o : 0)) * n_pad * 2 + (4 * g + (is_re ? 0 : 2)) * 2;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int rt = wave + W * i;
      const bool in = rt < RT && o < N;
      const d2* p = reinterpret_cast<const d2*>(Cg + (rt < RT ? rt : 0) * 32);
      const d2 v0 = p[0], v1 = p[1];
      const double r0 = swap8(is_re ? v0[1] : v0[0]), r1 = swap8(is_re ? v1[1] : v1[0]);
      X[i][ct][0] = in ? (is_re ? v0[0] : r0) : 0.0;
      X[i][ct][1] = in ? (is_re ? v1[0] : r1) : 0.0;
      X[i][ct][2] = in ? (is_re ? r0 : v0[1]) : 0.0;
      X[i][ct][3] = in ? (is_re ? r1 : v1[1]) : 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) nrm[ct] = fma(X[i][ct][r], X[i][ct][r], nrm[ct]);
    }
    nrm[ct] += __shfl_xor(nrm[ct], 16);
    nrm[ct] += __shfl_xor(nrm[ct], 32);
    nrm[ct] += swap8(nrm[ct]);  // both parts
  }
  // scale of each orbital: a power of two above its norm, or by its largest
  // element where the squares leave the range
  double* part = reinterpret_cast<double*>(smem);  // [waves][NCT][16]
  if (g == 0)
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) part[(wave * NCT + ct) * 16 + col] = nrm[ct];
  __syncthreads();
  if (bscale == 0.0) return;  // left to the FP64 instructions
  double sx[NCT], isx[NCT];
  int odd = 0;  // of this lane's columns
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    double s = 0.0;
    for (int w = 0; w < W; ++w) s += part[(w * NCT + ct) * 16 + col];
    int ex = 0;
    (void)frexp(sqrt(s), &ex);
    sx[ct] = s > 0.0 ? ldexp(1.0, ex) : 1.0;
    isx[ct] = 1.0 / sx[ct];
    if (!(s >= 0x1p-900 && s <= 0x1p900) && (slab * NCT + ct) * 8 + (lane & 7) < N) odd |= 1 << ct;
  }
  if (__any(odd != 0)) {  // the same in every wave
    __syncthreads();
    double* part = reinterpret_cast<double*>(smem);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      double m = 0.0;
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) m = fabs(X[i][ct][r]) > m || X[i][ct][r] != X[i][ct][r] ? fabs(X[i][ct][r]) : m;
      for (int sh = 8; sh < 64; sh <<= 1) {
        const double o = __shfl_xor(m, sh);
        m = o > m || o != o ? o : m;
      }
      if (g == 0) part[(wave * NCT + ct) * 16 + col] = m;
    }
    __syncthreads();
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      double m = 0.0;
      for (int w = 0; w < W; ++w) {
        const double o = part[(w * NCT + ct) * 16 + col];
        m = o > m || o != o ? o : m;
      }
      if (!(odd >> ct & 1)) continue;
      int ex = 0;
      (void)frexp(m, &ex);  // 2 n elements: the norm is below 2^5 of the largest
      sx[ct] = m > 0.0 ? ldexp(1.0, min(max(ex + 5, -1000), 1020)) : 1.0;
      isx[ct] = 1.0 / sx[ct];
      if (!(m <= 0x1.fffffffffffffp1023)) sx[ct] = m - m;  // not a number, as the result then is
    }
  }
  __syncthreads();
  for (int i = tid; i < buf_bytes / 8; i += 64 * W) reinterpret_cast<i4*>(smem)[i] = i4{0, 0, 0, 0};
  __syncthreads();

  // lane k: exponent of the scale of b_k of a unit orbital by its bound sum_{m >= k}
  // (m - k + 1) |c_m|, and the levels of the product with it
  int eb = 0, lv = 1;
  {
    double s = lane <= K ? fabs(cb[CHEB_COEF + 2 * lane]) + fabs(cb[CHEB_COEF + 2 * lane + 1]) : 0.0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass)
      for (int sh = 1; sh < 64; sh <<= 1) {
        const double o = __shfl_down(s, sh);
        s += lane + sh < 64 ? o : 0.0;
      }
    int es = 0;
    eb = scale_exponent(s);
    (void)frexp(2.0 * invr * bscale, &es);
    lv = min(max((kBits + 6 + es + eb + 7) >> 3, 1), 8);  // a ninth would lie below what B and b hold
  }

  double b1[NR][NCT][4], b2[NR][NCT][4];
  const unsigned char* Bg = reinterpret_cast<const unsigned char*>(c.Bt + (size_t)t * c.b_stride);
  // digits of b1 = b_m into a buffer
  auto put_digits = [&](int i, int m, unsigned char* dig) {
    const double sb = ldexp(1.0, -__builtin_amdgcn_readlane(eb, m));
    const int S = __builtin_amdgcn_readlane(lv, m), rt = wave + W * i;
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        const double sc = sb * isx[ct];
        double v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = b1[i][ct][r] * sc;
        unsigned w[kDigits];
        unsigned* d = reinterpret_cast<unsigned*>(dig + ((size_t)ct * kDigits * KB + (rt >> 2)) * 1024 + lane * 16 + (rt & 3) * 4);
        if (S <= 3) {
          split_digits<3>(v, w);
#pragma unroll
          for (int a = 0; a < 3; ++a) d[(size_t)a * KB * 256] = w[a];
        } else {
          split_digits(v, w);
#pragma unroll
          for (int a = 0; a < kDigits; ++a) d[(size_t)a * KB * 256] = w[a];
        }
      }
  };
  {
    const double cr = cb[CHEB_COEF + 2 * K], ci = cb[CHEB_COEF + 2 * K + 1];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double x = X[i][ct][r], xp = swap8(x);
          b1[i][ct][r] = is_re ? cr * x - ci * xp : cr * x + ci * xp;
          b2[i][ct][r] = 0.0;
        }
  }
#pragma unroll
  for (int i = 0; i < NR; ++i)
    if (wave + W * i < RT) put_digits(i, K, smem);
  __syncthreads();
  for (int k = K - 1; k >= 0; --k) {
    unsigned char* cur = smem + ((K - 1 - k) & 1) * buf_bytes;
    unsigned char* nxt = smem + ((K - k) & 1) * buf_bytes;
    const int LV = __builtin_amdgcn_readlane(lv, k + 1);
    const double unit = ldexp(bscale, __builtin_amdgcn_readlane(eb, k + 1) - 12);
    const double cr = cb[CHEB_COEF + 2 * k], ci0 = cb[CHEB_COEF + 2 * k + 1], ci = is_re ? -ci0 : ci0;
    const double scale = (k == 0 ? 1.0 : 2.0) * invr;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int rt = wave + W * i;
      if (rt >= RT) continue;
      double y[NCT][4];
      const unsigned char* Arow = Bg + (size_t)rt * KB * kDigits * 1024;
      switch (LV) {
        case 1: product<1, NCT>(Arow, cur, KB, half, lane, y); break;
        case 2: product<2, NCT>(Arow, cur, KB, half, lane, y); break;
        case 3: product<3, NCT>(Arow, cur, KB, half, lane, y); break;
        case 4: product<4, NCT>(Arow, cur, KB, half, lane, y); break;
        case 5: product<5, NCT>(Arow, cur, KB, half, lane, y); break;
        case 6: product<6, NCT>(Arow, cur, KB, half, lane, y); break;
        case 7: product<7, NCT>(Arow, cur, KB, half, lane, y); break;
        default: product<8, NCT>(Arow, cur, KB, half, lane, y); break;
      }
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        const double us = is_re ? unit * sx[ct] : -unit * sx[ct];  // the sign of the product's part
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double x = X[i][ct][r];
          const double cx = fma(cr, x, fma(ci, swap8(x), -b2[i][ct][r]));
          const double atb = fma(lam[rt * 16 + 4 * g + r], b1[i][ct][r], swap8(y[ct][r]) * us);
          const double bk = fma(scale, atb, cx);
          b2[i][ct][r] = b1[i][ct][r];
          b1[i][ct][r] = bk;
        }
      }
      if (k > 0) put_digits(i, k, nxt);
    }
    if (k > 0) __syncthreads();
  }

  double* rn = c.rown + ((size_t)t * ((N + 7) >> 3) + slab) * n_pad;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int rt = wave + W * i;
    if (rt >= RT) continue;
    double s[4] = {};
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const int o = (slab * NCT + ct) * 8 + (lane & 7);
      const double(&xv)[4] = b1[i][ct];
      const double r0 = swap8(is_re ? xv[2] : xv[0]), r1 = swap8(is_re ? xv[3] : xv[1]);
      if (o < N) {
        d2* p = reinterpret_cast<d2*>(c.C64 + ((size_t)t * N + o) * n_pad * 2 + (4 * g + (is_re ? 0 : 2)) * 2 + rt * 32);
        p[0] = d2{is_re ? xv[0] : r0, is_re ? r0 : xv[2]};
        p[1] = d2{is_re ? xv[1] : r1, is_re ? r1 : xv[3]};
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] = fma(xv[r], xv[r], s[r]);
    }
    // squared row norms over the slab's orbitals, for the no-hop bound
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      for (int sh = 1; sh < 16; sh <<= 1) s[r] += __shfl_xor(s[r], sh);
      if (col == 0) rn[rt * 16 + 4 * g + r] = s[r];
    }
  }
}

// Classes that propagate this way: from 7 row tiles on, where the products
// outweigh the rest.  512 trajectories of N = M/2, thermal, dt = 20, ms, FP64
// instructions / digits: 5 row tiles 0.195 / 0.254, 6 0.281 / 0.259 (at whose
// gain the line is not worth moving), 7 0.430 / 0.358, 8 0.580 / 0.366, 9 0.814 /
// 0.638, 10 1.10 / 0.74; 16 trajectories 0.061 / 0.045 at 5, 0.104 / 0.046 at 7.
// Narrow classes gain least: 256 trajectories of M = 143, N = 17 lose 5% of a step.
inline bool chosen(int n_pad) { return n_pad / 16 >= 7; }

// Waves of a work-group, row tiles to a wave and orbital tiles to a work-group,
// as many as the registers of two waves to a SIMD hold.  Two orbital tiles
// share the loads of B; at 9 to 12 row tiles two work-groups of four waves with
// one each, whose phases overlap, are faster all the same (10 row tiles 0.76
// against 0.87 ms, 11 0.90 against 1.07), at 13 to 16 they spill (13: 7.2
// against 6.8), at 8 they only load more (0.40 against 0.37).
struct Shape {
  int waves, nr, nct;
};
inline Shape shape(int n_pad) {
  const int rt = n_pad / 16;
  return rt <= 8 ? Shape{8, 1, 2} : rt <= 12 ? Shape{4, 3, 1} : rt <= 16 ? Shape{8, 2, 2} : Shape{8, 3, 1};
}
inline size_t lds_bytes(int n_pad) {
  return (size_t)2 * shape(n_pad).nct * kDigits * kblocks(n_pad) * 1024 + sizeof(double) * n_pad;
}

typedef void (*Kernel)(ClassDev);
inline Kernel kernel(int n_pad) {
  const Shape s = shape(n_pad);
  return s.nr == 1 ? k_prop_i8<8, 1, 2> : s.nr == 2 ? k_prop_i8<8, 2, 2> : s.waves == 4 ? k_prop_i8<4, 3, 1> : k_prop_i8<8, 3, 1>;
}

}  // namespace prop_i8
}  // namespace iesh
