// Orbital propagation of the mixed path in the interaction picture (the
// arrowhead classes; k_eig.hip, ip_setup, derives the form and its error):
//   C <- (E_post e^{iL} e^{-M} e^{-iL} E_pre)^s C,
// E diagonal phases, L = Z D Z^T of rank R <= 8, M real, antisymmetric and
// small, so e^{-M} is a Taylor polynomial of p terms by Horner's rule,
//   w <- x - M w / i,  i = p .. 1.
// Against the Chebyshev series of the same propagator (8 terms at M = 200,
// dt = 20, 18 at the scattering workload's bandwidth) p is 2 to 4, and M acts
// on real and imaginary parts alone.
//
// The products run on the f16 matrix instructions with FP32 accumulation, M
// and w each split into two f16 numbers (22 bits): hi hi + hi lo + lo hi.
// They give M w to about 2^-21 of its own size, and M w is beta = ||M|| of w,
// so the products' error is about 2^-21 beta of the orbitals (beta ~ 5e-3),
// far below the FP32 rounding of the phases.
//
// One wave owns 16 columns (8 orbitals as [Re of 8 | Im of 8]) and keeps all
// rows of x and w in registers; M streams through LDS, one or two row tiles
// at a time (double-buffered, direct-to-LDS loads), shared by the waves of
// the work-group.  The accumulator of a 16-row tile holds rows 4g .. 4g + 3
// of column l & 15 in lane l = 16 g + (l & 15); two row tiles make one
// 32-row operand if the product's inner index is read in the order (tile,
// group, row) instead of ascending, so M is stored in that order and w needs
// no exchange between lanes: the product's output, rounded, is the next
// product's operand.
#pragma once

#include "iesh_internal.hpp"

namespace iesh {
namespace prop_ip {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// k-blocks of M in flight from LDS per wave (three where four would spill)
constexpr int ring(int rt) { return rt == 12 || rt == 13 ? 3 : 4; }

// Row tiles up to which a wave fits 256 registers (two waves per SIMD); wider
// baths take one wave per SIMD with 512.
constexpr int kNarrowRT = 13;
__host__ __device__ constexpr int max_waves(int rt) { return rt <= kNarrowRT ? 8 : 4; }
constexpr int waves_per_simd(int rt) { return rt <= 2 ? 4 : rt <= 6 ? 3 : rt <= kNarrowRT ? 2 : 1; }
// row tiles per LDS buffer
__host__ __device__ constexpr int chunk_tiles(int rt) { return (rt + 1) / 2 <= 7 ? 2 : 1; }

// LDS of the two buffers of M; the row norms reuse it (64 rows of 17 floats a wave)
__host__ __device__ constexpr int buffer_bytes(int rt) {
  const int buf = 2 * chunk_tiles(rt) * ((rt + 1) / 2) * 2048, rows = max_waves(rt) * 64 * 17 * 4;
  return buf > rows ? buf : rows;
}

// Value of lane l ^ 8 (a rotation by 8 within 16 lanes).
__device__ inline float swap8(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xf, 0xf, false));
}

// Four values in f16 pairs: hi rounds toward zero, lo takes what is left.
__device__ inline void split4(const float* v, unsigned* hi, unsigned* lo) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto h = __builtin_amdgcn_cvt_pkrtz(v[2 * i], v[2 * i + 1]);
    const auto l = __builtin_amdgcn_cvt_pkrtz(v[2 * i] - (float)h[0], v[2 * i + 1] - (float)h[1]);
    hi[i] = __builtin_bit_cast(unsigned, h);
    lo[i] = __builtin_bit_cast(unsigned, l);
  }
}

// The R columns of Z on the four rows of a lane in one row tile: fn(f, z).
template <int R, typename F>
__device__ inline void each_column(const float* zp, int n_pad, int row, F fn) {
#pragma unroll
  for (int f = 0; f < R; ++f) fn(f, *reinterpret_cast<const f4*>(zp + f * n_pad + row));
}

// Ends a row tile's part of a loop over all rows: keeps the loads of one tile
// in flight instead of all, and the values of one loop from being kept in
// registers for the next.
__device__ inline void tile_end() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// T += (F2 + i sigma D) P over the R columns; sig: sigma on the imaginary
// lanes, -sigma on the real ones (their partner holds the other part).
template <int R>
__device__ inline void apply_small(const float (&P)[R], float (&T)[R], const float* ips, float sig) {
  float S[R];
#pragma unroll
  for (int q = 0; q < R; ++q) S[q] = sig * swap8(P[q]);
#pragma unroll
  for (int f = 0; f < R; ++f) {
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < R; ++q) s = fmaf(ips[IP_D + f * R + q], S[q], fmaf(ips[IP_F2 + f * R + q], P[q], s));
    T[f] += s;
  }
}

// What a wave needs to know of its work-group.
struct Group {
  const float* ips;          // this trajectory's plan
  const float* pl;           // LDS: planes of ipv
  unsigned char* buf;        // LDS: two buffers of M
  const unsigned char* Mg;   // M in memory
  int sub, p, nw, wave, lane;
  float unscale;
};

// One buffer of M into LDS: 1 KB pieces dealt to the waves.
template <int RT>
__device__ inline void load_chunk(const Group& gr, int cc, int parity) {
  constexpr int G = chunk_tiles(RT), kTileBytes = (RT + 1) / 2 * 2048;
  const int tiles_here = (cc + 1) * G <= RT ? G : RT - cc * G;
  const unsigned char* src = gr.Mg + (size_t)cc * G * kTileBytes;
  unsigned char* dst = gr.buf + (parity & 1) * G * kTileBytes;
  for (int i = gr.wave; i < tiles_here * (kTileBytes >> 10); i += gr.nw)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + i * 1024 + gr.lane * 16),
                                     (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, 0, 0);
}

// Waits for this wave's loads into LDS, then for every wave's.
__device__ inline void arrive() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// One sub-interval: u = E_pre x (kept in x); with w0 = u + Z T1 (e^{-iL} u),
// y = (e^{-M} - 1) w0 and T2 from e^{iL} (w0 + y), x <- E_post (u + d),
// d = y + Z (T1 + T2).  The small parts stay out of u until the last
// rounding: added one by one to numbers of 24 bits, whatever is below half
// a unit would be lost in every step the same way (at M = 44 with two
// sub-steps the orbitals were 1.6e-6 off after 99 steps that way, 0.7e-6
// with the Chebyshev series).
template <int RT, int R>
__device__ inline void sub_intervals(const Group& gr, float (&x)[RT][4]) {
  constexpr int n_pad = 16 * RT;
  constexpr int KB = (RT + 1) / 2;       // k-blocks of 32 columns
  constexpr int G = chunk_tiles(RT);     // row tiles per buffer
  constexpr int NC = (RT + G - 1) / G;   // buffers per pass over M
  constexpr int kTileBytes = KB * 2048;  // one row tile of M
  constexpr int kRing = ring(RT);
  const float* ips = gr.ips;
  const float* pl = gr.pl;
  const float* zp = pl + IPV_Z * n_pad;
  unsigned char* buf = gr.buf;
  const int lane = gr.lane, g = lane >> 4, sub = gr.sub, p = gr.p;
  const float sg = (lane & 15) < 8 ? -1.0f : 1.0f, unscale = gr.unscale;
  int ch = 0;  // buffers of M consumed (its parity names the buffer in use)
  for (int it = 0; it < sub; ++it) {
    float T[R] = {}, P[R] = {};
    float m = 0.0f;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int row = rt * 16 + 4 * g;
      const f4 c0 = *reinterpret_cast<const f4*>(pl + IPV_PRE * n_pad + row);
      const f4 s0 = *reinterpret_cast<const f4*>(pl + (IPV_PRE + 1) * n_pad + row);
      const f4 cl = *reinterpret_cast<const f4*>(pl + (IPV_PRE + 2) * n_pad + row);
      const f4 sl = *reinterpret_cast<const f4*>(pl + (IPV_PRE + 3) * n_pad + row);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float xr = x[rt][r], xp = sg * swap8(xr);
        x[rt][r] = fmaf(s0[r], xp, fmaf(c0[r], xr, fmaf(sl[r], xp, cl[r] * xr)));
        m = fmaxf(m, fabsf(x[rt][r]));
      }
      each_column<R>(zp, n_pad, row, [&](int f, f4 z) {
#pragma unroll
        for (int r = 0; r < 4; ++r) P[f] = fmaf(z[r], x[rt][r], P[f]);
      });
      tile_end();
    }
    // power-of-two scale of each column that keeps u and w within f16's range
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    int ex = 0;
    if (m > 0x1p-100f && m < 0x1p100f) (void)frexpf(m, &ex);
    const float sx = ldexpf(1.0f, 10 - ex);
    auto sum_groups = [&] {
#pragma unroll
      for (int f = 0; f < R; ++f) {
        P[f] += __shfl_xor(P[f], 16);
        P[f] += __shfl_xor(P[f], 32);
      }
    };
    sum_groups();
    // the two lanes of an orbital may scale differently: T in true units first
    apply_small<R>(P, T, ips, -sg);
#pragma unroll
    for (int f = 0; f < R; ++f) T[f] *= sx;
    u4 wh[KB], wl[KB];
    auto put = [](u4* h, u4* l, int rt, const float* v) {
      unsigned hi[2], lo[2];
      split4(v, hi, lo);
      // computed here: left alone, the compiler sinks the splits of all row
      // tiles to the end of the pass and holds their inputs until then
      asm volatile("" : "+v"(hi[0]), "+v"(hi[1]), "+v"(lo[0]), "+v"(lo[1]));
      h[rt >> 1][2 * (rt & 1)] = hi[0];
      h[rt >> 1][2 * (rt & 1) + 1] = hi[1];
      l[rt >> 1][2 * (rt & 1)] = lo[0];
      l[rt >> 1][2 * (rt & 1) + 1] = lo[1];
    };
    auto add_low_rank = [&](int rt, float* v) {  // v += Z T
      each_column<R>(zp, n_pad, rt * 16 + 4 * g, [&](int f, f4 z) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(z[r], T[f], v[r]);
      });
    };
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = x[rt][r] *= sx;
      add_low_rank(rt, v);
      put(wh, wl, rt, v);
      tile_end();
    }
    if constexpr (RT & 1) {
      wh[KB - 1][2] = wh[KB - 1][3] = 0u;
      wl[KB - 1][2] = wl[KB - 1][3] = 0u;
    }
    // pass over M: out(rt, y) takes the product M w of a row tile
    auto pass = [&](bool last_pass, auto out) {
#pragma unroll
      for (int cc = 0; cc < NC; ++cc) {
        // the next buffer while this one is in use (the last one of a pass
        // fetches the first of the next)
        const unsigned char* cur = buf + (ch & 1) * G * kTileBytes;
        if (!(cc == NC - 1 && last_pass)) {
          const int nx = cc == NC - 1 ? 0 : cc + 1;
          load_chunk<RT>(gr, nx, ch + 1);
        }
        // M's operands kRing k-blocks ahead in registers
        const h8* A = reinterpret_cast<const h8*>(cur) + lane;
        constexpr int kSteps = G * KB;
        const int steps = (cc + 1) * G <= RT ? kSteps : (RT - cc * G) * KB;
        h8 ah[kRing], al[kRing];
#pragma unroll
        for (int q = 0; q < kRing - 1; ++q)
          if (q < steps) {
            ah[q] = A[q * 128];
            al[q] = A[q * 128 + 64];
          }
        f4 y0, y1;
#pragma unroll
        for (int q = 0; q < kSteps; ++q) {
          if (q < steps) {
            const int kb = q % KB, rt = cc * G + q / KB, nq = q + kRing - 1;
            if (nq < steps) {
              ah[nq % kRing] = A[nq * 128];
              al[nq % kRing] = A[nq * 128 + 64];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kb == 0) y0 = y1 = f4{0.0f, 0.0f, 0.0f, 0.0f};
            const h8 bh = __builtin_bit_cast(h8, wh[kb]), bl = __builtin_bit_cast(h8, wl[kb]);
            y0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[q % kRing], bh, y0, 0, 0, 0);
            y1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[q % kRing], bl, y1, 0, 0, 0);
            y1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[q % kRing], bh, y1, 0, 0, 0);
            if (kb == KB - 1) out(rt, y0 + y1);
          }
        }
        ++ch;
        arrive();
      }
    };
    for (int i = p; i > 1; --i) {
      const float ci = -unscale / (float)i;
      u4 nh[KB], nl[KB];
      pass(false, [&](int rt, f4 y) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(ci, y[r], x[rt][r]);
        add_low_rank(rt, v);
        put(nh, nl, rt, v);
      });
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        wh[kb] = nh[kb];
        wl[kb] = nl[kb];
      }
      if constexpr (RT & 1) {
        wh[KB - 1][2] = wh[KB - 1][3] = 0u;
        wl[KB - 1][2] = wl[KB - 1][3] = 0u;
      }
    }
    float y[RT][4];
#pragma unroll
    for (int f = 0; f < R; ++f) P[f] = 0.0f;
    pass(it == sub - 1, [&](int rt, f4 yv) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        y[rt][r] = -unscale * yv[r];
        asm volatile("" : "+v"(y[rt][r]));
      }
    });
    const float ux = ldexpf(1.0f, ex - 10);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = x[rt][r] + y[rt][r];
      add_low_rank(rt, v);
      each_column<R>(zp, n_pad, rt * 16 + 4 * g, [&](int f, f4 z) {
#pragma unroll
        for (int r = 0; r < 4; ++r) P[f] = fmaf(z[r], v[r], P[f]);
      });
      tile_end();
    }
    sum_groups();
#pragma unroll
    for (int f = 0; f < R; ++f) {
      P[f] *= ux;
      T[f] *= ux;
    }
    apply_small<R>(P, T, ips, sg);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int row = rt * 16 + 4 * g;
      float dv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) dv[r] = y[rt][r] * ux;
      add_low_rank(rt, dv);
      const f4 c0 = *reinterpret_cast<const f4*>(pl + IPV_POST * n_pad + row);
      const f4 s0 = *reinterpret_cast<const f4*>(pl + (IPV_POST + 1) * n_pad + row);
      const f4 cl = *reinterpret_cast<const f4*>(pl + (IPV_POST + 2) * n_pad + row);
      const f4 sl = *reinterpret_cast<const f4*>(pl + (IPV_POST + 3) * n_pad + row);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float xr = x[rt][r] * ux, xp = sg * swap8(xr), dp = sg * swap8(dv[r]);
        const float low = fmaf(s0[r], dp, fmaf(c0[r], dv[r], fmaf(sl[r], xp, cl[r] * xr)));
        x[rt][r] = fmaf(s0[r], xp, fmaf(c0[r], xr, low));
      }
      tile_end();
    }
  }
}

template <int RT>
__global__ __launch_bounds__(64 * max_waves(RT))
    __attribute__((amdgpu_waves_per_eu(waves_per_simd(RT), waves_per_simd(RT)))) void k_prop_ip(ClassDev c, int groups) {
  constexpr int n_pad = 16 * RT;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* buf = smem;                                              // [2][row tiles][k-blocks][2][64][16 B]
  float* pl = reinterpret_cast<float*>(smem + buffer_bytes(RT));          // planes of ipv

  // blocks b, b + 8, ... share an XCD: the work-groups of a trajectory share M in its L2
  const int b = blockIdx.x, local = b >> 3;
  const int grp = local % groups, t = (local / groups) * 8 + (b & 7);
  if (t >= live_slots(c) || (c.status[t] & kFreezeMask)) return;
  const float* ips = c.ips + (size_t)t * kIpStride;
  const int sub = (int)ips[IP_SUB];
  if (sub == 0) return;  // Chebyshev series
  const int p = (int)ips[IP_TERMS], R = (int)ips[IP_RANK];
  const float unscale = ips[IP_UNSCALE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int g = lane >> 4, col = lane & 15;
  const bool is_re = col < 8;
  const int N = c.md.N, tiles = (N + 7) >> 3;
  // the tiles of a trajectory over its work-groups, balanced
  const int base = tiles / groups, rem = tiles % groups;
  const int tile = grp * base + (grp < rem ? grp : rem) + wave;
  const bool active = wave < base + (grp < rem ? 1 : 0);
  const int o = tile * 8 + (lane & 7);

  const unsigned char* Mg = reinterpret_cast<const unsigned char*>(c.Bt32 + (size_t)t * c.b_stride);
  Group gr{ips, pl, buf, Mg, sub, p, nw, wave, lane, unscale};
  load_chunk<RT>(gr, 0, 0);

  const float* ipv = c.ipv + (size_t)t * kIpPlanes * n_pad;
  for (int i = tid; i < (IPV_Z + R) * n_pad; i += blockDim.x) pl[i] = ipv[i];

  // x: rows 16 rt + 4 g + r of the lane's column.  A lane reads two complex
  // rows; the lane of the orbital's other part has the two others.
  float x[RT][4];
  float* Cg = c.C32 + ((size_t)t * N + (active && o < N ? o : 0)) * n_pad * 2;
  const bool mine = active && o < N;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const f4 v = *reinterpret_cast<const f4*>(Cg + (rt * 16 + 4 * g + (is_re ? 0 : 2)) * 2);
    const float r0 = swap8(is_re ? v[1] : v[0]), r1 = swap8(is_re ? v[3] : v[2]);
    x[rt][0] = is_re ? v[0] : r0;
    x[rt][1] = is_re ? v[2] : r1;
    x[rt][2] = is_re ? r0 : v[1];
    x[rt][3] = is_re ? r1 : v[3];
    if (!mine)  // idle columns read orbital 0
#pragma unroll
      for (int r = 0; r < 4; ++r) x[rt][r] = 0.0f;
  }
  arrive();

  if (R == 2)
    sub_intervals<RT, 2>(gr, x);
  else if (R == 4)
    sub_intervals<RT, 4>(gr, x);
  else
    sub_intervals<RT, 8>(gr, x);

#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const float r0 = swap8(is_re ? x[rt][2] : x[rt][0]), r1 = swap8(is_re ? x[rt][3] : x[rt][1]);
    f4 v;
    v[0] = is_re ? x[rt][0] : r0;
    v[1] = is_re ? r0 : x[rt][2];
    v[2] = is_re ? x[rt][1] : r1;
    v[3] = is_re ? r1 : x[rt][3];
    if (mine) *reinterpret_cast<f4*>(Cg + (rt * 16 + 4 * g + (is_re ? 0 : 2)) * 2) = v;
  }
  // squared row norms over the tile's orbitals (of the stored values, summed
  // in FP64), for the no-hop bound: 64 rows at a time through the wave's part
  // of the LDS (every wave has left the buffers of M)
  if (active) {
    float* wl_ = reinterpret_cast<float*>(buf) + wave * 64 * 17;
    double* rn = c.rown + ((size_t)t * tiles + tile) * n_pad;
#pragma unroll
    for (int r0 = 0; r0 < RT; r0 += 4) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (r0 + q < RT)
#pragma unroll
          for (int r = 0; r < 4; ++r) wl_[(q * 16 + 4 * g + r) * 17 + col] = x[r0 + q][r];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      double acc = 0.0;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const double v = (double)wl_[lane * 17 + q];
        acc = fma(v, v, acc);
      }
      if (r0 * 16 + lane < n_pad) rn[r0 * 16 + lane] = acc;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
}

template <int RT>
size_t lds_bytes() {
  return buffer_bytes(RT) + (size_t)kIpPlanes * 16 * RT * 4;
}

// The kernel for rt row tiles: reserves its LDS, or launches it.
struct Launch {
  const ClassDev* c;
  dim3 grid;
  int threads, groups;
  hipStream_t stream;
  bool prepare;
};

template <int RT = 1>
hipError_t dispatch(int rt, const Launch& l) {
  if constexpr (16 * RT > kMaxStates) {
    return hipErrorInvalidValue;
  } else {
    if (rt != RT) return dispatch<RT + 1>(rt, l);
    if (l.prepare)
      return hipFuncSetAttribute((const void*)k_prop_ip<RT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)lds_bytes<RT>());
    hipLaunchKernelGGL((k_prop_ip<RT>), l.grid, dim3(l.threads), lds_bytes<RT>(), l.stream, *l.c, l.groups);
    return hipGetLastError();
  }
}

}  // namespace prop_ip
}  // namespace iesh
