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
// rows of x and w in registers; M passes through LDS, one or two row tiles
// at a time (a ring of buffers, direct-to-LDS loads), shared by the waves of
// the work-group.  The accumulator of a 16-row tile holds rows 4g .. 4g + 3
// of column l & 15 in lane l = 16 g + (l & 15); two row tiles make one
// 32-row operand if the product's inner index is read in the order (tile,
// group, row) instead of ascending, so M is stored in that order and w needs
// no exchange between lanes: the product's output, rounded, is the next
// product's operand.
//
// Bound by latency: at M = 200 a compute unit holds one work-group of seven
// waves, which loads, multiplies and stores in turn (matrix instructions busy 27%
// of the cycles, vector ones 35%, the LDS, from which every wave reads all of M
// in each product, 31%; waves wait for 37% of their time), at M = 256 and 320 four
// waves (19, 22 to 24 and 21%).  Per step of a batch, ms, Chebyshev series / this with M
// in two buffers and its loads waited for before every LDS read / now:
//   4096 trajectories, M = 200, N = 100                   5.53 / 1.26 / 1.08
//   1536, two leads, M = 256, N = 128                     3.98 / 1.51 / 1.29
//   768, M = 200, N = 100                                 1.04 / .26 / .24
//   4 x 512 at M = 40 to 320, scattering bath   7.89 / 1.97 / 1.93
#pragma once

#include <algorithm>

#include "iesh_internal.hpp"

namespace iesh {
namespace prop_ip {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// Waves per SIMD by row tiles (what their registers allow; x, w and the next
// w take 12 per row tile) and most waves to a work-group.
__host__ __device__ constexpr int waves_per_simd(int rt) { return rt <= 2 ? 4 : rt <= 6 ? 3 : rt <= 13 ? 2 : 1; }
__host__ __device__ constexpr int max_waves(int rt) { return rt <= 13 ? 8 : 4; }
// k-blocks of M in flight from LDS per wave (three where four would spill)
constexpr int ring(int rt) { return rt == 12 || rt == 13 ? 3 : 4; }

// M in LDS: chunks of one or two row tiles in a ring of buffers.  A launch
// whose ring holds all of M keeps it for every pass; the others stream it with
// the other buffers' chunks in flight: the first pass reads M from memory,
// whose latency is several chunks long.
__host__ __device__ constexpr int chunk_tiles(int rt) { return (rt + 1) / 2 <= 7 ? 2 : 1; }
__host__ __device__ constexpr int chunk_bytes(int rt) { return chunk_tiles(rt) * ((rt + 1) / 2) * 2048; }
__host__ __device__ constexpr int chunks(int rt) { return (rt + chunk_tiles(rt) - 1) / chunk_tiles(rt); }
constexpr int kLdsBytes = 160 * 1024;
__host__ __device__ constexpr int plane_bytes(int rt) { return kIpPlanes * 16 * rt * 4; }

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
  const unsigned char* buf;  // LDS: the buffers of M
  unsigned buf_lds;          // and their byte address there
  const unsigned char* Mg;   // M in memory
  int sub, p, nw, wave, lane;
  int loads;                 // of each wave per chunk of M
  int nbuf;                  // buffers of M (all its chunks: loaded once)
  float unscale;
};

// 1 KB from memory (src + 16 lane) to LDS at byte `lds`, asynchronously.  In
// assembly: the compiler waits for loads into LDS that it knows of before any
// LDS read it cannot tell apart, here the phases and Z, which cost the whole
// latency of M (10,000 cycles a work-group).  It has no register result;
// arrive() waits for it.
__device__ inline void load_to_lds(const unsigned char* src, unsigned voff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds), "v"(voff), "s"(src) : "memory", "m0");
}

// One chunk of M into a buffer: 1 KB pieces dealt to the waves, the same
// number of loads to each (the last piece again where there is none left).
template <int RT>
__device__ inline void load_chunk(const Group& gr, int cc, int slot) {
  constexpr int G = chunk_tiles(RT), kTilePieces = (RT + 1) / 2 * 2;
  const int last = ((cc + 1) * G <= RT ? G : RT - cc * G) * kTilePieces - 1;
  const unsigned char* src = gr.Mg + (size_t)cc * chunk_bytes(RT);
  const unsigned dst = gr.buf_lds + slot * chunk_bytes(RT);
  for (int k = 0; k < gr.loads; ++k) {
    const int i = min(gr.wave + k * gr.nw, last);
    load_to_lds(src + i * 1024, gr.lane * 16, dst + i * 1024);
  }
}

// Waits until at most n of this wave's loads are outstanding (or fewer), then
// for every wave.
__device__ inline void arrive(int n) {
#define IESH_IP_WAIT(k) asm volatile("s_waitcnt vmcnt(" #k ")" ::: "memory")
  if (n < 8) {
    if (n < 3)
      IESH_IP_WAIT(0);
    else if (n < 6)
      IESH_IP_WAIT(3);
    else
      IESH_IP_WAIT(6);
  } else if (n < 16) {
    if (n < 12)
      IESH_IP_WAIT(8);
    else
      IESH_IP_WAIT(12);
  } else if (n < 24) {
    if (n < 20)
      IESH_IP_WAIT(16);
    else
      IESH_IP_WAIT(20);
  } else {
    IESH_IP_WAIT(24);
  }
#undef IESH_IP_WAIT
  // no fence: it would wait for the loads still in flight.  What the barrier
  // orders, the LDS reads of the chunk that is given up and the loads into
  // it, is complete or not yet issued.
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// One sub-interval: u = E_pre x (kept in x); with w0 = u + Z T1 (e^{-iL} u),
// y = (e^{-M} - 1) w0 and T2 from e^{iL} (w0 + y), x <- E_post (u + d),
// d = y + Z (T1 + T2).  The small parts stay out of u until the last
// rounding: added one by one to numbers of 24 bits, whatever is below half
// a unit would be lost in every step the same way.  For the same reason the
// cosine's term of a phase is added last: the phase of a state near the Fermi
// level is small, its cosine's term nearly the whole number, and rounded
// before the sine's it is off by the same amount step after step (M = 106,
// Gauss-Legendre bath, two sub-steps, 99 steps: orbitals 8.8e-7 off,
// 6.2e-7 with the Chebyshev series, 4.1e-7 this way).
template <int RT, int R>
__device__ inline void sub_intervals(const Group& gr, float (&x)[RT][4]) {
  constexpr int n_pad = 16 * RT;
  constexpr int KB = (RT + 1) / 2;       // k-blocks of 32 columns
  constexpr int G = chunk_tiles(RT);     // row tiles per buffer
  constexpr int NC = chunks(RT);         // chunks per pass over M
  constexpr int kTileBytes = KB * 2048;  // one row tile of M
  constexpr int kRing = ring(RT);
  const float* ips = gr.ips;
  const float* pl = gr.pl;
  const float* zp = pl + IPV_Z * n_pad;
  const unsigned char* buf = gr.buf;
  const int lane = gr.lane, g = lane >> 4, sub = gr.sub, p = gr.p;
  const float sg = (lane & 15) < 8 ? -1.0f : 1.0f, unscale = gr.unscale;
  const int nbuf = gr.nbuf;
  const bool resident = nbuf == NC;
  const int ahead = (nbuf - 2) * gr.loads;  // loads outstanding when a chunk has arrived
  int slot = 0;                             // buffer in use
  int left = sub * p * NC - (nbuf - 1);     // chunks still to be requested
  for (int it = 0; it < sub; ++it) {
    float T[R] = {}, P[R] = {};
    float m = 0.0f;
    auto phase = [&](int plane, int rt, f4 (&c)[4]) {  // cos, sin and their low parts
#pragma unroll
    for (int q = 0; q < 4; ++q) c[q] = *reinterpret_cast<const f4*>(pl + (plane + q) * n_pad + rt * 16 + 4 * g);
    };
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      f4 c[4];
      phase(IPV_PRE, rt, c);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float xr = x[rt][r], xp = sg * swap8(xr);
        x[rt][r] = fmaf(c[0][r], xr, fmaf(c[1][r], xp, fmaf(c[3][r], xp, c[2][r] * xr)));
        m = fmaxf(m, fabsf(x[rt][r]));
      }
      each_column<R>(zp, n_pad, rt * 16 + 4 * g, [&](int f, f4 z) {
#pragma unroll
        for (int r = 0; r < 4; ++r) P[f] = fmaf(z[r], x[rt][r], P[f]);
      });
      if (rt & 1) tile_end();
    }
    auto sum_groups = [&] {
#pragma unroll
      for (int f = 0; f < R; ++f) {
        P[f] += __shfl_xor(P[f], 16);
        P[f] += __shfl_xor(P[f], 32);
      }
    };
    sum_groups();
    // power-of-two scale of each column that keeps u and w within f16's range;
    // T in true units first, the two lanes of an orbital may scale differently
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    int ex = 0;
    if (m > 0.0f && m <= 3.4028234e38f) (void)frexpf(m, &ex);
    ex = max(ex, -115);  // FP32 holds the scale and its inverse
    const float sx = ldexpf(1.0f, 10 - ex);
    apply_small<R>(P, T, ips, -sg);
#pragma unroll
    for (int f = 0; f < R; ++f) T[f] *= sx;
    u4 wh[KB], wl[KB];
    auto put = [](u4 (&h)[KB], u4 (&l)[KB], int rt, const float* v) {
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
    auto pad = [](u4 (&h)[KB]) {  // rows past an odd last tile
      if constexpr (RT & 1)
        h[KB - 1][2] = h[KB - 1][3] = 0u;
    };
    auto add_low_rank = [&](int rt, float (&v)[4]) {  // v += Z T
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
      if (rt & 1) tile_end();
    }
    pad(wh);
    pad(wl);
    if (resident && it == 0) arrive(0);
    // pass over M: out(rt, y) takes the products M w of a row tile
    auto pass = [&](auto out) {
#pragma unroll
      for (int cc = 0; cc < NC; ++cc) {
        const unsigned char* cur;
        if (resident) {
          cur = buf + cc * chunk_bytes(RT);
        } else {
          // this chunk has arrived once those requested after it may be
          // outstanding; then the buffer before it is free for the next
          arrive(left > 0 ? ahead : 0);
          if (left > 0)
            load_chunk<RT>(gr, cc + nbuf - 1 < NC ? cc + nbuf - 1 : cc + nbuf - 1 - NC, slot == 0 ? nbuf - 1 : slot - 1);
          --left;
          cur = buf + slot * chunk_bytes(RT);
          slot = slot == nbuf - 1 ? 0 : slot + 1;
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
            if (kb == KB - 1) {
              float y[4];
#pragma unroll
              for (int r = 0; r < 4; ++r) y[r] = y0[r] + y1[r];
              out(rt, y);
            }
          }
        }
      }
    };
    for (int i = p; i > 1; --i) {
      const float ci = -unscale / (float)i;
      u4 nh[KB], nl[KB];
      pass([&](int rt, const float (&y)[4]) {
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
      pad(wh);
      pad(wl);
    }
    float y[RT][4];
    pass([&](int rt, const float (&yv)[4]) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        y[rt][r] = -unscale * yv[r];
        asm volatile("" : "+v"(y[rt][r]));
      }
    });
#pragma unroll
    for (int f = 0; f < R; ++f) P[f] = 0.0f;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = x[rt][r] + y[rt][r];
      f4 zr[R];
      each_column<R>(zp, n_pad, rt * 16 + 4 * g, [&](int f, f4 z) {
        zr[f] = z;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(z[r], T[f], v[r]);
      });
#pragma unroll
      for (int f = 0; f < R; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) P[f] = fmaf(zr[f][r], v[r], P[f]);
      if (rt & 1) tile_end();
    }
    sum_groups();
    const float ux = ldexpf(1.0f, ex - 10);
#pragma unroll
    for (int f = 0; f < R; ++f) {
      P[f] *= ux;
      T[f] *= ux;
    }
    apply_small<R>(P, T, ips, sg);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float dv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) dv[r] = y[rt][r] * ux;
      add_low_rank(rt, dv);
      f4 c[4];
      phase(IPV_POST, rt, c);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float xr = x[rt][r] * ux, xp = sg * swap8(xr), dr = dv[r], dp = sg * swap8(dr);
        const float low = fmaf(c[1][r], dp, fmaf(c[0][r], dr, fmaf(c[3][r], xp, c[2][r] * xr)));
        x[rt][r] = fmaf(c[0][r], xr, fmaf(c[1][r], xp, low));
      }
      if (rt & 1) tile_end();
    }
  }
}

template <int RT>
__global__ __launch_bounds__(64 * max_waves(RT))
    __attribute__((amdgpu_waves_per_eu(waves_per_simd(RT), waves_per_simd(RT)))) void k_prop_ip(ClassDev c, int groups, int nbuf, int buf_bytes) {
  constexpr int n_pad = 16 * RT;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* buf = smem;                                // [buffers][row tiles][k-blocks][2][64][16 B]
  float* pl = reinterpret_cast<float*>(smem + buf_bytes);   // planes of ipv

  // blocks b, b + 8, ... share an XCD: the work-groups of a trajectory share M in its L2
  const int b = blockIdx.x, local = b >> 3;
  const int grp = local % groups, t = (local / groups) * 8 + (b & 7);
  if (t >= c.n_live) return;
  // everything is requested before the first answer is looked at
  const int live = live_slots(c), status = c.status[t];
  const float* ips = c.ips + (size_t)t * kIpStride;
  const f4 plan = *reinterpret_cast<const f4*>(ips);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int g = lane >> 4, col = lane & 15;
  const bool is_re = col < 8;
  const int N = c.md.N, tiles = (N + 7) >> 3;
  // the tiles of a trajectory over its work-groups, balanced, one to a wave
  const int base = tiles / groups, rem = tiles % groups;
  const int first = grp * base + (grp < rem ? grp : rem), end = first + base + (grp < rem ? 1 : 0);
  const int tile = first + wave;

  const unsigned char* Mg = reinterpret_cast<const unsigned char*>(c.Bt32 + (size_t)t * c.b_stride);
  const float* ipv = c.ipv + (size_t)t * kIpPlanes * n_pad;
  for (int i = wave; i * 1024 < plane_bytes(RT); i += nw)
    if (i * 1024 + lane * 16 < plane_bytes(RT))
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(reinterpret_cast<const unsigned char*>(ipv) + i * 1024 + lane * 16),
          (__attribute__((address_space(3))) void*)(reinterpret_cast<unsigned char*>(pl) + i * 1024), 16, 0, 0);

  // x: rows 16 rt + 4 g + r of the lane's column.  A lane reads two complex
  // rows; the lane of the orbital's other part has the two others.
  float x[RT][4];
  f4 cv[RT];
  const int o = tile * 8 + (lane & 7);
  const bool mine = tile < end && o < N;  // idle columns read orbital 0
  float* Cg = c.C32 + ((size_t)t * N + (mine ? o : 0)) * n_pad * 2 + (4 * g + (is_re ? 0 : 2)) * 2;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) cv[rt] = *reinterpret_cast<const f4*>(Cg + rt * 32);
  __builtin_amdgcn_sched_barrier(0);
  const int sub = (int)plan[IP_SUB], p = (int)plan[IP_TERMS], R = (int)plan[IP_RANK];
  const float unscale = plan[IP_UNSCALE];
  if (t >= live || (status & kFreezeMask) || sub == 0) {  // sub == 0: Chebyshev series
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // no load into LDS outlives the work-group
    return;
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const f4 v = cv[rt];
    const float r0 = swap8(is_re ? v[1] : v[0]), r1 = swap8(is_re ? v[3] : v[2]);
    x[rt][0] = mine ? (is_re ? v[0] : r0) : 0.0f;
    x[rt][1] = mine ? (is_re ? v[2] : r1) : 0.0f;
    x[rt][2] = mine ? (is_re ? r0 : v[1]) : 0.0f;
    x[rt][3] = mine ? (is_re ? r1 : v[3]) : 0.0f;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();  // planes
  // M is requested once the orbitals are there: requested first, it would
  // hold them up, and the phases below cover its latency
  const int loads = (chunk_bytes(RT) / 1024 + nw - 1) / nw;
  const unsigned buf_lds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)buf;
  const Group gr{ips, pl, buf, buf_lds, Mg, sub, p, nw, wave, lane, loads, nbuf, unscale};
  for (int q = 0; q < (nbuf == chunks(RT) ? nbuf : nbuf - 1); ++q) load_chunk<RT>(gr, q, q);

  if (R == 2)
    sub_intervals<RT, 2>(gr, x);
  else if (R == 4)
    sub_intervals<RT, 4>(gr, x);
  else
    sub_intervals<RT, 8>(gr, x);

#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const float(&xv)[4] = x[rt];
      const float r0 = swap8(is_re ? xv[2] : xv[0]), r1 = swap8(is_re ? xv[3] : xv[1]);
      f4 v;
      v[0] = is_re ? xv[0] : r0;
      v[1] = is_re ? r0 : xv[2];
      v[2] = is_re ? xv[1] : r1;
      v[3] = is_re ? r1 : xv[3];
      if (mine) *reinterpret_cast<f4*>(Cg + rt * 32) = v;
    }
  // squared row norms over the tile's orbitals (of the stored values, summed
  // in FP64), for the no-hop bound: 64 rows at a time through the wave's part
  // of the LDS, once every wave has left the buffers of M
  __syncthreads();
  float* sq = reinterpret_cast<float*>(buf) + wave * 64 * 17;
  if (tile < end) {
    double* rn = c.rown + ((size_t)t * tiles + tile) * n_pad;
#pragma unroll
    for (int r0 = 0; r0 < RT; r0 += 4) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (r0 + q < RT)
#pragma unroll
        for (int r = 0; r < 4; ++r) sq[(q * 16 + 4 * g + r) * 17 + col] = x[r0 + q][r];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      double acc = 0.0;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const double v = (double)sq[lane * 17 + q];
        acc = fma(v, v, acc);
      }
      if (r0 * 16 + lane < n_pad) rn[r0 * 16 + lane] = acc;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// The kernel for rt row tiles: reserves its LDS, or launches it.
struct Launch {
  const ClassDev* c;
  dim3 grid;
  int waves, groups;
  hipStream_t stream;
  bool prepare;
};

template <int RT = 1>
hipError_t dispatch(int rt, const Launch& l) {
  if constexpr (16 * RT > kMaxStates) {
    return hipErrorInvalidValue;
  } else {
    if (rt != RT) return dispatch<RT + 1>(rt, l);
    // buffers: what the LDS holds beside the work-groups that the registers
    // allow on a compute unit; the row norms reuse them (64 rows of 17 floats
    // a wave)
    const int per_cu = std::max(1, 4 * waves_per_simd(RT) / l.waves);
    const int fit = (kLdsBytes / per_cu - plane_bytes(RT)) / chunk_bytes(RT);
    const int nbuf = std::min(std::max(fit, 2), chunks(RT));
    const int buf = std::max(nbuf * chunk_bytes(RT), l.waves * 64 * 17 * 4), lds = buf + plane_bytes(RT);
    if (l.prepare)
      return hipFuncSetAttribute((const void*)k_prop_ip<RT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 kLdsBytes);
    hipLaunchKernelGGL((k_prop_ip<RT>), l.grid, dim3(64 * l.waves), lds, l.stream, *l.c, l.groups, nbuf, buf);
    return hipGetLastError();
  }
}

}  // namespace prop_ip
}  // namespace iesh
