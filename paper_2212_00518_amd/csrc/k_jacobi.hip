// Batched eigen-decomposition of general dense symmetric matrices by cyclic
// two-sided Jacobi rotations: the fallback for a one-electron Hamiltonian
// that is not an arrowhead (the arrowhead case has its own secular solver).
//
// A sweep visits every index pair once in m - 1 rounds of m/2 disjoint pairs
// (round-robin schedule over m = n rounded up to even; pairs with the padding
// index are skipped), so the rotations of a round are independent, and
// A <- J^T A J takes one pass over 2x2 blocks (rows of one pair, columns of
// another), each a function of itself alone, so a round works in place.  The
// rotation of pair (p, q)
// annihilates a_pq (Golub and Van Loan, symmetric Schur decomposition):
//   tau = (a_qq - a_pp) / (2 a_pq),  t = sign(tau) / (|tau| + sqrt(1 + tau^2)),
//   c = 1 / sqrt(1 + t^2),  s = t c,  A <- J^T A J,  V <- V J,
// with J the identity except J_pp = J_qq = c, J_pq = s, J_qp = -s.  A pair is
// skipped once |a_pq| <= eps sqrt(|a_pp a_qq|) (eps the FP64 unit roundoff
// times 2; the relative-accuracy stopping rule of Demmel and Veselic) or
// a_pq = 0; the iteration ends after a sweep without rotations or whose
// rotations were all below kSmallRot (or reports non-convergence after
// max_sweeps).
//
// Orders up to IESH_JACOBI_LDS_N: one work-group per matrix, A and the
// accumulated rotations V in LDS (k_jacobi).
//
// Larger orders: A and V together exceed the LDS, and with both in memory
// every round moves them once each way (1.3 MB at n = 201, 26 us a round at the
// memory's rate with 128 matrices).  But V does not feed back into A, and A is
// symmetric.  So k_jacobi_sweep makes one sweep of A alone, one work-group a
// matrix, on its strict lower triangle (in LDS up to n = 201, where it just
// fits; the diagonal lives in registers), and writes the sweep's rotations to
// memory; k_jacobi_vectors then applies them to V, whose rows are independent:
// a wave takes kRows of them through the whole sweep in LDS, without barriers.
// The host launches both for each of the first kPairs sweeps, where those of a
// converged matrix return at once, and one more kernel that makes what is left
// in a work-group a matrix (2 us for each launch that has nothing to do: with
// 60 pairs a diagonal matrix of n = 97 took 0.43 ms, now 0.19).  Past n = 201 a sweep works on all of A
// in memory (its triangle alone took 2.3 times as long), still
// without V.  Measured with the copies of a call, one kernel for all / now:
// 128 matrices of n = 97 7.5 / 4.3 ms, of 201 53.5 / 20.5, of 320 196 / 134, one
// of 201 44 / 10.

#include <algorithm>

#include "iesh_internal.hpp"

namespace iesh {
namespace {

constexpr int kJacThreads = 1024;
constexpr int kJacWaves = kJacThreads / 64;
// A sweep whose rotations all have |tan| below this ends the iteration: the
// off-diagonal elements it leaves are about the square of its largest
// rotation relative to the gaps, so the next sweep would only rotate by
// angles near rounding.
constexpr double kSmallRot = 1e-8;

constexpr int kMaxSweeps = 60;
// Sweeps with a pair of kernels of their own: random matrices of n = 97 to 336
// take 9 to 11, singular ones 10 to 18 (23 at most of those tried).
constexpr int kPairs = 16;

// LDS bytes of k_jacobi: A and V, the rotations of a round and the pairs.
size_t jacobi_lds(int n) {
  const int m = n + (n & 1);
  return sizeof(double) * (2 * (size_t)m * (m + 1) + m) + sizeof(int) * (m + 4);
}

__global__ __launch_bounds__(kJacThreads) void k_jacobi(const double* __restrict__ H, int n,
                                                       double* __restrict__ lam,
                                                       double* __restrict__ Q, int32_t* sweeps_out,
                                                       int max_sweeps) {
  extern __shared__ double sm[];
  const int b = blockIdx.x, tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int m = n + (n & 1), half = m / 2;
  const int ld = m + 1;             // row stride: a column walk spreads over the LDS banks
  double* A = sm;                   // [m][ld]
  double* V = A + (size_t)m * ld;   // [m][ld]
  const auto vix = [ld](int i, int j) { return i * ld + j; };
  double* cs = V + (size_t)m * ld;  // [half] cosines of the round
  double* sn = cs + half;           // [half] sines
  int* pq = reinterpret_cast<int*>(sn + half);  // [m]: p, q of each pair
  int* flag = pq + m;               // [2]: a rotation, a rotation above kSmallRot in this sweep

  const double* Hb = H + (size_t)b * n * n;
  for (int idx = tid; idx < m * m; idx += kJacThreads) {
    const int i = idx / m, j = idx - i * m;
    A[(size_t)i * ld + j] = (i < n && j < n) ? Hb[(size_t)i * n + j] : 0.0;
    V[vix(i, j)] = (i == j) ? 1.0 : 0.0;
  }
  __syncthreads();

  int sweep = 0;
  bool converged = false;
  for (; sweep < max_sweeps; ++sweep) {
    if (tid == 0) {
      flag[0] = 0;
      flag[1] = 0;
    }
    __syncthreads();
    for (int r = 0; r < m - 1; ++r) {
      // the pairs of round r and their rotations
      for (int k = tid; k < half; k += kJacThreads) {
        int p, q;
        if (k == 0) {
          p = r;
          q = m - 1;
        } else {
          p = (r + k) % (m - 1);
          q = (r - k + (m - 1)) % (m - 1);
        }
        if (p > q) {
          const int x = p;
          p = q;
          q = x;
        }
        double c = 1.0, s = 0.0;
        if (q < n) {
          const double apq = A[(size_t)p * ld + q];
          const double app = A[(size_t)p * ld + p], aqq = A[(size_t)q * ld + q];
          if (apq != 0.0 && fabs(apq) > 2.220446049250313e-16 * sqrt(fabs(app) * fabs(aqq))) {
            const double tau = (aqq - app) / (2.0 * apq);
            const double t = copysign(1.0, tau) / (fabs(tau) + sqrt(1.0 + tau * tau));
            c = 1.0 / sqrt(1.0 + t * t);
            s = t * c;
            flag[0] = 1;
            if (fabs(t) > kSmallRot) flag[1] = 1;
          }
        }
        pq[2 * k] = p;
        pq[2 * k + 1] = q;
        cs[k] = c;
        sn[k] = s;
      }
      __syncthreads();
      // A <- J^T A J in one pass: the 2x2 block of rows (p_a, q_a) and
      // columns (p_b, q_b) becomes J_a^T B J_b and depends on that block
      // only, so a lane reads and then writes its own four elements (a wave
      // takes row pairs a = wave, wave + 16, ..., a lane column pairs
      // b = lane, lane + 64, ...; blocks of two pairs without rotation stay).
      // V <- V J_a in the same pass (columns p_a, q_a of V).
      for (int a = wave; a < half; a += kJacWaves) {
        const int pa = pq[2 * a], qa = pq[2 * a + 1];
        const double ca = cs[a], sa = sn[a];
        double* rp = A + (size_t)pa * ld;
        double* rq = A + (size_t)qa * ld;
#pragma unroll 1
        for (int bb = lane; bb < half; bb += 64) {
          const double sb = sn[bb];
          if (sa == 0.0 && sb == 0.0) continue;
          const int pb = pq[2 * bb], qb = pq[2 * bb + 1];
          const double cb = cs[bb];
          const double a_pp = rp[pb], a_pq = rp[qb], a_qp = rq[pb], a_qq = rq[qb];
          // rows: J_a^T B
          const double xpp = ca * a_pp - sa * a_qp, xpq = ca * a_pq - sa * a_qq;
          const double xqp = sa * a_pp + ca * a_qp, xqq = sa * a_pq + ca * a_qq;
          // columns: (J_a^T B) J_b; the annihilated pair is set to zero
          rp[pb] = cb * xpp - sb * xpq;
          rp[qb] = (bb == a) ? 0.0 : sb * xpp + cb * xpq;
          rq[pb] = (bb == a) ? 0.0 : cb * xqp - sb * xqq;
          rq[qb] = sb * xqp + cb * xqq;
        }
        if (sa != 0.0) {
#pragma unroll 1
          for (int j = lane; j < m; j += 64) {
            const double vp = V[vix(j, pa)], vq = V[vix(j, qa)];
            V[vix(j, pa)] = ca * vp - sa * vq;
            V[vix(j, qa)] = sa * vp + ca * vq;
          }
        }
      }
      __syncthreads();
    }
    const int any = flag[0], large = flag[1];
    __syncthreads();
    if (!any || !large) {
      converged = true;
      break;
    }
  }

  // ascending order (ties by index) and the phase: the first component of
  // each eigenvector above 1e-12 of its largest is made positive
  int* rank = pq;  // reuse: [m]
  for (int j = tid; j < n; j += kJacThreads) {
    const double dj = A[(size_t)j * ld + j];
    int rk = 0;
    for (int i = 0; i < n; ++i) {
      const double di = A[(size_t)i * ld + i];
      rk += (di < dj || (di == dj && i < j)) ? 1 : 0;
    }
    rank[j] = rk;
  }
  __syncthreads();
  for (int j = tid; j < n; j += kJacThreads) {
    double vmax = 0.0;
    for (int i = 0; i < n; ++i) vmax = fmax(vmax, fabs(V[vix(i, j)]));
    double sgn = 1.0;
    for (int i = 0; i < n; ++i) {
      const double v = V[vix(i, j)];
      if (fabs(v) > 1e-12 * vmax) {
        sgn = v < 0.0 ? -1.0 : 1.0;
        break;
      }
    }
    const int rk = rank[j];
    lam[(size_t)b * n + rk] = A[(size_t)j * ld + j];
    double* Qb = Q + (size_t)b * n * n;
    for (int i = 0; i < n; ++i) Qb[(size_t)i * n + rk] = sgn * V[vix(i, j)];
  }
  if (tid == 0 && sweeps_out) sweeps_out[b] = converged ? sweep + 1 : -1;
}

// ---- orders beyond IESH_JACOBI_LDS_N ----------------------------------------

constexpr int kRows = 8;        // rows of V to a wave
constexpr int kSlots = (kMaxStates / 2 + 63) / 64;  // pairs of a round to a lane
constexpr size_t kJacLds = 160 * 1024;

// A matrix in the work space (2 m (m + 1) doubles): V, A, its diagonal, and
// the number of the sweep that converged (0: none yet) and whether the last one
// rotated.  A is the strict
// lower triangle (row i at i (i - 1) / 2) and one element that stays zero, or,
// past the order whose triangle fits into the LDS, the whole [m][m].
struct JacWork {
  double *V, *A, *diag;
  int32_t *done, *rotated;
};

__host__ __device__ constexpr int tri_size(int n) { return n * (n - 1) / 2; }

size_t jacobi_sweep_lds(int n) { return sizeof(double) * (tri_size(n) + 1 + 2 * ((n + 1) / 2)) + sizeof(int) * ((n + 1) / 2); }

__device__ inline JacWork jac_work(double* work, int n, int b) {
  const int m = n + (n & 1);
  JacWork w;
  w.diag = work + (size_t)b * 2 * m * (m + 1);
  w.done = reinterpret_cast<int32_t*>(w.diag + n);
  w.rotated = w.done + 1;
  w.V = w.diag + n + 1;
  w.A = w.V + (size_t)n * n;
  return w;
}

// Rotations of one sweep, [round][pair][c, s] without the padding pair: n (n - 1)
// doubles, kept where the eigenvectors will be written.
__device__ inline double* jac_rot(double* Q, int n, int b) { return Q + (size_t)b * n * n; }

// Pair k of round r, p < q; q = n is the padding index.
__device__ inline void jac_pair(int r, int k, int m, int& p, int& q) {
  const int R = m - 1;
  int x = r + k, y = r - k;
  if (x >= R) x -= R;
  if (y < 0) y += R;
  if (k == 0) y = R;
  p = min(x, y);
  q = max(x, y);
}

// Sweep number `sweep` of A.  The first wave computes a round's rotations; its
// lanes hold the diagonal in the round-robin order, where a round moves every
// element to a neighbouring pair.  Then every thread updates 2x2 blocks of two
// pairs a and b = a + d, d = 1 .. half/2, each unordered pair of pairs once.
// Bound by the vector instructions of the blocks (about 80 each, a quarter of
// them FP64) and the LDS (at n = 201 6,600 of 11,000 cycles a round, more than
// half of them bank conflicts, though the triangular row offsets keep a column
// walk off single banks), then by the rotations' serial chain.
__device__ __forceinline__ void sweep_lds(const double* __restrict__ H, int n, double* Q, const JacWork& w, int b, int sweep,
                                          double* sm) {
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int m = n + (n & 1), half = m / 2, odd = n & 1, nt = tri_size(n);
  double* T = sm;            // strict lower triangle, [nt] is zero
  double* cs = sm + nt + 1;  // [half] cosine, sine
  int* pq = reinterpret_cast<int*>(cs + 2 * half);  // [half] p + (q << 16)
  double* rot = jac_rot(Q, n, b);
  const int np = n / 2;  // pairs of a round without the padding one

  if (sweep == 0) {
    const double* Hb = H + (size_t)b * n * n;
    for (int idx = tid; idx < n * n; idx += kJacThreads) {
      const int j = idx / n, i = idx - j * n;
      if (i > j) T[tri_size(i) + j] = Hb[idx];
      if (i == j) w.diag[i] = Hb[idx];
    }
    if (tid == 0) T[nt] = 0.0;
  } else {
    for (int idx = tid; idx <= nt; idx += kJacThreads) T[idx] = w.A[idx];
  }
  __syncthreads();
  // diagonal elements of the indices r + k (dx) and r - k (dy) of pair k
  double dx[kSlots] = {}, dy[kSlots] = {};
  bool any = false, large = false;
  if (wave == 0) {
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const int k = lane + 64 * u;
      if (k < half) {
        dx[u] = w.diag[k];
        const int y = k == 0 ? m - 1 : m - 1 - k;
        dy[u] = y < n ? w.diag[y] : 0.0;
      }
    }
  }
  const int a0 = tid % half, d0 = tid / half + 1, da = kJacThreads % half, dd = kJacThreads / half;
  for (int r = 0; r < m - 1; ++r) {
    if (wave == 0) {
#pragma unroll
      for (int u = 0; u < kSlots; ++u) {
        const int k = lane + 64 * u;
        if (k < half) {
          int p, q;
          jac_pair(r, k, m, p, q);
          const bool swap = (r + k >= m - 1 ? r + k - (m - 1) : r + k) != p;  // p is r - k
          double c = 1.0, s = 0.0;
          if (q < n) {
            const int e = tri_size(q) + p;
            const double apq = T[e], app = swap ? dy[u] : dx[u], aqq = swap ? dx[u] : dy[u];
            if (apq != 0.0 && fabs(apq) > 2.220446049250313e-16 * sqrt(fabs(app) * fabs(aqq))) {
              const double tau = (aqq - app) / (2.0 * apq);
              const double t = copysign(1.0, tau) / (fabs(tau) + sqrt(1.0 + tau * tau));
              c = 1.0 / sqrt(1.0 + t * t);
              s = t * c;
              any = true;
              large |= fabs(t) > kSmallRot;
              const double np_ = c * (c * app - s * apq) - s * (c * apq - s * aqq);
              const double nq_ = s * (s * app + c * apq) + c * (s * apq + c * aqq);
              dx[u] = swap ? nq_ : np_;
              dy[u] = swap ? np_ : nq_;
              T[e] = 0.0;
            }
            double* ro = rot + 2 * ((size_t)r * np + k - odd);
            ro[0] = c;
            ro[1] = s;
          }
          cs[2 * k] = c;
          cs[2 * k + 1] = s;
          pq[k] = p | (q << 16);
        }
      }
    }
    __syncthreads();
    for (int a = a0, d = d0; d <= half / 2;) {
      if (2 * d != half || a < d) {
        const int bb = a + d < half ? a + d : a + d - half;
        const double ca = cs[2 * a], sa = cs[2 * a + 1], cb = cs[2 * bb], sb = cs[2 * bb + 1];
        if (sa != 0.0 || sb != 0.0) {
          const int qa = pq[a], qb = pq[bb];
          // element of two indices; any with the padding index is the zero one
          const auto at = [&](int i, int j) {
            const int hi = max(i, j), lo = min(i, j);
            return min((int)(__umul24(hi, hi - 1) >> 1) + lo, nt);
          };
          const int pai = qa & 0xffff, qai = qa >> 16, pbi = qb & 0xffff, qbi = qb >> 16;
          const int epp = at(pai, pbi), epq = at(pai, qbi), eqp = at(qai, pbi), eqq = at(qai, qbi);
          const double a_pp = T[epp], a_pq = T[epq], a_qp = T[eqp], a_qq = T[eqq];
          // rows: J_a^T B
          const double xpp = ca * a_pp - sa * a_qp, xpq = ca * a_pq - sa * a_qq;
          const double xqp = sa * a_pp + ca * a_qp, xqq = sa * a_pq + ca * a_qq;
          // columns: (J_a^T B) J_b
          T[epp] = cb * xpp - sb * xpq;
          T[epq] = sb * xpp + cb * xpq;
          T[eqp] = cb * xqp - sb * xqq;
          T[eqq] = sb * xqp + cb * xqq;
        }
      }
      a += da;
      d += dd;
      if (a >= half) {
        a -= half;
        ++d;
      }
    }
    if (wave == 0) {  // the diagonal moves on to the pairs of the next round
      double nx[kSlots], ny[kSlots];
#pragma unroll
      for (int u = 0; u < kSlots; ++u) {
        const int k = lane + 64 * u;
        double x = __shfl(dx[u], (lane + 1) & 63), y = __shfl(dy[u], (lane + 63) & 63);
        if (u + 1 < kSlots) {
          const double x1 = __shfl(dx[u + 1 < kSlots ? u + 1 : u], 0);
          x = lane == 63 ? x1 : x;
        }
        if (u > 0) {
          const double y1 = __shfl(dy[u > 0 ? u - 1 : 0], 63);
          y = lane == 0 ? y1 : y;
        } else {
          const double x0 = __shfl(dx[0], 0);
          y = k == 0 ? dy[0] : k == 1 ? x0 : y;
        }
        nx[u] = k == half - 1 ? dy[u] : x;
        ny[u] = y;
      }
#pragma unroll
      for (int u = 0; u < kSlots; ++u) {
        dx[u] = nx[u];
        dy[u] = ny[u];
      }
    }
    __syncthreads();
  }
  for (int idx = tid; idx <= nt; idx += kJacThreads) w.A[idx] = T[idx];
  if (wave == 0) {  // a whole sweep of rounds has brought every element back
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const int k = lane + 64 * u;
      if (k < half) {
        w.diag[k] = dx[u];
        const int y = k == 0 ? m - 1 : m - 1 - k;
        if (y < n) w.diag[y] = dy[u];
      }
    }
    const bool some = __any(any), more = some && __any(large);
    if (lane == 0) {
      *w.done = more ? 0 : sweep + 1;
      *w.rotated = some;
    }
  }
}

__global__ __launch_bounds__(kJacThreads) void k_jacobi_sweep(const double* __restrict__ H, int n, double* Q,
                                                             double* work, int sweep) {
  extern __shared__ double sm[];
  const JacWork w = jac_work(work, n, blockIdx.x);
  if (sweep > 0 && *w.done != 0) return;
  sweep_lds(H, n, Q, w, blockIdx.x, sweep, sm);
}

// The same with all of A in memory, where a round reads and writes it once:
// rows of a pair by lanes along the columns, both triangles.
__device__ __forceinline__ void sweep_mem(const double* __restrict__ H, int n, double* Q, const JacWork& w, int b, int sweep) {
  __shared__ double cs[kMaxStates / 2], sn[kMaxStates / 2];
  __shared__ int pq[kMaxStates], flag[2];  // a rotation, a rotation above kSmallRot
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int m = n + (n & 1), half = m / 2, odd = n & 1, np = n / 2;
  double* A = w.A;
  double* rot = jac_rot(Q, n, b);
  if (sweep == 0) {
    const double* Hb = H + (size_t)b * n * n;
    for (int idx = tid; idx < m * m; idx += kJacThreads) {
      const int i = idx / m, j = idx - i * m;
      A[idx] = (i < n && j < n) ? Hb[(size_t)i * n + j] : 0.0;
    }
  }
  if (tid < 2) flag[tid] = 0;
  __syncthreads();
  for (int r = 0; r < m - 1; ++r) {
    if (tid < half) {
      int p, q;
      jac_pair(r, tid, m, p, q);
      double c = 1.0, s = 0.0;
      if (q < n) {
        const double apq = A[p * m + q], app = A[p * m + p], aqq = A[q * m + q];
        if (apq != 0.0 && fabs(apq) > 2.220446049250313e-16 * sqrt(fabs(app) * fabs(aqq))) {
          const double tau = (aqq - app) / (2.0 * apq);
          const double t = copysign(1.0, tau) / (fabs(tau) + sqrt(1.0 + tau * tau));
          c = 1.0 / sqrt(1.0 + t * t);
          s = t * c;
          flag[0] = 1;
          if (fabs(t) > kSmallRot) flag[1] = 1;
        }
        double* ro = rot + 2 * ((size_t)r * np + tid - odd);
        ro[0] = c;
        ro[1] = s;
      }
      pq[2 * tid] = p;
      pq[2 * tid + 1] = q;
      cs[tid] = c;
      sn[tid] = s;
    }
    __syncthreads();
    for (int a = wave; a < half; a += kJacWaves) {
      const double ca = cs[a], sa = sn[a];
      double* rp = A + pq[2 * a] * m;
      double* rq = A + pq[2 * a + 1] * m;
#pragma unroll 1
      for (int bb = lane; bb < half; bb += 64) {
        const double sb = sn[bb];
        if (sa == 0.0 && sb == 0.0) continue;
        const int pb = pq[2 * bb], qb = pq[2 * bb + 1];
        const double cb = cs[bb];
        const double a_pp = rp[pb], a_pq = rp[qb], a_qp = rq[pb], a_qq = rq[qb];
        const double xpp = ca * a_pp - sa * a_qp, xpq = ca * a_pq - sa * a_qq;
        const double xqp = sa * a_pp + ca * a_qp, xqq = sa * a_pq + ca * a_qq;
        rp[pb] = cb * xpp - sb * xpq;
        rp[qb] = (bb == a) ? 0.0 : sb * xpp + cb * xpq;
        rq[pb] = (bb == a) ? 0.0 : cb * xqp - sb * xqq;
        rq[qb] = sb * xqp + cb * xqq;
      }
    }
    __syncthreads();
  }
  if (tid < n) w.diag[tid] = A[tid * m + tid];
  if (tid == 0) {
    *w.done = flag[0] && flag[1] ? 0 : sweep + 1;
    *w.rotated = flag[0];
  }
}

__global__ __launch_bounds__(kJacThreads) void k_jacobi_sweep_mem(const double* __restrict__ H, int n, double* Q,
                                                                 double* work, int sweep) {
  const JacWork w = jac_work(work, n, blockIdx.x);
  if (sweep > 0 && *w.done != 0) return;
  sweep_mem(H, n, Q, w, blockIdx.x, sweep);
}

// V <- V J over the rotations of one sweep, kRows rows from i0 on, by one wave
// with row: LDS [kRows][n].  Bound by the LDS (each round reads and writes every
// element of V once).
__device__ __forceinline__ void rotate_rows(int n, const double* rot, const JacWork& w, int i0, int sweep, double* row) {
  const int lane = threadIdx.x & 63, ld = n;
  const int m = n + (n & 1), half = m / 2, odd = n & 1, np = n / 2;
  const bool rotated = *w.rotated != 0;
  if (!rotated && sweep > 0) return;
  for (int x = 0; x < kRows; ++x)
    for (int j = lane; j < n; j += 64)
      row[x * ld + j] = sweep == 0 || i0 + x >= n ? (j == i0 + x ? 1.0 : 0.0) : w.V[(size_t)(i0 + x) * n + j];
  double c[kSlots], s[kSlots];
  const auto load = [&](int r) {
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const int k = lane + 64 * u;
      c[u] = 1.0;
      s[u] = 0.0;
      if (k >= odd && k < half) {
        const double* ro = rot + 2 * ((size_t)r * np + k - odd);
        c[u] = ro[0];
        s[u] = ro[1];
      }
    }
  };
  if (rotated) load(0);
  for (int r = 0; r < m - 1 && rotated; ++r) {
    double cc[kSlots], ss[kSlots];
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      cc[u] = c[u];
      ss[u] = s[u];
    }
    if (r + 1 < m - 1) load(r + 1);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      if (ss[u] != 0.0) {  // never the padding pair or one past the last
        int p, q;
        jac_pair(r, lane + 64 * u, m, p, q);
        double vp[kRows], vq[kRows];
#pragma unroll
        for (int x = 0; x < kRows; ++x) {
          vp[x] = row[x * ld + p];
          vq[x] = row[x * ld + q];
        }
#pragma unroll
        for (int x = 0; x < kRows; ++x) {
          row[x * ld + p] = cc[u] * vp[x] - ss[u] * vq[x];
          row[x * ld + q] = ss[u] * vp[x] + cc[u] * vq[x];
        }
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int x = 0; x < kRows && i0 + x < n; ++x)
    for (int j = lane; j < n; j += 64) w.V[(size_t)(i0 + x) * n + j] = row[x * ld + j];
}

__global__ __launch_bounds__(64) void k_jacobi_vectors(int n, int groups, double* Q, double* work, int sweep) {
  extern __shared__ double row[];
  const int b = blockIdx.x / groups;
  const JacWork w = jac_work(work, n, b);
  const int done = *w.done;
  if (done != 0 && done != sweep + 1) return;  // converged before this sweep
  rotate_rows(n, jac_rot(Q, n, b), w, (blockIdx.x - b * groups) * kRows, sweep, row);
}

// The sweeps from `first` on of the matrices that need them, A and V in one
// work-group (`waves` of it share the rows of V, as many as their LDS holds).
template <bool kTri>
__global__ __launch_bounds__(kJacThreads) void k_jacobi_rest(const double* __restrict__ H, int n, double* Q, double* work,
                                                            int first, int waves) {
  extern __shared__ double sm[];
  const int b = blockIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const JacWork w = jac_work(work, n, b);
  if (*w.done != 0) return;
  for (int sweep = first; sweep < kMaxSweeps; ++sweep) {
    if constexpr (kTri)
      sweep_lds(H, n, Q, w, b, sweep, sm);
    else
      sweep_mem(H, n, Q, w, b, sweep);
    __syncthreads();  // A's and V's parts of the LDS are the same, and V reads the sweep's rotations
    if (wave < waves)
      for (int i0 = wave * kRows; i0 < n; i0 += waves * kRows)
        rotate_rows(n, jac_rot(Q, n, b), w, i0, sweep, sm + (size_t)wave * kRows * n);
    const int done = *w.done;
    __syncthreads();  // every wave has read it, and left V's part, before the next sweep
    if (done != 0) break;
  }
}

// Ascending order (ties by index) and the phase: the first component of each
// eigenvector above 1e-12 of its largest is made positive.  Column j of V is
// shared by threads j, j + n, ...
__global__ __launch_bounds__(kJacThreads) void k_jacobi_order(int n, double* __restrict__ lam, double* __restrict__ Q,
                                                             int32_t* sweeps_out, double* work) {
  __shared__ double d[kMaxStates], part[kJacThreads];
  __shared__ double sgn[kMaxStates];
  __shared__ int rank[kMaxStates], first[kMaxStates];
  const int b = blockIdx.x, tid = threadIdx.x;
  const JacWork w = jac_work(work, n, b);
  const int groups = kJacThreads / n, grp = tid / n, j = tid - grp * n;
  const bool on = grp < groups;
  if (tid < n) {
    d[tid] = w.diag[tid];
    first[tid] = n;
  }
  __syncthreads();
  double vmax = 0.0;
  if (on)
    for (int i = grp; i < n; i += groups) vmax = fmax(vmax, fabs(w.V[(size_t)i * n + j]));
  part[tid] = vmax;
  if (tid < n) {
    const double dj = d[tid];
    int rk = 0;
    for (int i = 0; i < n; ++i) rk += (d[i] < dj || (d[i] == dj && i < tid)) ? 1 : 0;
    rank[tid] = rk;
    lam[(size_t)b * n + rk] = dj;
  }
  __syncthreads();
  if (on) {
    for (int g = 0; g < groups; ++g) vmax = fmax(vmax, part[g * n + j]);
    for (int i = grp; i < n; i += groups)
      if (fabs(w.V[(size_t)i * n + j]) > 1e-12 * vmax) {
        atomicMin(&first[j], i);
        break;
      }
  }
  __syncthreads();
  if (tid < n) sgn[tid] = first[tid] < n && w.V[(size_t)first[tid] * n + tid] < 0.0 ? -1.0 : 1.0;
  __syncthreads();
  if (on)
    for (int i = grp; i < n; i += groups) Q[((size_t)b * n + i) * n + rank[j]] = sgn[j] * w.V[(size_t)i * n + j];
  if (tid == 0 && sweeps_out) sweeps_out[b] = *w.done != 0 ? *w.done : -1;
}

hipError_t launch_jacobi_large(const double* H, int n, int batch, double* lam, double* Q, int32_t* sweeps,
                               double* work, hipStream_t s) {
  const size_t lds = jacobi_sweep_lds(n), vlds = sizeof(double) * kRows * n;
  const bool tri = lds <= kJacLds;
  const int groups = (n + kRows - 1) / kRows;
  // LDS of the kernel for the rest (beside sweep_mem's own arrays)
  const size_t own = tri ? 0 : sizeof(double) * kMaxStates + sizeof(int) * (kMaxStates + 2) + 64;
  const int waves = (int)std::min<size_t>(kJacWaves, (kJacLds - own) / vlds);
  const size_t rlds = std::max(tri ? lds : 0, waves * vlds);
  const void* rest = tri ? (const void*)k_jacobi_rest<true> : (const void*)k_jacobi_rest<false>;
  hipError_t e = hipFuncSetAttribute(rest, hipFuncAttributeMaxDynamicSharedMemorySize, (int)rlds);
  if (e == hipSuccess && tri)
    e = hipFuncSetAttribute((const void*)k_jacobi_sweep, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  for (int sweep = 0; sweep < kPairs; ++sweep) {
    if (tri)
      hipLaunchKernelGGL(k_jacobi_sweep, dim3(batch), dim3(kJacThreads), lds, s, H, n, Q, work, sweep);
    else
      hipLaunchKernelGGL(k_jacobi_sweep_mem, dim3(batch), dim3(kJacThreads), 0, s, H, n, Q, work, sweep);
    hipLaunchKernelGGL(k_jacobi_vectors, dim3(batch * groups), dim3(64), vlds, s, n, groups, Q, work, sweep);
  }
  if (tri)
    hipLaunchKernelGGL(k_jacobi_rest<true>, dim3(batch), dim3(kJacThreads), rlds, s, H, n, Q, work, kPairs, waves);
  else
    hipLaunchKernelGGL(k_jacobi_rest<false>, dim3(batch), dim3(kJacThreads), rlds, s, H, n, Q, work, kPairs, waves);
  hipLaunchKernelGGL(k_jacobi_order, dim3(batch), dim3(kJacThreads), 0, s, n, lam, Q, sweeps, work);
  return hipGetLastError();
}

}  // namespace

size_t jacobi_work_elems(int n, int batch) {
  if (n <= IESH_JACOBI_LDS_N) return 0;
  const size_t m = n + (n & 1);
  return (size_t)batch * 2 * m * (m + 1);
}

hipError_t launch_jacobi(const double* H, int n, int batch, double* lam, double* Q, int32_t* sweeps,
                         double* work, hipStream_t s) {
  if (n > IESH_JACOBI_LDS_N) return launch_jacobi_large(H, n, batch, lam, Q, sweeps, work, s);
  const size_t lds = jacobi_lds(n);
  const hipError_t e = hipFuncSetAttribute((const void*)k_jacobi, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_jacobi, dim3(batch), dim3(kJacThreads), lds, s, H, n, lam, Q, sweeps, kMaxSweeps);
  return hipGetLastError();
}

}  // namespace iesh
