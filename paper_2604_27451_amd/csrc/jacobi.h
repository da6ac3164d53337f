// jacobi.h -- one-workgroup parallel cyclic Jacobi eigensolver for a complex
// Hermitian n x n matrix (n <= 64) held in LDS, FP64.  Used for the
// subspace eigenproblems of both Davidson solvers (the projected matrix
// V^H M V of the full-space solver, the projected singles blocks and the
// folded matrices G(omega) of the folded solver).
//
// Pair (p,q) rotation J = [[c, w], [-conj(w), c]], a = (a_qq - a_pp)/2,
// r = sqrt(a^2 + |a_pq|^2), c = sqrt((r + |a|)/(2r)), w = sign(a) a_pq/(2 r c),
// zeroes a_pq of J^H A J; all n/2 disjoint pairs of a round-robin round are
// applied together.  Sweeps stop when the off-diagonal Frobenius norm is
// below 1e-15 of the whole (squared: 1e-30).
//
// A chain of short rounds (N - 1 a sweep, 6 to 10 sweeps): latency counts.  1024
// threads, thread (i, j) owning the 2 x 2 block of the pairs i <= j and applying
// both sides of the rotation to it (and its mirror) at once, so a round is two
// barriers; rows padded to an odd number of doubles, since columns are
// accessed as often as rows (unpadded, 64 lanes met one bank); two reciprocal
// square roots a rotation instead of three square roots and four divisions;
// eigenvalues ranked by counting, not by one thread.
#pragma once
#include <hip/hip_runtime.h>

#include "tile.h"

namespace adc2 {

constexpr int JMAX = 64;
constexpr int JLD = JMAX + 1;
constexpr int JSWEEPS = 40;
constexpr int JTHR = 1024;   // blockDim.x of every kernel that calls jacobi_lds

struct JacobiSmem {
  double ar[JMAX][JLD];     // real and imaginary parts of A (both triangles)
  double ai[JMAX][JLD];
  double2 zt[JMAX][JMAX];   // accumulated rotations: eigenvector c in row c
  double rc[JMAX / 2];
  double2 rw[JMAX / 2];
  double red[2][JTHR / 64];
  int perm[JMAX];           // ascending order of the eigenvalues ar[perm[i]][perm[i]]
  int done;                 // 1 once the sweeps converged
};

// Sum over the block of two values a thread, in every thread (two barriers).
__device__ __forceinline__ void jacobi_sum2(JacobiSmem& S, double& x, double& y) {
  for (int off = 32; off > 0; off >>= 1) {
    x += __shfl_xor(x, off);
    y += __shfl_xor(y, off);
  }
  if ((threadIdx.x & 63) == 0) {
    S.red[0][threadIdx.x >> 6] = x;
    S.red[1][threadIdx.x >> 6] = y;
  }
  __syncthreads();
  x = y = 0.0;
  for (int w = 0; w < JTHR / 64; ++w) {
    x += S.red[0][w];
    y += S.red[1][w];
  }
  __syncthreads();
}

// A (n x n, both triangles consistent) in S.ar / S.ai; blockDim.x == JTHR.
// On return (after a barrier): S.zt[c] holds eigenvector c (VEC) in the
// unsorted order of the diagonal of S.ar, S.perm the ascending order, S.done
// whether the sweeps converged within JSWEEPS.
template <bool VEC>
__device__ inline void jacobi_lds(JacobiSmem& S, int n) {
  const int tid = threadIdx.x;
  const int N = (n + 1) & ~1;   // even number of players: a decoupled zero row joins an odd n
  const int npair = N / 2;
  if (VEC)
    for (int e = tid; e < JMAX * JMAX; e += JTHR) {
      const int c = e >> 6, r = e & 63;
      S.zt[c][r] = make_double2(r == c ? 1.0 : 0.0, 0.0);
    }
  if (N > n && tid < N) S.ar[n][tid] = S.ai[n][tid] = S.ar[tid][n] = S.ai[tid][n] = 0.0;
  __syncthreads();
  const int pi = tid >> 5, pj = tid & 31;
  // the players of pair t in a round: player 0 fixed, players 1..N-1 rotate
  auto players = [&](int t, int round, int& p, int& q) {
    int a = 0, b = 1 + round;
    if (t > 0) {
      a = round + t;
      a = 1 + (a >= N - 1 ? a - (N - 1) : a);
      b = round - t;
      b = 1 + (b < 0 ? b + (N - 1) : b);
    }
    p = min(a, b);
    q = max(a, b);
  };
  bool conv = false;
  for (int sweep = 0; sweep <= JSWEEPS; ++sweep) {
    double off = 0.0, tot = 0.0;
    for (int e = tid; e < JMAX * JMAX; e += JTHR) {
      const int i = e >> 6, j = e & 63;
      if (i < n && j < n) {
        const double v = S.ar[i][j] * S.ar[i][j] + S.ai[i][j] * S.ai[i][j];
        tot += v;
        if (i != j) off += v;
      }
    }
    jacobi_sum2(S, off, tot);
    conv = off <= 1e-30 * tot || off == 0.0;
    if (conv || sweep == JSWEEPS) break;
    for (int round = 0; round < N - 1; ++round) {
      if (tid < npair) {
        int p, q;
        players(tid, round, p, q);
        double c = 1.0;
        double2 w = make_double2(0.0, 0.0);
        const double br = S.ar[p][q], bi = S.ai[p][q];
        const double b2 = br * br + bi * bi;
        const double app = S.ar[p][p], aqq = S.ar[q][q];
        const double sc = fabs(app) + fabs(aqq);
        if (b2 > 1e-290 && b2 > 1e-36 * sc * sc) {
          const double a = 0.5 * (aqq - app);
          const double ir = rsqrt(fma(a, a, b2));
          const double c2 = fma(0.5 * fabs(a), ir, 0.5);
          const double ic = rsqrt(c2);
          c = c2 * ic;
          const double f = (a >= 0.0 ? 0.5 : -0.5) * ir * ic;
          w = make_double2(f * br, f * bi);
        }
        S.rc[tid] = c;
        S.rw[tid] = w;
      }
      __syncthreads();
      if (pi <= pj && pj < npair) {
        int p, q, x, y;
        players(pi, round, p, q);
        players(pj, round, x, y);
        const double ci = S.rc[pi], cj = S.rc[pj];
        const double2 wi = S.rw[pi], wj = S.rw[pj], wjc = cconj(wj), wic = cconj(wi);
        const double2 a00 = make_double2(S.ar[p][x], S.ai[p][x]), a01 = make_double2(S.ar[p][y], S.ai[p][y]);
        const double2 a10 = make_double2(S.ar[q][x], S.ai[q][x]), a11 = make_double2(S.ar[q][y], S.ai[q][y]);
        // columns: new_x = c x - conj(w) y, new_y = w x + c y
        const double2 u00 = csub(cscale(a00, cj), cmul(wjc, a01)), u01 = cadd(cmul(wj, a00), cscale(a01, cj));
        const double2 u10 = csub(cscale(a10, cj), cmul(wjc, a11)), u11 = cadd(cmul(wj, a10), cscale(a11, cj));
        // rows: new_p = c p - w q, new_q = conj(w) p + c q
        double2 v00 = csub(cscale(u00, ci), cmul(wi, u10)), v01 = csub(cscale(u01, ci), cmul(wi, u11));
        double2 v10 = cadd(cmul(wic, u00), cscale(u10, ci)), v11 = cadd(cmul(wic, u01), cscale(u11, ci));
        if (pi == pj) {
          v00.y = v11.y = 0.0;
          if (wi.x != 0.0 || wi.y != 0.0) v01 = v10 = make_double2(0.0, 0.0);
        }
        S.ar[p][x] = v00.x;
        S.ai[p][x] = v00.y;
        S.ar[p][y] = v01.x;
        S.ai[p][y] = v01.y;
        S.ar[q][x] = v10.x;
        S.ai[q][x] = v10.y;
        S.ar[q][y] = v11.x;
        S.ai[q][y] = v11.y;
        if (pi != pj) {
          S.ar[x][p] = v00.x;
          S.ai[x][p] = -v00.y;
          S.ar[y][p] = v01.x;
          S.ai[y][p] = -v01.y;
          S.ar[x][q] = v10.x;
          S.ai[x][q] = -v10.y;
          S.ar[y][q] = v11.x;
          S.ai[y][q] = -v11.y;
        }
      }
      if (VEC)
        for (int t = tid >> 6; t < npair; t += JTHR / 64) {
          const int r = tid & 63;
          const double c = S.rc[t];
          const double2 w = S.rw[t];
          if (r < n && (w.x != 0.0 || w.y != 0.0)) {
            int p, q;
            players(t, round, p, q);
            const double2 zx = S.zt[p][r], zy = S.zt[q][r];
            S.zt[p][r] = csub(cscale(zx, c), cmul(cconj(w), zy));
            S.zt[q][r] = cadd(cmul(w, zx), cscale(zy, c));
          }
        }
      __syncthreads();
    }
  }
  if (tid == 0) S.done = conv ? 1 : 0;
  if (tid < n) {   // rank of each eigenvalue
    const double v = S.ar[tid][tid];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double u = S.ar[j][j];
      rank += (u < v || (u == v && j < tid)) ? 1 : 0;
    }
    S.perm[rank] = tid;
  }
  __syncthreads();
}

}  // namespace adc2
