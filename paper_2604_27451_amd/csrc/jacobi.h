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
// A chain of short rounds (N - 1 a sweep, 6 to 10 sweeps): latency and LDS traffic
// count.  1024 threads; an item is the 2 x 2 block of the pairs i <= j, to which both
// sides of the rotation are applied at once; only the upper triangle is read and
// kept (the mirror cost a third of the traffic).  A round is two barriers: the first
// wave forms the rotations of a round while the others apply those of the round before
// to the eigenvectors.  Rows padded to an odd number of doubles, since columns are
// accessed as often as rows (unpadded, 64 lanes met one bank); two reciprocal square
// roots a rotation instead of three square roots and four divisions; eigenvalues ranked by
// counting, not by one thread.
#pragma once
#include <hip/hip_runtime.h>

#include "tile.h"

namespace adc2 {

constexpr int JMAX = 64;
constexpr int JLD = JMAX + 1;
constexpr int JSWEEPS = 40;
constexpr int JTHR = 1024;   // blockDim.x of every kernel that calls jacobi_lds

struct JacobiSmem {
  double ar[JMAX][JLD];     // real and imaginary parts of A (upper triangle)
  double ai[JMAX][JLD];
  double2 zt[JMAX][JMAX];   // accumulated rotations: eigenvector c in row c
  double rc[2][JMAX / 2];   // rotations of this round and of the one before
  double2 rw[2][JMAX / 2];
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

// A (n x n, its upper triangle and a real diagonal) in S.ar / S.ai; blockDim.x == JTHR.
// On return (after a barrier): S.zt[c] holds eigenvector c in the
// unsorted order of the diagonal of S.ar, S.perm the ascending order, S.done
// whether the sweeps converged within JSWEEPS.
__device__ inline void jacobi_lds(JacobiSmem& S, int n) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int N = (n + 1) & ~1;   // even number of players: a decoupled zero row joins an odd n
  const int npair = N / 2;
  for (int e = tid; e < JMAX * JMAX; e += JTHR) {
    const int c = e >> 6, r = e & 63;
    S.zt[c][r] = make_double2(r == c ? 1.0 : 0.0, 0.0);
  }
  if (N > n && tid < N) S.ar[tid][n] = S.ai[tid][n] = 0.0;
  __syncthreads();
  // item tid = pj (pj + 1) / 2 + pi of the block update, pi <= pj
  int pj = (int)((sqrtf(8.0f * (float)tid + 1.0f) - 1.0f) * 0.5f);
  if (pj * (pj + 1) / 2 > tid) --pj;
  if ((pj + 1) * (pj + 2) / 2 <= tid) ++pj;
  const int pi = tid - pj * (pj + 1) / 2;
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
  auto geta = [&](int x, int y) {   // A[x][y]
    const int i = min(x, y), j = max(x, y);
    const double im = S.ai[i][j];
    return make_double2(S.ar[i][j], x > y ? -im : im);
  };
  auto puta = [&](int x, int y, double2 v) {
    const int i = min(x, y), j = max(x, y);
    S.ar[i][j] = v.x;
    S.ai[i][j] = x > y ? -v.y : v.y;
  };
  // eigenvector columns of the pairs t = t0, t0 + dt, ... under the rotations of a round
  auto vectors = [&](int round, int buf, int t0, int dt) {
    for (int t = t0; t < npair; t += dt) {
      const double c = S.rc[buf][t];
      const double2 w = S.rw[buf][t];
      if (lane < n && (w.x != 0.0 || w.y != 0.0)) {
        int p, q;
        players(t, round, p, q);
        const double2 zx = S.zt[p][lane], zy = S.zt[q][lane];
        S.zt[p][lane] = csub(cscale(zx, c), cmul(cconj(w), zy));
        S.zt[q][lane] = cadd(cmul(w, zx), cscale(zy, c));
      }
    }
  };
  bool conv = false;
  for (int sweep = 0; sweep <= JSWEEPS; ++sweep) {
    double off = 0.0, tot = 0.0;
    for (int e = tid; e < JMAX * JMAX; e += JTHR) {
      const int i = e >> 6, j = e & 63;
      if (i <= j && j < n) {
        const double v = S.ar[i][j] * S.ar[i][j] + S.ai[i][j] * S.ai[i][j];
        tot += i == j ? v : 2.0 * v;
        if (i != j) off += 2.0 * v;
      }
    }
    jacobi_sum2(S, off, tot);
    conv = off <= 1e-30 * tot || off == 0.0;
    if (conv || sweep == JSWEEPS) break;
    for (int round = 0; round < N - 1; ++round) {
      const int buf = round & 1;
      if (wv == 0) {
        if (lane < npair) {
          int p, q;
          players(lane, round, p, q);
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
          S.rc[buf][lane] = c;
          S.rw[buf][lane] = w;
        }
      } else if (round > 0) {
        vectors(round - 1, buf ^ 1, wv - 1, JTHR / 64 - 1);
      }
      __syncthreads();
      if (pj < npair) {
        int p, q, x, y;
        players(pi, round, p, q);
        players(pj, round, x, y);
        const double ci = S.rc[buf][pi], cj = S.rc[buf][pj];
        const double2 wi = S.rw[buf][pi], wj = S.rw[buf][pj], wjc = cconj(wj), wic = cconj(wi);
        const double2 a00 = geta(p, x), a01 = geta(p, y), a10 = geta(q, x), a11 = geta(q, y);
        // columns: new_x = c x - conj(w) y, new_y = w x + c y
        const double2 u00 = csub(cscale(a00, cj), cmul(wjc, a01)), u01 = cadd(cmul(wj, a00), cscale(a01, cj));
        const double2 u10 = csub(cscale(a10, cj), cmul(wjc, a11)), u11 = cadd(cmul(wj, a10), cscale(a11, cj));
        // rows: new_p = c p - w q, new_q = conj(w) p + c q
        double2 v00 = csub(cscale(u00, ci), cmul(wi, u10)), v01 = csub(cscale(u01, ci), cmul(wi, u11));
        double2 v10 = cadd(cmul(wic, u00), cscale(u10, ci)), v11 = cadd(cmul(wic, u01), cscale(u11, ci));
        if (pi == pj) {
          v00.y = v11.y = 0.0;
          if (wi.x != 0.0 || wi.y != 0.0) v01 = make_double2(0.0, 0.0);
          puta(p, p, v00);
          puta(p, q, v01);
          puta(q, q, v11);
        } else {
          puta(p, x, v00);
          puta(p, y, v01);
          puta(q, x, v10);
          puta(q, y, v11);
        }
      }
      __syncthreads();
    }
    vectors(N - 2, N & 1, wv, JTHR / 64);
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
