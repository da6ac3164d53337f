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
// A chain of short rounds (N - 1 a sweep, 6 to 10 sweeps): latency, instructions
// and LDS traffic count.  1024 threads; an item is the 2 x 2 block of the pairs i <= j,
// to which both sides of the rotation are applied at once; only the upper triangle
// is read and kept.  The players of a round sit at fixed places, pair t at t and
// t + N/2, and the tournament moves the data: what an item writes goes where the
// next round finds it, so all addresses are constants of a thread (players of
// changing index cost more instructions than the rotations: 3500 cycles a round of 48).
// While the first wave forms the rotations of a round, the others apply those of the
// round before to the eigenvectors.  Rows padded to 65 entries, so that neither rows nor
// columns meet one bank; two reciprocal square roots a rotation instead of three square
// roots and four divisions; eigenvalues ranked by counting, not by one thread.
#pragma once
#include <hip/hip_runtime.h>

#include "eigorder.h"
#include "tile.h"

namespace adc2 {

constexpr int JMAX = 64;
constexpr int JLD = JMAX + 1;
constexpr int JSWEEPS = 40;
constexpr int JTHR = 1024;   // blockDim.x of every kernel that calls jacobi_lds

struct JacobiSmem {
  double2 a[JMAX][JLD];     // A (upper triangle)
  double2 zt[JMAX][JMAX];   // accumulated rotations: eigenvector c in row c
  double rc[2][JMAX / 2];   // rotations of this round and of the one before
  double2 rw[2][JMAX / 2];
  double red[2][JTHR / 64];
  int perm[JMAX];           // ascending order of the eigenvalues a[perm[i]][perm[i]].x
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

// A (n x n, its upper triangle and a real diagonal) in S.a; blockDim.x == JTHR.
// On return (after a barrier): S.zt[c] holds eigenvector c in the
// unsorted order of the diagonal of S.a, S.perm the ascending order, S.done
// whether the sweeps converged within JSWEEPS.
__device__ inline void jacobi_lds(JacobiSmem& S, int n) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int N = (n + 1) & ~1;   // even number of players: a decoupled zero row joins an odd n
  const int np = N / 2;
  for (int e = tid; e < JMAX * JMAX; e += JTHR) {
    const int c = e >> 6, r = e & 63;
    S.zt[c][r] = make_double2(r == c ? 1.0 : 0.0, 0.0);
  }
  if (N > n && tid < N) S.a[tid][n] = make_double2(0.0, 0.0);
  // where the player at place x is in the next round: 0 stays, the others go round
  // 1 .. np - 1 downwards, then np .. N - 1 upwards
  auto next = [&](int x) {
    if (x == 0 || np == 1) return x;
    if (x < np) return x == 1 ? np : x - 1;
    return x == N - 1 ? np - 1 : x + 1;
  };
  // item tid = pj (pj + 1) / 2 + pi of the block update, pi <= pj
  int pj = (int)((sqrtf(8.0f * (float)tid + 1.0f) - 1.0f) * 0.5f);
  if (pj * (pj + 1) / 2 > tid) --pj;
  if ((pj + 1) * (pj + 2) / 2 <= tid) ++pj;
  const int pi = tid - pj * (pj + 1) / 2;
  const bool item = pj < np;
  // its entries (pi, pj), (pi, pj + np), (pi + np, pj) and (pi + np, pj + np), the third kept as
  // the conjugate of (pj, pi + np); where they go, and which go below the diagonal
  const int pic = item ? pi : 0, pjc = item ? pj : 0;
  double2* const r00 = &S.a[pic][pjc];
  double2* const r01 = &S.a[pic][pjc + np];
  double2* const r10 = &S.a[pjc][pic + np];
  double2* const r11 = &S.a[pic + np][pjc + np];
  const int xi = next(pic), yi = next(pic + np), xj = next(pjc), yj = next(pjc + np);
  double2* const w00 = &S.a[min(xi, xj)][max(xi, xj)];
  double2* const w01 = &S.a[min(xi, yj)][max(xi, yj)];
  double2* const w10 = &S.a[min(yi, xj)][max(yi, xj)];
  double2* const w11 = &S.a[min(yi, yj)][max(yi, yj)];
  const double s00 = xi > xj ? -1.0 : 1.0, s01 = xi > yj ? -1.0 : 1.0, s10 = yi > xj ? -1.0 : 1.0,
               s11 = yi > yj ? -1.0 : 1.0;
  // eigenvectors: waves 1 .. 15 take the pairs wv - 1 + 15 u
  constexpr int NZ = (JMAX / 2 + JTHR / 64 - 2) / (JTHR / 64 - 1);
  double2 zx[NZ], zy[NZ];
  auto zturn = [&](int buf) {
#pragma unroll
    for (int u = 0; u < NZ; ++u) {
      const int t = wv - 1 + (JTHR / 64 - 1) * u;
      if (wv > 0 && t < np) {
        const double c = S.rc[buf][t];
        const double2 w = S.rw[buf][t], x = S.zt[t][lane], y = S.zt[t + np][lane];
        zx[u] = csub(cscale(x, c), cmul(cconj(w), y));
        zy[u] = cadd(cmul(w, x), cscale(y, c));
      }
    }
  };
  auto zmove = [&]() {
#pragma unroll
    for (int u = 0; u < NZ; ++u) {
      const int t = wv - 1 + (JTHR / 64 - 1) * u;
      if (wv > 0 && t < np) {
        S.zt[next(t)][lane] = zx[u];
        S.zt[next(t + np)][lane] = zy[u];
      }
    }
  };
  __syncthreads();
  auto sums = [&](double& off, double& tot) {   // squares off the diagonal, and all
    off = tot = 0.0;
    for (int e = tid; e < JMAX * JMAX; e += JTHR) {
      const int i = e >> 6, j = e & 63;
      if (i <= j && j < n) {
        const double2 x = S.a[i][j];
        const double v = x.x * x.x + x.y * x.y;
        tot += i == j ? v : 2.0 * v;
        if (i != j) off += 2.0 * v;
      }
    }
    jacobi_sum2(S, off, tot);
  };
  bool conv = false;
  int up = 0;   // A is held times 2^up where its squares leave the range of the rotations
  for (int sweep = 0; sweep <= JSWEEPS; ++sweep) {
    double off, tot;
    sums(off, tot);
    if (sweep == 0 && !(tot > 1e-200 && tot < 1e200)) {
      double big = 0.0;
      for (int e = tid; e < JMAX * JMAX; e += JTHR) {
        const int i = e >> 6, j = e & 63;
        if (i <= j && j < n) big = fmax(big, fmax(fabs(S.a[i][j].x), fabs(S.a[i][j].y)));
      }
      for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o));
      if (lane == 0) S.red[0][wv] = big;
      __syncthreads();
      for (int w = 0; w < JTHR / 64; ++w) big = fmax(big, S.red[0][w]);
      __syncthreads();
      if (big > 0.0 && big <= 0x1.fffffffffffffp1023) {
        up = -ilogb(big);
        for (int e = tid; e < JMAX * JMAX; e += JTHR) {
          const int i = e >> 6, j = e & 63;
          if (i <= j && j < n) S.a[i][j] = make_double2(ldexp(S.a[i][j].x, up), ldexp(S.a[i][j].y, up));
        }
        __syncthreads();
        sums(off, tot);
      }
    }
    conv = off <= 1e-30 * tot || off == 0.0;
    if (conv || sweep == JSWEEPS) break;
    for (int round = 0; round < N - 1; ++round) {
      const int buf = round & 1;
      if (wv == 0) {
        if (lane < np) {
          double c = 1.0;
          double2 w = make_double2(0.0, 0.0);
          const double2 b = S.a[lane][lane + np];
          const double b2 = b.x * b.x + b.y * b.y;
          const double app = S.a[lane][lane].x, aqq = S.a[lane + np][lane + np].x;
          const double sc = fabs(app) + fabs(aqq);
          if (b2 > 1e-290 && b2 > 1e-36 * sc * sc) {
            const double a = 0.5 * (aqq - app);
            const double ir = rsqrt(fma(a, a, b2));
            const double c2 = fma(0.5 * fabs(a), ir, 0.5);
            const double ic = rsqrt(c2);
            c = c2 * ic;
            const double f = (a >= 0.0 ? 0.5 : -0.5) * ir * ic;
            w = make_double2(f * b.x, f * b.y);
          }
          S.rc[buf][lane] = c;
          S.rw[buf][lane] = w;
        }
      } else if (round > 0) {
        zturn(buf ^ 1);
      }
      __syncthreads();
      if (round > 0) zmove();
      double2 v00, v01, v10, v11;
      if (item) {
        const double ci = S.rc[buf][pi], cj = S.rc[buf][pj];
        const double2 wi = S.rw[buf][pi], wj = S.rw[buf][pj], wjc = cconj(wj), wic = cconj(wi);
        const double2 a00 = *r00, a01 = *r01, a10 = cconj(*r10), a11 = *r11;
        // columns: new_x = c x - conj(w) y, new_y = w x + c y
        const double2 u00 = csub(cscale(a00, cj), cmul(wjc, a01)), u01 = cadd(cmul(wj, a00), cscale(a01, cj));
        const double2 u10 = csub(cscale(a10, cj), cmul(wjc, a11)), u11 = cadd(cmul(wj, a10), cscale(a11, cj));
        // rows: new_p = c p - w q, new_q = conj(w) p + c q
        v00 = csub(cscale(u00, ci), cmul(wi, u10));
        v01 = csub(cscale(u01, ci), cmul(wi, u11));
        v10 = cadd(cmul(wic, u00), cscale(u10, ci));
        v11 = cadd(cmul(wic, u01), cscale(u11, ci));
        if (pi == pj) {
          v00.y = v11.y = 0.0;
          if (wi.x != 0.0 || wi.y != 0.0) v01 = make_double2(0.0, 0.0);
        }
      }
      __syncthreads();
      if (item) {
        *w00 = make_double2(v00.x, s00 * v00.y);
        *w01 = make_double2(v01.x, s01 * v01.y);
        if (pi != pj) *w10 = make_double2(v10.x, s10 * v10.y);
        *w11 = make_double2(v11.x, s11 * v11.y);
      }
      __syncthreads();
    }
    zturn(N & 1);   // the last round, N - 2
    __syncthreads();
    zmove();
    __syncthreads();
  }
  if (up != 0) {
    if (tid < n) S.a[tid][tid].x = ldexp(S.a[tid][tid].x, -up);
    __syncthreads();
  }
  if (tid == 0) S.done = conv ? 1 : 0;
  if (tid < n) {   // rank of each eigenvalue
    const double v = S.a[tid][tid].x;
    int rank = 0;
    for (int j = 0; j < n; ++j) rank += eig_before(S.a[j][j].x, j, v, tid) ? 1 : 0;
    S.perm[rank] = tid;
  }
  __syncthreads();
}

}  // namespace adc2
