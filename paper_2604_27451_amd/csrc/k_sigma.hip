// k_sigma.hip -- sigma = M x for the CVS-ADC(2) matrix (paper Eq. 11-12,
// CVS section), FP64 complex on the FP64 MFMA.
//
// With r = [r1 (I,a) | r2 (I,j,a<b)] and the doubles state a+_a a+_b a_j a_I:
//   M21[(Ijab),(Kc)] = d_IK <ab||cj> - d_ac <Kb||Ij> + d_bc <Ka||Ij>
//   M22 = diag(e_a + e_b - e_I - e_j),  M12 = M21^H.
// The three-virtual integral <ab||cj> = (ac|bj) - (aj|bc) is never formed:
//   X^P_{Ia}  = sum_c L^P_{ac} r_{Ic}                                  (X-build)
//   Z_{Ij}[a][b] = sum_P X^P_{Ia} L^P_{bj}                             (sigma2 GEMM)
//   s2_{Ijab} = Z_ab - Z_ba + sum_K (<Ka||Ij> r_Kb - r_Ka <Kb||Ij>) + D r2 (pack)
//   Y^P_{Ic}  = sum_{jd} conj(L^P_{dj}) r_{Ijcd}                          (Y GEMM)
//   s1_{Ia}   = sum_{Jb} M11 r1 + sum_{Pc} L^P_{ac} Y^P_{Ic}
//             - sum_{I',jb} conj(<Ib||I'j>) r_{I'jab}                    (sigma1)
// The two heavy contractions (8 nc no nv^2 naux flops per vector each) are
// plain complex GEMMs on 128x128 tiles (zgemm.h) with no redundant work; the
// antisymmetrisation, the denominators and the light core terms run in
// bandwidth-bound kernels around them.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <vector>

#include <mutex>

#include "internal.h"
#include "rns.h"
#include "tile.h"
#include "zgemm.h"
#include "zgemm32.h"
#include "zgemmb.h"

namespace adc2 {

__host__ __device__ static inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }
static inline unsigned grid_for(long n, long per = 256, long cap = 16384) {
  long g = (n + per - 1) / per;
  return (unsigned)std::max<long>(1, std::min<long>(g, cap));
}

// storage conversions of the precision form (complex64 operands, FP64 arithmetic around them)
__device__ __forceinline__ double2 to_d2(double2 v) { return v; }
__device__ __forceinline__ double2 to_d2(float2 v) { return make_double2((double)v.x, (double)v.y); }
template <class T> __device__ __forceinline__ T from_d2(double2 v);
template <> __device__ __forceinline__ double2 from_d2<double2>(double2 v) { return v; }
template <> __device__ __forceinline__ float2 from_d2<float2>(double2 v) { return make_float2((float)v.x, (float)v.y); }

// ---------------------------------------------------------------------------
// generic  C[i][j] = alpha * sum_k A[i][k] B^T[j][k]  (both k-contiguous)
// ---------------------------------------------------------------------------
template <bool CA, bool CB>
__global__ __launch_bounds__(256) void k_gemm_rr(int M, int N, int K, const double2* __restrict__ A, long lda,
                                                  const double2* __restrict__ B, long ldb,
                                                  double2* __restrict__ C, long ldc, double alpha, int accumulate) {
  __shared__ TileSmem s;
  const int nbj = cdiv(N, TN);
  const int i0 = (blockIdx.x / nbj) * TM, j0 = (blockIdx.x % nbj) * TN;
  SrcR<CA> sa{A + (long)i0 * lda, lda, K, M - i0, 1.0};
  SrcR<CB> sb{B + (long)j0 * ldb, ldb, K, N - j0, 1.0};
  Acc acc;
  acc.zero();
  mainloop(s, sa, sb, 0, cdiv(K, TK), acc);
  for_each_acc(acc, [&](int r, int c, double2 v) {
    const int i = i0 + r, j = j0 + c;
    if (i < M && j < N) {
      double2* p = C + (long)i * ldc + j;
      v = cscale(v, alpha);
      *p = accumulate ? cadd(*p, v) : v;
    }
  });
}

adc2_status gemm_rr(int M, int N, int K, const double2* A, long lda, bool conjA, const double2* B, long ldb,
                    bool conjB, double2* C, long ldc, double alpha, bool accumulate, hipStream_t st) {
  if (M <= 0 || N <= 0) return ADC2_OK;
  const int nblk = cdiv(M, TM) * cdiv(N, TN);
  if (!conjA && !conjB)
    k_gemm_rr<false, false><<<nblk, 256, 0, st>>>(M, N, K, A, lda, B, ldb, C, ldc, alpha, accumulate);
  else if (conjA && !conjB)
    k_gemm_rr<true, false><<<nblk, 256, 0, st>>>(M, N, K, A, lda, B, ldb, C, ldc, alpha, accumulate);
  else if (!conjA && conjB)
    k_gemm_rr<false, true><<<nblk, 256, 0, st>>>(M, N, K, A, lda, B, ldb, C, ldc, alpha, accumulate);
  else
    k_gemm_rr<true, true><<<nblk, 256, 0, st>>>(M, N, K, A, lda, B, ldb, C, ldc, alpha, accumulate);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// ---------------------------------------------------------------------------
// X-build:  X[mI][(P,a)] = sum_c r1[m][I][c] Lvv[P][a][c]
// ---------------------------------------------------------------------------
struct SrcR1Rows {   // element (k=c, i=mI) = r1 of vector m, core I
  static constexpr int MAP = RMAJOR;
  const double2* x;
  long dim;
  int nc, nv, nrows, i0;
  __device__ __forceinline__ double2 get(int k, int i) const {
    const int mi = i0 + i;
    if (k >= nv || mi >= nrows) return czero();
    const int m = mi / nc, I = mi - m * nc;
    return x[(long)m * dim + (long)I * nv + k];
  }
};

template <class TO, int MR>
__global__ __launch_bounds__(256) void k_xbuild(const double2* __restrict__ x, long dim, int nc, int nv, int naux,
                                                 int nrows, const double2* __restrict__ Lvv,
                                                 TO* __restrict__ X) {
  __shared__ TileSmem s;
  const long ncol = (long)naux * nv;
  const int nbj = cdiv(ncol, TN);
  const long nblocks = (long)cdiv(nrows, MR) * nbj;
  const long lid = xcd_remap(blockIdx.x, nblocks);
  const int i0 = (int)(lid / nbj) * MR;
  const long j0 = (lid % nbj) * TN;
  SrcR1Rows sa{x, dim, nc, nv, nrows, i0};
  SrcR<false> sb{Lvv + j0 * nv, nv, nv, (int)min((long)TN, ncol - j0), 1.0};
  AccT<MR> acc;
  acc.zero();
  mainloop(s, sa, sb, 0, cdiv(nv, TK), acc);
  for_each_acc(acc, [&](int r, int c, double2 v) {
    const int mi = i0 + r;
    const long j = j0 + c;
    if (mi < nrows && j < ncol) X[(long)mi * ncol + j] = from_d2<TO>(v);
  });
}

// ---------------------------------------------------------------------------
// X-build and back-contraction of at most 16 rows (mI)
// ---------------------------------------------------------------------------
// Both read Lvv once and are bound by that where rows are few; tiles of 64
// rows do the matrix work of 64 rows whatever their number (nc=6 no=120 nv=600
// naux=3000, two vectors: 8.9 and 9.0 ms; of 32 rows 5.0 and 5.6).  Here a wave
// multiplies 16 rows with 64 columns of Lvv on the 16x16x4 FP64 MFMA (4.0 ms
// each), operands straight from global memory: a lane's element of a column tile
// is Lvv[column][k] with four k of a column in one 64-byte piece and four steps
// of k unrolled, so whole lines are used; the row operand stays in cache.
//
// acc[c] += A(rows, k) B(k, columns 16 c + ..) over k < K; a(k) and b(c, k) give
// this lane's elements, zero past the ends.
template <class FA, class FB>
__device__ __forceinline__ void thin_mma(int K, d4 (&re)[4], d4 (&im)[4], FA&& fa, FB&& fb) {
  const int lk = (threadIdx.x & 63) >> 4;
  for (int k0 = 0; k0 < K; k0 += 16) {
    double2 a[4], b[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = fa(k0 + 4 * u + lk);
#pragma unroll
      for (int c = 0; c < 4; ++c) b[u][c] = fb(c, k0 + 4 * u + lk);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        re[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, b[u][c].x, re[c], 0, 0, 0);
        re[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[u].y, b[u][c].y, re[c], 0, 0, 0);
        im[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, b[u][c].y, im[c], 0, 0, 0);
        im[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].y, b[u][c].x, im[c], 0, 0, 0);
      }
  }
}

// Where the thin kernels are the faster ones: up to 16 rows of an Lvv of at least 2^23
// entries (few workgroups below: nc=6 no=10 nv=40 naux=150, one vector, 14 and 16 us
// against 7 and 8 on 32-row tiles).
static bool thin_rows(const Dims& d, int rows) {
  return rows <= 16 && (double)d.naux * d.nv * d.nv >= 8388608.0;
}

// Rows of the LDS tiles, 32, 48 or 64: those that pad the rows least, the larger on a
// tie (no=12 nv=100, 24 rows: 24 and 30 us on 32-row tiles, 37 and 46 on 64-row ones;
// no=25 nv=380, 30 rows: 1.00 and 1.04 ms, two thin tiles of 16 rows 1.22 and 1.46;
// no=45 nv=310, 42 rows: 1.09 and 0.97 ms on 48-row tiles, 1.23 and 1.12 on 64).
static int row_tile(int rows) {
  int best = 64;
  for (int t : {48, 32})
    if (cdiv(rows, t) * t < cdiv(rows, best) * best) best = t;
  return best;
}

template <class TO>
__global__ __launch_bounds__(256) void k_xbuild_thin(const double2* __restrict__ x, long dim, int nc, int nv, int naux,
                                                     int nrows, const double2* __restrict__ Lvv, TO* __restrict__ X) {
  const int lane = threadIdx.x & 63, li = lane & 15;
  const long ncol = (long)naux * nv;
  const long j0 = (xcd_remap(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6)) * 64;
  if (j0 >= ncol) return;
  const bool oka = li < nrows;
  const int mm = oka ? li : 0, m = mm / nc;
  const double2* pa = x + (long)m * dim + (long)(mm - m * nc) * nv;
  const double2* pb[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) pb[c] = Lvv + min(j0 + 16 * c + li, ncol - 1) * nv;   // past the end: never stored
  d4 re[4], im[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) re[c] = im[c] = d4{0.0, 0.0, 0.0, 0.0};
  thin_mma(
      nv, re, im, [&](int k) { return oka && k < nv ? pa[k] : czero(); },
      [&](int c, int k) { return k < nv ? pb[c][k] : czero(); });
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int mi = (lane >> 4) + 4 * r;
      const long j = j0 + 16 * c + li;
      if (mi < nrows && j < ncol) X[(long)mi * ncol + j] = from_d2<TO>(make_double2(re[c][r], im[c][r]));
    }
}

// part[split][mI][a] = sum_{P in split} sum_c Y[mI][P][c] Lvv[P][a][c]: a workgroup
// owns a split and 64 values of a, its waves share the split's P.
__global__ __launch_bounds__(256) void k_backc_thin(const double2* __restrict__ Y, const double2* __restrict__ Lvv,
                                                    int nrows, int nv, int naux, int nsplit, double2* __restrict__ part) {
  __shared__ double2 red[3][64][17];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15;
  const int nba = (nv + 63) / 64;
  const int split = blockIdx.x / nba, a0 = (blockIdx.x % nba) * 64;
  const int per = (naux + nsplit - 1) / nsplit;
  const int P0 = split * per, P1 = min(naux, P0 + per);
  const bool oka = li < nrows;
  d4 re[4], im[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) re[c] = im[c] = d4{0.0, 0.0, 0.0, 0.0};
  for (int P = P0 + w; P < P1; P += 4) {
    const double2* pb[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) pb[c] = Lvv + ((long)P * nv + min(a0 + 16 * c + li, nv - 1)) * nv;
    const double2* pa = Y + ((long)(oka ? li : 0) * naux + P) * nv;
    thin_mma(
        nv, re, im, [&](int k) { return oka && k < nv ? pa[k] : czero(); },
        [&](int c, int k) { return k < nv ? pb[c][k] : czero(); });
  }
  double2* out = part + (long)split * nrows * nv;
  if (w > 0)   // the four waves' sums, in order
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[w - 1][lane][4 * c + r] = make_double2(re[c][r], im[c][r]);
  __syncthreads();
  if (w > 0) return;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double2 v = make_double2(re[c][r], im[c][r]);
#pragma unroll
      for (int q = 0; q < 3; ++q) v = cadd(v, red[q][lane][4 * c + r]);
      const int mi = (lane >> 4) + 4 * r, a = a0 + 16 * c + li;
      if (mi < nrows && a < nv) out[(long)mi * nv + a] = v;
    }
}

template <class TO>
static adc2_status xbuild_launch(const double2* x, const Dims& d, int rows, const double2* Lvv, TO* X, hipStream_t st) {
  if (thin_rows(d, rows)) {
    const unsigned nblk = (unsigned)cdiv((long)d.naux * d.nv, 256);
    k_xbuild_thin<TO><<<nblk, 256, 0, st>>>(x, d.dim, d.nc, d.nv, d.naux, rows, Lvv, X);
  } else {
    const int mr = row_tile(rows);
    const unsigned nblk = (unsigned)((long)cdiv(rows, mr) * cdiv((long)d.naux * d.nv, TN));
    if (mr == 32) k_xbuild<TO, 32><<<nblk, 256, 0, st>>>(x, d.dim, d.nc, d.nv, d.naux, rows, Lvv, X);
    else if (mr == 48) k_xbuild<TO, 48><<<nblk, 256, 0, st>>>(x, d.dim, d.nc, d.nv, d.naux, rows, Lvv, X);
    else k_xbuild<TO, 64><<<nblk, 256, 0, st>>>(x, d.dim, d.nc, d.nv, d.naux, rows, Lvv, X);
  }
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// Y-build A: element (k = (j, d), i = P) = conj(L^P_{d j}) = conj(Lvo[nc+j][P][d]);
// k runs over j-blocks of cpe chunks (d padded to a multiple of BK).
template <int NS>
struct SrcLconjRows {
  static constexpr int MAP = RMAJOR;
  const double2* base;   // Lvo + nc*naux*nv
  long jstride;          // naux*nv
  int nv, cpe, nrows;
  long off[NS];
  unsigned okmask;
  int kk;
  __device__ __forceinline__ void begin(int tid, int i0) {
    kk = tid & 15;
    okmask = 0;
#pragma unroll
    for (int e = 0; e < NS; ++e) {
      const int P = i0 + (tid >> 4) + 16 * e;
      off[e] = (long)P * nv;
      if (P < nrows) okmask |= 1u << e;
    }
  }
  __device__ __forceinline__ void load(int kc, RegsN<NS>& r) const {
    const int j = kc / cpe;
    const int d = (kc - j * cpe) * BK + kk;
    const long jo = (long)j * jstride + d;
    const bool dok = d < nv;
#pragma unroll
    for (int e = 0; e < NS; ++e) {
      if (((okmask >> e) & 1u) && dok) {
        const double2 v = base[off[e] + jo];
        r.v[e] = make_double2(v.x, -v.y);
      } else {
        r.v[e] = czero();
      }
    }
  }
};

// Y-build B: element (k = (j, d), col = (mI, c)) = R_{mI j}[c][d] from the
// unpacked antisymmetric doubles Rf[mI][j][c][d].
template <int NS>
struct SrcRfull {
  static constexpr int MAP = RMAJOR;
  const double2* R;
  int nv, no, cpe, ncols;
  long off[NS];
  unsigned okmask;
  int kk;
  __device__ __forceinline__ void begin(int tid, int i0) {
    kk = tid & 15;
    okmask = 0;
#pragma unroll
    for (int e = 0; e < NS; ++e) {
      const int col = i0 + (tid >> 4) + 16 * e;
      const int g = col / nv, c = col - g * nv;
      off[e] = ((long)g * no * nv + c) * nv;
      if (col < ncols) okmask |= 1u << e;
    }
  }
  __device__ __forceinline__ void load(int kc, RegsN<NS>& r) const {
    const int j = kc / cpe;
    const int d = (kc - j * cpe) * BK + kk;
    const long jo = (long)j * nv * nv + d;
    const bool dok = d < nv;
#pragma unroll
    for (int e = 0; e < NS; ++e) r.v[e] = (((okmask >> e) & 1u) && dok) ? R[off[e] + jo] : czero();
  }
};

// sigma2 core:  Z[mI][j][a][b] = sum_P X[mI][P][a] Lvo[nc+j][P][b]
// G3: three-multiplication 128x64 tiles; otherwise four-multiplication 128x128.
template <bool G3>
__global__ __launch_bounds__(256) void k_zsig2(const double2* __restrict__ X, const double2* __restrict__ Lvo,
                                                int rows, int nc, int no, int nv, int naux,
                                                double2* __restrict__ Z) {
  constexpr int TNC = G3 ? BT3N : BT;
  constexpr int NSB = G3 ? 4 : 8;
  const int ncols = no * nv;
  const int nbm = (rows + BT - 1) / BT, nbn = (ncols + TNC - 1) / TNC;
  const long lid = xcd_remap(blockIdx.x, (long)nbm * nbn);
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * TNC;
  const long lds = (long)naux * nv;
  SrcGroupedK<8> A{X, lds, nv, nv, rows, naux};
  SrcGroupedK<NSB> B{Lvo + (long)nc * lds, lds, nv, nv, ncols, naux};
  A.begin(threadIdx.x, i0);
  B.begin(threadIdx.x, j0);
  auto store = [&](int r, int c, double2 v) {
    const int i = i0 + r, jc = j0 + c;
    if (i < rows && jc < ncols) {
      const int mI = i / nv, a = i - mI * nv;
      const int j = jc / nv, b = jc - j * nv;
      Z[(((long)mI * no + j) * nv + a) * nv + b] = v;
    }
  };
  const int nkc = (naux + BK - 1) / BK;
  if constexpr (G3) {
    __shared__ BigSmem3 s;
    BigAcc3 acc;
    acc.zero();
    big_mainloop3(s, A, B, 0, nkc, acc);
    big_for_each3(acc, store);
  } else {
    __shared__ BigSmem s[2];
    BigAcc acc;
    acc.zero();
    big_mainloop(s, A, B, 0, nkc, acc);
    big_for_each(acc, store);
  }
}

// Y-build:  Y[mI][P][c] = sum_{(j,d)} LvT[(j,d)][P] Rt[(j,d)][(mI,c)]
//                      = sum_{j,d} conj(L^P_{dj}) R_{mIj}[c][d]
// Both operands are k-major rows (contiguous in P and in (mI,c)).
template <bool G3>
__global__ __launch_bounds__(256) void k_ygemm(const double2* __restrict__ LvT, const double2* __restrict__ Rt,
                                                int rows, int nc, int no, int nv, int naux,
                                                double2* __restrict__ Y) {
  constexpr int TNC = G3 ? BT3N : BT;
  constexpr int NSB = G3 ? 4 : 8;
  const int ncols = rows * nv;
  const int nbm = (naux + BT - 1) / BT, nbn = (ncols + TNC - 1) / TNC;
  const long lid = xcd_remap(blockIdx.x, (long)nbm * nbn);
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * TNC;
  const int K = no * nv;
  SrcGroupedK<8> A{LvT, 0, naux, naux, naux, K};
  SrcGroupedK<NSB> B{Rt, 0, ncols, ncols, ncols, K};
  A.begin(threadIdx.x, i0);
  B.begin(threadIdx.x, j0);
  // split over K: blockIdx.y of gridDim.y writes its own partial of Y
  const int nchunks = (K + BK - 1) / BK;
  const int per = (nchunks + gridDim.y - 1) / gridDim.y;
  const int kc0 = blockIdx.y * per, kc1 = min(nchunks, kc0 + per);
  double2* Ys = Y + (long)blockIdx.y * ((long)rows * naux * nv);
  auto store = [&](int r, int c, double2 v) {
    const int P = i0 + r, col = j0 + c;
    if (P < naux && col < ncols) {
      const int mI = col / nv, cc = col - mI * nv;
      Ys[((long)mI * naux + P) * nv + cc] = v;
    }
  };
  if constexpr (G3) {
    __shared__ BigSmem3 s;
    BigAcc3 acc;
    acc.zero();
    big_mainloop3(s, A, B, kc0, kc1, acc);
    big_for_each3(acc, store);
  } else {
    __shared__ BigSmem s[2];
    BigAcc acc;
    acc.zero();
    big_mainloop(s, A, B, kc0, kc1, acc);
    big_for_each(acc, store);
  }
}

// The same two contractions on the two-per-CU engine (128 x 64 tiles, chunks
// of 8 k).  The Y-build's K-splits are cut at the 16-k boundaries of the
// 128 x 128 kernel, so both kernels sum every partial in the same order.
__global__ __launch_bounds__(256, 2) void k_zsig2_mid(const double2* __restrict__ X,
                                                       const double2* __restrict__ Lvo, int rows, int nc, int no,
                                                       int nv, int naux, double2* __restrict__ Z) {
  __shared__ MidSmem s[2];
  const int ncols = no * nv;
  const int nbm = (rows + BT - 1) / BT, nbn = (ncols + MTN - 1) / MTN;
  const long lid = xcd_remap(blockIdx.x, (long)nbm * nbn);
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * MTN;
  const long lds = (long)naux * nv;
  SrcGroupedK8<4> A{X, lds, nv, nv, rows, naux};
  SrcGroupedK8<2> B{Lvo + (long)nc * lds, lds, nv, nv, ncols, naux};
  A.begin(threadIdx.x, i0);
  B.begin(threadIdx.x, j0);
  MidAcc acc;
  acc.zero();
  mid_mainloop(s, A, B, 0, (naux + MBK - 1) / MBK, acc);
  mid_for_each(acc, [&](int r, int c, double2 v) {
    const int i = i0 + r, jc = j0 + c;
    if (i < rows && jc < ncols) {
      const int mI = i / nv, a = i - mI * nv;
      const int j = jc / nv, b = jc - j * nv;
      Z[(((long)mI * no + j) * nv + a) * nv + b] = v;
    }
  });
}

__global__ __launch_bounds__(256, 2) void k_ygemm_mid(const double2* __restrict__ LvT,
                                                       const double2* __restrict__ Rt, int rows, int no, int nv,
                                                       int naux, double2* __restrict__ Y) {
  __shared__ MidSmem s[2];
  const int ncols = rows * nv;
  const int nbm = (naux + BT - 1) / BT, nbn = (ncols + MTN - 1) / MTN;
  const long lid = xcd_remap(blockIdx.x, (long)nbm * nbn);
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * MTN;
  const int K = no * nv;
  SrcGroupedK8<4> A{LvT, 0, naux, naux, naux, K};
  SrcGroupedK8<2> B{Rt, 0, ncols, ncols, ncols, K};
  A.begin(threadIdx.x, i0);
  B.begin(threadIdx.x, j0);
  const int n16 = (K + BK - 1) / BK;
  const int per = (n16 + gridDim.y - 1) / gridDim.y;   // in 16-k chunks
  const int kc0 = 2 * blockIdx.y * per, kc1 = min((K + MBK - 1) / MBK, kc0 + 2 * per);
  double2* Ys = Y + (long)blockIdx.y * ((long)rows * naux * nv);
  MidAcc acc;
  acc.zero();
  mid_mainloop(s, A, B, kc0, kc1, acc);
  mid_for_each(acc, [&](int r, int c, double2 v) {
    const int P = i0 + r, col = j0 + c;
    if (P < naux && col < ncols) {
      const int mI = col / nv, cc = col - mI * nv;
      Ys[((long)mI * naux + P) * nv + cc] = v;
    }
  });
}

// The same two contractions on the eight-wave engine (128 x 128 tiles, 16-k
// chunks, two waves per SIMD).
__global__ __launch_bounds__(512) void k_zsig2_wide(const double2* __restrict__ X, const double2* __restrict__ Lvo,
                                                     int rows, int nc, int no, int nv, int naux,
                                                     double2* __restrict__ Z) {
  __shared__ BigSmem s[2];
  const int ncols = no * nv;
  const int nbm = (rows + BT - 1) / BT, nbn = (ncols + BT - 1) / BT;
  const long lid = xcd_remap(blockIdx.x, (long)nbm * nbn);
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * BT;
  const long lds = (long)naux * nv;
  SrcGroupedK8<4, BK> A{X, lds, nv, nv, rows, naux};
  SrcGroupedK8<4, BK> B{Lvo + (long)nc * lds, lds, nv, nv, ncols, naux};
  A.begin(threadIdx.x, i0);
  B.begin(threadIdx.x, j0);
  MidAcc acc;
  acc.zero();
  wide_mainloop(s, A, B, 0, (naux + BK - 1) / BK, acc);
  wide_for_each(acc, [&](int r, int c, double2 v) {
    const int i = i0 + r, jc = j0 + c;
    if (i < rows && jc < ncols) {
      const int mI = i / nv, a = i - mI * nv;
      const int j = jc / nv, b = jc - j * nv;
      Z[(((long)mI * no + j) * nv + a) * nv + b] = v;
    }
  });
}

__global__ __launch_bounds__(512) void k_ygemm_wide(const double2* __restrict__ LvT, const double2* __restrict__ Rt,
                                                     int rows, int no, int nv, int naux, double2* __restrict__ Y) {
  __shared__ BigSmem s[2];
  const int ncols = rows * nv;
  const int nbm = (naux + BT - 1) / BT, nbn = (ncols + BT - 1) / BT;
  const long lid = xcd_remap(blockIdx.x, (long)nbm * nbn);
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * BT;
  const int K = no * nv;
  SrcGroupedK8<4, BK> A{LvT, 0, naux, naux, naux, K};
  SrcGroupedK8<4, BK> B{Rt, 0, ncols, ncols, ncols, K};
  A.begin(threadIdx.x, i0);
  B.begin(threadIdx.x, j0);
  const int nchunks = (K + BK - 1) / BK;
  const int per = (nchunks + gridDim.y - 1) / gridDim.y;
  const int kc0 = blockIdx.y * per, kc1 = min(nchunks, kc0 + per);
  double2* Ys = Y + (long)blockIdx.y * ((long)rows * naux * nv);
  MidAcc acc;
  acc.zero();
  wide_mainloop(s, A, B, kc0, kc1, acc);
  wide_for_each(acc, [&](int r, int c, double2 v) {
    const int P = i0 + r, col = j0 + c;
    if (P < naux && col < ncols) {
      const int mI = col / nv, cc = col - mI * nv;
      Ys[((long)mI * naux + P) * nv + cc] = v;
    }
  });
}

// Precision form: the two heavy contractions on complex64 operands with the
// FP32 MFMA and FP32 accumulation.  Each kernel body is an "item" (one output
// tile and one K-split) so that the plain launches below and the grouped
// launches of several systems (GemmJobs) share it.
//   sigma2: Z[mI][j][a][b] = sum_P X^P_{(mI)a} L^P_{bj}      (rows = m*nc*nv)
//   Y-build: Y[s][mI][P][c] = sum_{(j,d) in split s} conj(L^P_dj) Rt[(j,d)][(mI,c)]
__device__ __forceinline__ void zsig2_c64_item(BigSmemF (&s)[2], const float2* __restrict__ X32,
                                               const float2* __restrict__ Lv32, int rows, int no, int nv, int naux,
                                               float2* __restrict__ Z, long lid) {
  const int ncols = no * nv;
  const int nbm = (rows + BT - 1) / BT, nbn = (ncols + BT - 1) / BT;
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * BT;
  const long lds = (long)naux * nv;
  SrcGroupedKF A{X32, lds, nv, nv, rows, naux};
  SrcGroupedKF B{Lv32, lds, nv, nv, ncols, naux};
  A.begin(threadIdx.x, i0);
  B.begin(threadIdx.x, j0);
  BigAccF acc;
  acc.zero();
  big_mainloopF(s, A, B, 0, (naux + BK - 1) / BK, acc);
  big_for_eachF(acc, [&](int r, int c, float2 v) {
    const int i = i0 + r, jc = j0 + c;
    if (i < rows && jc < ncols) {
      const int mI = i / nv, a = i - mI * nv;
      const int j = jc / nv, b = jc - j * nv;
      Z[(((long)mI * no + j) * nv + a) * nv + b] = v;
    }
  });
}

__device__ __forceinline__ void ygemm_c64_item(BigSmemF (&s)[2], const float2* __restrict__ LvT32,
                                               const float2* __restrict__ Rt32, int rows, int no, int nv, int naux,
                                               double2* __restrict__ Y, long lid, int split, int nsplit) {
  const int ncols = rows * nv;
  const int nbm = (naux + BT - 1) / BT, nbn = (ncols + BT - 1) / BT;
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * BT;
  const int K = no * nv;
  SrcGroupedKF A{LvT32, 0, naux, naux, naux, K};
  SrcGroupedKF B{Rt32, 0, ncols, ncols, ncols, K};
  A.begin(threadIdx.x, i0);
  B.begin(threadIdx.x, j0);
  const int nchunks = (K + BK - 1) / BK;
  const int per = (nchunks + nsplit - 1) / nsplit;
  const int kc0 = split * per, kc1 = min(nchunks, kc0 + per);
  double2* Ys = Y + (long)split * ((long)rows * naux * nv);
  BigAccF acc;
  acc.zero();
  big_mainloopF(s, A, B, kc0, kc1, acc);
  big_for_eachF(acc, [&](int r, int c, float2 v) {
    const int P = i0 + r, col = j0 + c;
    if (P < naux && col < ncols) {
      const int mI = col / nv, cc = col - mI * nv;
      Ys[((long)mI * naux + P) * nv + cc] = make_double2((double)v.x, (double)v.y);
    }
  });
}

// Precision form, split-BF16 variant: the same two contractions on the BF16
// matrix cores with hi/lo operands in the blocked split layout (zgemmb.h),
// FP32 accumulation, 512-thread workgroups (consumer waves 0-3 write the
// tile).  XB, LvB: sigma2 operands (rows (mI,a) and (j,b), K = naux); LvTB, RB:
// Y-build operands (rows P and (mI,c), K = (j,d)).
__device__ __forceinline__ void zsig2_b3_item(BigSmemB (&s)[2], const __bf16* __restrict__ XB,
                                              const __bf16* __restrict__ LvB, int rows, int no, int nv, int naux,
                                              float2* __restrict__ Z, long lid) {
  const int ncols = no * nv;
  const int nbm = (rows + BT - 1) / BT, nbn = (ncols + BT - 1) / BT;
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * BT;
  const int nkc = (naux + BKB - 1) / BKB;
  SrcBL A{(const char*)XB, nkc};
  SrcBL B{(const char*)LvB, nkc};
  A.begin(threadIdx.x & 255, i0);
  B.begin(threadIdx.x & 255, j0);
  BigAccF acc;
  acc.zero();
  big_mainloopB(s, A, B, 0, nkc, acc);
  if (wave_id() >= 4) return;
  big_for_eachF(acc, [&](int r, int c, float2 v) {
    const int i = i0 + r, jc = j0 + c;
    if (i < rows && jc < ncols) {
      const int mI = i / nv, a = i - mI * nv;
      const int j = jc / nv, b = jc - j * nv;
      Z[(((long)mI * no + j) * nv + a) * nv + b] = v;
    }
  });
}

__device__ __forceinline__ void ygemm_b3_item(BigSmemB (&s)[2], const __bf16* __restrict__ LvTB,
                                              const __bf16* __restrict__ RB, int rows, int no, int nv, int naux,
                                              double2* __restrict__ Y, long lid, int split, int nsplit) {
  const int ncols = rows * nv;
  const int nbm = (naux + BT - 1) / BT, nbn = (ncols + BT - 1) / BT;
  int bm, bn;
  big_tile_coords(lid, nbm, nbn, bm, bn);
  const int i0 = bm * BT, j0 = bn * BT;
  const int nchunks = (no * nv + BKB - 1) / BKB;
  SrcBL A{(const char*)LvTB, nchunks};
  SrcBL B{(const char*)RB, nchunks};
  A.begin(threadIdx.x & 255, i0);
  B.begin(threadIdx.x & 255, j0);
  const int per = (nchunks + nsplit - 1) / nsplit;
  const int kc0 = split * per, kc1 = min(nchunks, kc0 + per);
  double2* Ys = Y + (long)split * ((long)rows * naux * nv);
  BigAccF acc;
  acc.zero();
  big_mainloopB(s, A, B, kc0, kc1, acc);
  if (wave_id() >= 4) return;
  big_for_eachF(acc, [&](int r, int c, float2 v) {
    const int P = i0 + r, col = j0 + c;
    if (P < naux && col < ncols) {
      const int mI = col / nv, cc = col - mI * nv;
      Ys[((long)mI * naux + P) * nv + cc] = make_double2((double)v.x, (double)v.y);
    }
  });
}

// Split a K-major complex operand (element (k, row) at src[g*gstride +
// x*xstride + k*ld], row = g*inner + x < R, k < K; complex64, or complex128
// rounded to complex64 first) into the blocked split layout of zgemmb.h (rows
// padded to 128, k to 32, padding zero).  Thread t of a block's 512 owns row
// r = (t / 4) % 128 and the k-group stored in 16-byte slot t % 4 of that row,
// so every plane store of a wave covers 16 whole 64-byte rows (1 KB
// contiguous); with xstride 1 the source reads of a wave are 4 runs of 16 rows.
template <class TS>
__global__ void k_split_pack(const TS* __restrict__ src, long gstride, long xstride, long ld, int inner, int R,
                             int K, int nrt, int nkc, __bf16* __restrict__ dst) {
  const long total = (long)nrt * nkc * 512;
  for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < total; t += (long)gridDim.x * blockDim.x) {
    const int slot = (int)(t & 3), r = (int)((t >> 2) & 127);
    const long blk = t >> 9;
    const int kc = (int)(blk % nkc), rt = (int)(blk / nkc);
    const int row = rt * BT + r;
    const int k0 = kc * BKB + 8 * (slot ^ ((r >> 1) & 3));
    float re[8], im[8];
    if (row < R) {
      const int g = row / inner;
      const TS* p = src + (long)g * gstride + (long)(row - g * inner) * xstride;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float2 v = make_float2(0.f, 0.f);
        if (k0 + e < K) {
          const TS w = p[(long)(k0 + e) * ld];
          v = make_float2((float)w.x, (float)w.y);
        }
        re[e] = v.x;
        im[e] = v.y;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) re[e] = im[e] = 0.f;
    }
    bf8 rh, rl, ih, il;
    split8(re, rh, rl);
    split8(im, ih, il);
    const long o0 = split_block_offset(row, k0, 0, nkc);   // = plane-0 base of the block + r*32 + 8*slot
    const long ps = (long)BT * BLDB;                      // plane stride
    *(bf8*)(dst + o0) = rh;
    *(bf8*)(dst + o0 + ps) = rl;
    *(bf8*)(dst + o0 + 2 * ps) = ih;
    *(bf8*)(dst + o0 + 3 * ps) = il;
  }
}

long split_bytes(long R, long K) { return (long)cdiv(R, BT) * cdiv(K, BKB) * BLOCK_BYTES; }

template <class TS>
static adc2_status split_pack(const TS* src, long gstride, long ld, int inner, long R, long K, __bf16* dst,
                              hipStream_t st, long xstride = 1) {
  const int nrt = cdiv(R, BT), nkc = cdiv(K, BKB);
  const long total = (long)nrt * nkc * 512;
  k_split_pack<TS><<<grid_for(total, 256, 1L << 20), 256, 0, st>>>(src, gstride, xstride, ld, inner, (int)R, (int)K,
                                                                    nrt, nkc, dst);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

__global__ __launch_bounds__(256) void k_zsig2_c64(const float2* __restrict__ X32, const float2* __restrict__ Lv32,
                                                    int rows, int no, int nv, int naux, float2* __restrict__ Z) {
  __shared__ BigSmemF s[2];
  const long nt = (long)((rows + BT - 1) / BT) * ((no * nv + BT - 1) / BT);
  zsig2_c64_item(s, X32, Lv32, rows, no, nv, naux, Z, xcd_remap(blockIdx.x, nt));
}

// Two workgroups per CU: the accumulators then live in the unified register
// file (no AGPR split) within 256 registers per lane.
__global__ __launch_bounds__(256, 2) void k_ygemm_c64(const float2* __restrict__ LvT32, const float2* __restrict__ Rt32,
                                                    int rows, int no, int nv, int naux, double2* __restrict__ Y) {
  __shared__ BigSmemF s[2];
  const long nt = (long)((naux + BT - 1) / BT) * ((rows * nv + BT - 1) / BT);
  ygemm_c64_item(s, LvT32, Rt32, rows, no, nv, naux, Y, xcd_remap(blockIdx.x, nt), blockIdx.y, gridDim.y);
}

__global__ __launch_bounds__(512) void k_zsig2_b3(const __bf16* __restrict__ XB, const __bf16* __restrict__ LvB,
                                                   int rows, int no, int nv, int naux, float2* __restrict__ Z) {
  __shared__ BigSmemB s[2];
  const long nt = (long)((rows + BT - 1) / BT) * ((no * nv + BT - 1) / BT);
  zsig2_b3_item(s, XB, LvB, rows, no, nv, naux, Z, xcd_remap(blockIdx.x, nt));
}

__global__ __launch_bounds__(512) void k_ygemm_b3(const __bf16* __restrict__ LvTB, const __bf16* __restrict__ RB,
                                                   int rows, int no, int nv, int naux, double2* __restrict__ Y) {
  __shared__ BigSmemB s[2];
  const long nt = (long)((naux + BT - 1) / BT) * ((rows * nv + BT - 1) / BT);
  ygemm_b3_item(s, LvTB, RB, rows, no, nv, naux, Y, xcd_remap(blockIdx.x, nt), blockIdx.y, gridDim.y);
}

// ---------------------------------------------------------------------------
// Grouped launches of the heavy GEMMs over several systems (batching form).
// One job per system; its work items are (K-split, tile) pairs.  Job q owns
// the slots [w0, w0 + npad) of the launch, npad = its item count rounded up
// to a multiple of 8 and w0 a multiple of 8, so that slot w runs on XCD
// w mod 8 and every job is spread evenly over the eight XCDs (the items of
// different systems differ in K, hence in cost, by an order of magnitude:
// an equal item count per XCD would leave some XCDs idle).  Within a job,
// xcd_remap gives each XCD a contiguous run of items, which share operand
// panels in its L2.  Jobs are ordered by decreasing cost per item, so the
// tail of the launch is made of the cheapest items.  Workgroup b takes slots
// b, b + gridDim.x, ... (gridDim.x a multiple of 8).
constexpr int GMAX = 16;   // systems per grouped launch
struct GemmJob {
  const void* A;     // Y-build: LvT32 (complex64) or LvTB (split);  sigma2: X32 or XB
  const void* B;     // Y-build: Rt32 or RB;  sigma2: Lv32 or LvB
  void* C;           // Y (double2, nsplit partials) or Z (float2)
  int rows, no, nv, naux, nsplit;
  long ntile;        // output tiles of one K-split
  long w0;           // first slot (a multiple of 8)
};
struct GemmJobs {
  int n;
  long total;
  GemmJob j[GMAX];
};

__device__ __forceinline__ int job_of(const GemmJobs& J, long item) {
  int q = 0;
  for (int t = 1; t < J.n; ++t)
    if (item >= J.j[t].w0) q = t;
  return q;
}

// Item of slot w of job g, or -1 for a padding slot.
__device__ __forceinline__ long job_item(const GemmJob& g, long w) {
  const long nit = g.ntile * g.nsplit;
  const long item = xcd_remap(w - g.w0, (nit + 7) & ~7L);
  return item < nit ? item : -1;
}

template <bool YBUILD>
__global__ __launch_bounds__(256, 2) void k_gemm_c64_grouped(const GemmJobs J) {
  __shared__ BigSmemF s[2];
  for (long w = blockIdx.x; w < J.total; w += gridDim.x) {
    const GemmJob& g = J.j[job_of(J, w)];
    const long loc = job_item(g, w);
    if (loc < 0) continue;
    const int split = (int)(loc / g.ntile);
    const long lid = loc - (long)split * g.ntile;
    if (YBUILD)
      ygemm_c64_item(s, (const float2*)g.A, (const float2*)g.B, g.rows, g.no, g.nv, g.naux, (double2*)g.C, lid,
                     split, g.nsplit);
    else
      zsig2_c64_item(s, (const float2*)g.A, (const float2*)g.B, g.rows, g.no, g.nv, g.naux, (float2*)g.C, lid);
  }
}

template <bool YBUILD>
__global__ __launch_bounds__(512) void k_gemm_b3_grouped(const GemmJobs J) {
  __shared__ BigSmemB s[2];
  for (long w = blockIdx.x; w < J.total; w += gridDim.x) {
    const GemmJob& g = J.j[job_of(J, w)];
    const long loc = job_item(g, w);
    if (loc < 0) continue;
    const int split = (int)(loc / g.ntile);
    const long lid = loc - (long)split * g.ntile;
    if (YBUILD)
      ygemm_b3_item(s, (const __bf16*)g.A, (const __bf16*)g.B, g.rows, g.no, g.nv, g.naux, (double2*)g.C, lid,
                    split, g.nsplit);
    else
      zsig2_b3_item(s, (const __bf16*)g.A, (const __bf16*)g.B, g.rows, g.no, g.nv, g.naux, (float2*)g.C, lid);
  }
}

__global__ void k_to_c64(const double2* __restrict__ src, long n, float2* __restrict__ dst) {
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x)
    dst[e] = make_float2((float)src[e].x, (float)src[e].y);
}

// Y = sum of the split partials (in place into split 0)
__global__ void k_ysum(double2* __restrict__ Y, long len, int nsplit) {
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < len; e += (long)gridDim.x * blockDim.x) {
    double2 a = Y[e];
    for (int s = 1; s < nsplit; ++s) a = cadd(a, Y[(long)s * len + e]);
    Y[e] = a;
  }
}

__device__ __forceinline__ long pair_offset(int a, int b, int nv) {
  return (long)a * nv - (long)a * (a + 1) / 2 + (b - a - 1);
}

// Unpack the doubles of the nrow (vector, core) pairs mI0 <= mI into the
// k-major Y-build operand
//   Rt[(j, d)][(mI - mI0, c)] = R_{mI j}[c][d]   (c<d packed, c>d negated, 0 on c=d)
// with row (j,d) = j*nv + d of length nrow*nv.  One workgroup per
// (mI, j, 32x32 tile pair cb <= db): the packed upper tile is read along d
// (contiguous) and written both straight and, through LDS, transposed; every
// global access is coalesced.
constexpr int UT = 32;
template <class TO, bool WTS>
__global__ __launch_bounds__(256) void k_unpack(const double2* __restrict__ xin, long dim, int mI0, int nrow, int nc,
                                                 int no, int nv, TO* __restrict__ Rt,
                                                 const double* __restrict__ wts) {
  __shared__ double2 t[UT][UT + 1];
  const int nb = (nv + UT - 1) / UT;
  const int ntp = nb * (nb + 1) / 2;
  const long g = blockIdx.x / ntp;           // g = (mI - mI0)*no + j
  int tt = blockIdx.x % ntp, cbk = 0;
  while (tt >= nb - cbk) {
    tt -= nb - cbk;
    ++cbk;
  }
  const int dbk = cbk + tt;
  const int c0 = cbk * UT, d0 = dbk * UT;
  const long ns = (long)nc * nv;
  const long npair = (long)nv * (nv - 1) / 2;
  const int ml = (int)(g / no), j = (int)(g % no);
  const int mI = mI0 + ml;
  const int mv = mI / nc, I = mI - mv * nc;
  const double2* r2 = xin + (long)mv * dim + ns + ((long)I * no + j) * npair;
  const long ld = (long)nrow * nv;
  TO* R = Rt + (long)j * nv * ld + (long)ml * nv;   // R[d*ld + c] = R_{mIj}[c][d]
  const int tid = threadIdx.x;
  for (int e = tid; e < UT * UT; e += 256) {
    const int rc = e / UT, cd = e % UT;
    const int c = c0 + rc, d = d0 + cd;
    double2 v = czero();
    if (c < nv && d < nv && c < d) v = r2[pair_offset(c, d, nv)];
    if (WTS) v = cscale(v, wts[mv]);
    t[rc][cd] = v;    // t[c][d] = R[c][d] on the upper tile
  }
  __syncthreads();
  // rows d of the d-tile, columns c of the c-tile: R[c][d] = t[c][d] (c<d)
  for (int e = tid; e < UT * UT; e += 256) {
    const int rd = e / UT, cc = e % UT;
    const int d = d0 + rd, c = c0 + cc;
    if (c < nv && d < nv) {
      double2 v;
      if (cbk == dbk) v = (c < d) ? t[cc][rd] : (c > d ? cneg(t[rd][cc]) : czero());
      else v = t[cc][rd];
      R[(long)d * ld + c] = from_d2<TO>(v);
    }
  }
  if (cbk != dbk) {
    // rows c of the c-tile, columns d of the d-tile: R[d][c] = -R[c][d]
    for (int e = tid; e < UT * UT; e += 256) {
      const int rc = e / UT, cd = e % UT;
      const int c = c0 + rc, d = d0 + cd;
      if (c < nv && d < nv) R[(long)c * ld + d] = from_d2<TO>(cneg(t[rc][cd]));
    }
  }
}

// One-time conjugate transpose of the occupied Cholesky block:
//   LoT[(l, d)][P] = conj(L^P_{d l}) = conj(Lvo[l][P][d])   for every occupied l.
// Its valence rows are the Y-build operand; the adjoint also uses the core rows.
__global__ __launch_bounds__(256) void k_lvo_transpose(const double2* __restrict__ Lvo, int nv, int naux,
                                                        double2* __restrict__ LoT) {
  __shared__ double2 t[UT][UT + 1];
  const int nbd = (nv + UT - 1) / UT, nbp = (naux + UT - 1) / UT;
  const int l = blockIdx.x / (nbd * nbp);
  const int rem = blockIdx.x % (nbd * nbp);
  const int p0 = (rem / nbd) * UT, d0 = (rem % nbd) * UT;
  const double2* src = Lvo + (long)l * naux * nv;
  for (int e = threadIdx.x; e < UT * UT; e += 256) {
    const int rp = e / UT, cd = e % UT;
    const int P = p0 + rp, d = d0 + cd;
    t[rp][cd] = (P < naux && d < nv) ? src[(long)P * nv + d] : czero();
  }
  __syncthreads();
  for (int e = threadIdx.x; e < UT * UT; e += 256) {
    const int rd = e / UT, cp = e % UT;
    const int d = d0 + rd, P = p0 + cp;
    if (P < naux && d < nv) LoT[((long)l * nv + d) * naux + P] = cconj(t[cp][rd]);
  }
}

// light sigma1 term, partial over a group of 4 valence j:
//   Tp[mI][jg][K][c] = sum_{j in group} sum_d conj(<Kd||Ij>) R_{mIj}[c][d]
//                    = sum_j sum_d conj(Vt[I][j][K][d]) Rt[(j,d)][(mI,c)]
// One workgroup per (mI, group, 64 values of c): wave w takes the group's j = w,
// lanes run over c (coalesced), the coefficients are broadcast from LDS, and
// the four waves' sums are added in order.  Bound by the one read of Rt; small
// tiles and one j a wave keep short systems and short chunks from running on a
// few workgroups (nc=6 no=10 nv=40, one vector: 59 us before on 18 workgroups
// that each walked four j; a chunk of eight rows at nv=300: 0.55 ms).
constexpr int LJG = 4;
constexpr int LC = 64;   // columns a workgroup
constexpr int LD = 64;   // d per staged run of coefficients
// DS waves share the d of a run
template <class TI, int DS>
__global__ __launch_bounds__(256 * DS) void k_light1(const TI* __restrict__ Rt, const double2* __restrict__ Vt, int mI0,
                                                      int nrow, int nc, int no, int nv, double2* __restrict__ Tp) {
  constexpr int NW = LJG * DS;
  constexpr int NQ = DS > 1 ? 4 : 8;   // values of q reduced at a time
  static_assert(NQ * (NW - 1) * 64 <= 64 * 64, "LDS");
  __shared__ double2 sh[NW * NQ * 64 > LJG * LD * 8 ? NW * NQ * 64 : LJG * LD * 8];
  double2(*vs)[LD][8] = (double2(*)[LD][8])sh;
  const int ncb = (nv + LC - 1) / LC;
  const int njg = (no + LJG - 1) / LJG;
  const int cb = blockIdx.x % ncb;
  const int jg = (blockIdx.x / ncb) % njg;
  const int ml = blockIdx.x / (ncb * njg), mI = mI0 + ml;
  const int I = mI % nc;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, w = wave % LJG, ds = wave / LJG;
  const int c = cb * LC + lane;
  const int cs = c < nv ? c : 0;
  const int j = jg * LJG + w;
  const bool jok = j < no;
  const long ld = (long)nrow * nv;
  const TI* R = Rt + (long)(jok ? j : 0) * nv * ld + (long)ml * nv + cs;   // R[d*ld]
  const double2* V = Vt + ((long)I * no + (jok ? j : 0)) * nc * nv;
  for (int K0 = 0; K0 < nc; K0 += 8) {
    double2 acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = czero();
    for (int d0 = 0; d0 < nv; d0 += LD) {
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 8 / DS; ++u) {
        const int q = u * DS + ds, K = K0 + q, d = d0 + lane;
        vs[w][lane][q] = (jok && K < nc && d < nv) ? cconj(V[(long)K * nv + d]) : czero();
      }
      __syncthreads();
      const int dend = min((ds + 1) * (LD / DS), nv - d0);
      // eight loads in flight a lane; past the end of the run the last row is read again and its
      // coefficients are zero; a lane past the last column reads column 0, its sums are never stored
      for (int dd = ds * (LD / DS); dd < dend; dd += 8) {
        TI r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) r[u] = R[(long)min(d0 + dd + u, nv - 1) * ld];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const double2 x = to_d2(r[u]);
#pragma unroll
          for (int q = 0; q < 8; ++q) acc[q] = cadd(acc[q], cmul(vs[w][dd + u][q], x));
        }
      }
    }
#pragma unroll
    for (int q0 = 0; q0 < 8; q0 += NQ) {
      __syncthreads();
      if (wave > 0)
#pragma unroll
        for (int q = 0; q < NQ; ++q) sh[((wave - 1) * NQ + q) * 64 + lane] = acc[q0 + q];
      __syncthreads();
      if (wave == 0 && c < nv)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          if (K0 + q0 + q >= nc) break;
          double2 t = acc[q0 + q];
          for (int v = 0; v < NW - 1; ++v) t = cadd(t, sh[(v * NQ + q) * 64 + lane]);
          Tp[(((long)mI * njg + jg) * nc + K0 + q0 + q) * nv + c] = t;
        }
    }
  }
}

// the partials of nrow rows from mI0 on (R: their unpacked doubles)
template <class TI>
static void light1_launch(const TI* R, const double2* Vt, int mI0, int nrow, const Dims& d, double2* Tp,
                          hipStream_t st) {
  const int per = cdiv(d.no, LJG) * cdiv(d.nv, LC);
  // By the system alone, not by the rows: every chunking of a block sums in the same order.
  // Up to 128 workgroups a vector four waves share a run: 23 us against 42 us with one (24 rows
  // of no=12 nv=100), 12 against 18 (6 rows of no=10 nv=40).  From there the chip is full with
  // one: 0.30 ms against 0.32 ms with four (a chunk of 12 rows of no=60 nv=300).
  if (per * d.nc <= 128)
    k_light1<TI, 4><<<(unsigned)((long)nrow * per), 1024, 0, st>>>(R, Vt, mI0, nrow, d.nc, d.no, d.nv, Tp);
  else
    k_light1<TI, 1><<<(unsigned)((long)nrow * per), 256, 0, st>>>(R, Vt, mI0, nrow, d.nc, d.no, d.nv, Tp);
}

// sigma2 = Z_ab - Z_ba + D r2 + sum_K (<Ka||Ij> r1_Kb - r1_Ka <Kb||Ij>), a < b, packed.
// One workgroup per (g = (mI - mI0, j), 32x32 tile pair ab <= bb); the mirror tile
// is staged in LDS so that both reads of Z are coalesced.  Bound by Z and r2 read and sigma2
// written: all of a thread's loads are issued at once and a column's coefficients read once for its
// four rows (loaded in turn behind the barrier: 0.57 ms a chunk of 2.1 GB, no=60 nv=300; 0.46 ms).
constexpr int PT = 32;
constexpr int PK = 8;    // core spinors staged in LDS by the pack kernel (more read from global memory)
template <class TZ>
__global__ __launch_bounds__(256) void k_pack2(const TZ* __restrict__ Z, const double2* __restrict__ xin,
                                                double2* __restrict__ sout, long dim, const double2* __restrict__ Vt,
                                                const double* __restrict__ eps, int mI0, int nc, int no, int nv,
                                                int with_d) {
  __shared__ double2 zt[PT][PT + 1];
  __shared__ double2 va[PK][PT], vb[PK][PT], ra[PK][PT], rb[PK][PT];
  __shared__ double ea[PT], eb[PT];
  const int nb = (nv + PT - 1) / PT;
  const int ntp = nb * (nb + 1) / 2;
  const long g = blockIdx.x / ntp;
  int t = blockIdx.x % ntp, abk = 0;
  while (t >= nb - abk) {
    t -= nb - abk;
    ++abk;
  }
  const int bbk = abk + t;
  const int a0 = abk * PT, b0 = bbk * PT;
  const int mI = mI0 + (int)(g / no), j = (int)(g % no);
  const int mv = mI / nc, I = mI - mv * nc;
  const int o = nc + no;
  const TZ* Zg = Z + g * (long)nv * nv;
  const double2* r1 = xin + (long)mv * dim;
  const double2* V = Vt + ((long)I * no + j) * nc * nv;
  const int tid = threadIdx.x;
  const bool staged = nc <= PK;
  // this thread's column cb and rows ra0 + 8 u of the tile: all its loads are issued before the barrier
  constexpr int NU = PT * PT / 256;
  const int cb = tid % PT, ra0 = tid / PT, b = b0 + cb;
  const long ns = (long)nc * nv;
  const long npair = (long)nv * (nv - 1) / 2;
  const long off = (long)mv * dim + ns + ((long)I * no + j) * npair;
  TZ zm[NU], zd[NU];
  double2 xd[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {   // mirror tile Z[b][a]
    const int bm = b0 + ra0 + 8 * u, am = a0 + cb;
    zm[u] = Zg[bm < nv && am < nv ? (long)bm * nv + am : 0];
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int a = a0 + ra0 + 8 * u;
    const bool ok = a < b && b < nv;
    zd[u] = Zg[ok ? (long)a * nv + b : 0];
    xd[u] = with_d && ok ? xin[off + pair_offset(a, b, nv)] : czero();
  }
  if (staged) {
    for (int e = tid; e < nc * PT; e += 256) {
      const int K = e / PT, x = e % PT;
      const int a = a0 + x, bx = b0 + x;
      va[K][x] = a < nv ? V[(long)K * nv + a] : czero();
      ra[K][x] = a < nv ? r1[(long)K * nv + a] : czero();
      vb[K][x] = bx < nv ? V[(long)K * nv + bx] : czero();
      rb[K][x] = bx < nv ? r1[(long)K * nv + bx] : czero();
    }
  }
  if (tid < PT) ea[tid] = (a0 + tid < nv) ? eps[o + a0 + tid] : 0.0;
  else if (tid < 2 * PT) eb[tid - PT] = (b0 + tid - PT < nv) ? eps[o + b0 + tid - PT] : 0.0;
#pragma unroll
  for (int u = 0; u < NU; ++u) zt[ra0 + 8 * u][cb] = to_d2(zm[u]);
  __syncthreads();
  if (b >= nv) return;
  const double eIj = eps[I] + eps[nc + j];
  double2 v[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) v[u] = csub(to_d2(zd[u]), zt[cb][ra0 + 8 * u]);
  if (staged) {
    for (int K = 0; K < nc; ++K) {   // the column's coefficients serve all its rows
      const double2 rbk = rb[K][cb], vbk = vb[K][cb];
#pragma unroll
      for (int u = 0; u < NU; ++u)
        v[u] = cadd(v[u], csub(cmul(va[K][ra0 + 8 * u], rbk), cmul(ra[K][ra0 + 8 * u], vbk)));
    }
  } else {
    for (int K = 0; K < nc; ++K) {
      const double2 rbk = r1[(long)K * nv + b], vbk = V[(long)K * nv + b];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int a = min(a0 + ra0 + 8 * u, nv - 1);
        v[u] = cadd(v[u], csub(cmul(V[(long)K * nv + a], rbk), cmul(r1[(long)K * nv + a], vbk)));
      }
    }
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int a = a0 + ra0 + 8 * u;
    if (a >= b) continue;
    const double D = ea[ra0 + 8 * u] + eb[cb] - eIj;
    if (with_d) v[u] = make_double2(v[u].x + D * xd[u].x, v[u].y + D * xd[u].y);
    sout[off + pair_offset(a, b, nv)] = v[u];
  }
}

// ---------------------------------------------------------------------------
// back-contraction:  part[split][mI][a] = sum_{P in split} sum_c Y[mI][P][c] Lvv[P][a][c]
// ---------------------------------------------------------------------------
struct SrcYrows {    // element (k=(P,c), i=mI)
  static constexpr int MAP = RMAJOR;
  const double2* Y;
  int nrow_y, nv, cpe, nrows, i0;
  __device__ __forceinline__ double2 get(int k, int i) const {
    const int chunk = k / TK;
    const int P = chunk / cpe;
    const int c = (chunk - P * cpe) * TK + (k % TK);
    const int mi = i0 + i;
    if (c >= nv || mi >= nrows) return czero();
    return Y[((long)mi * nrow_y + P) * nv + c];
  }
};

struct SrcLvvT {     // element (k=(P,c), i=a) = Lvv[P][a][c]
  static constexpr int MAP = RMAJOR;
  const double2* Lvv;
  int nv, cpe, a0;
  __device__ __forceinline__ double2 get(int k, int i) const {
    const int chunk = k / TK;
    const int P = chunk / cpe;
    const int c = (chunk - P * cpe) * TK + (k % TK);
    const int a = a0 + i;
    if (c >= nv || a >= nv) return czero();
    return Lvv[((long)P * nv + a) * nv + c];
  }
};

template <int MR>
__global__ __launch_bounds__(256) void k_backc(const double2* __restrict__ Y, const double2* __restrict__ Lvv,
                                                int nrows, int nv, int naux, int nsplit,
                                                double2* __restrict__ part) {
  __shared__ TileSmem s;
  const int nbi = cdiv(nrows, MR), nba = cdiv(nv, TN);
  const long nblocks = (long)nbi * nba * nsplit;
  const long lid = xcd_remap(blockIdx.x, nblocks);
  const int split = (int)(lid / ((long)nbi * nba));
  const int tile = (int)(lid % ((long)nbi * nba));
  const int i0 = (tile / nba) * MR, a0 = (tile % nba) * TN;
  const int cpe = cdiv(nv, TK);
  const int nchunks = naux * cpe;
  const int per = cdiv(nchunks, nsplit);
  const int kc0 = split * per, kc1 = min(nchunks, kc0 + per);
  SrcYrows A{Y, naux, nv, cpe, nrows, i0};
  SrcLvvT B{Lvv, nv, cpe, a0};
  AccT<MR> acc;
  acc.zero();
  mainloop(s, A, B, kc0, kc1, acc);
  double2* out = part + (long)split * nrows * nv;
  for_each_acc(acc, [&](int r, int c, double2 v) {
    const int mi = i0 + r, a = a0 + c;
    if (mi < nrows && a < nv) out[(long)mi * nv + a] = v;
  });
}

// s1[m][K][a] += sum_split part[split][mK][a] - sum_{I,jg} Tp[mI][jg][K][a].
// One workgroup per 64 entries; its 16 waves share the two lists of partials
// (a thread per entry walked up to 256 + nc no/4 dependent loads: 72 us at
// nc=6 no=12 nv=100, four vectors), and their sums are added in order.
constexpr int FW = 16;
__global__ __launch_bounds__(64 * FW) void k_sigma1_finish(const double2* __restrict__ part, int nsplit,
                                                           const double2* __restrict__ Tp, int m, int nc, int no, int nv,
                                                           long dim, double2* __restrict__ sout) {
  __shared__ double2 red[FW][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long total = (long)m * nc * nv;
  const long e = (long)blockIdx.x * 64 + lane;
  const bool ok = e < total;
  const long ec = ok ? e : 0;
  const int njg = (no + LJG - 1) / LJG;
  const int a = (int)(ec % nv);
  const int mK = (int)(ec / nv);
  const int mv = mK / nc, K = mK - mv * nc;
  double2 acc = czero();
#pragma unroll 4
  for (int sp = w; sp < nsplit; sp += FW) acc = cadd(acc, part[((long)sp * m * nc + mK) * nv + a]);
  const double2* T = Tp + ((long)mv * nc * njg * nc + K) * nv + a;   // (I, jg) at stride nc nv
#pragma unroll 4
  for (int q = w; q < nc * njg; q += FW) acc = csub(acc, T[(long)q * nc * nv]);
  red[w][lane] = acc;
  __syncthreads();
  if (w == 0 && ok) {
    for (int t = 1; t < FW; ++t) acc = cadd(acc, red[t][lane]);
    double2* p = sout + (long)mv * dim + (long)K * nv + a;
    *p = cadd(*p, acc);
  }
}

// y[m][row] = sum_k M11[row][k] x[m][k] for the rows of the singles block: a wave
// owns MVR rows and MVM vectors, lanes along k.  Bound by the read of M11 (64 x 64
// MFMA tiles put ns/64 workgroups on it: 287 us at ns=1800, ten vectors).
constexpr int MVR = 4, MVM = 4;
__global__ __launch_bounds__(256) void k_m11_mv(const double2* __restrict__ M11, int ns, const double2* __restrict__ x,
                                                long dim, int m, double2* __restrict__ y) {
  const int lane = threadIdx.x & 63;
  const int row0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * MVR, m0 = blockIdx.y * MVM;
  if (row0 >= ns) return;
  double2 acc[MVR][MVM];
#pragma unroll
  for (int r = 0; r < MVR; ++r)
#pragma unroll
    for (int q = 0; q < MVM; ++q) acc[r][q] = czero();
  const double2 *pr[MVR], *px[MVM];   // rows and vectors past the end: the last one again, never stored
#pragma unroll
  for (int r = 0; r < MVR; ++r) pr[r] = M11 + (long)min(row0 + r, ns - 1) * ns;
#pragma unroll
  for (int q = 0; q < MVM; ++q) px[q] = x + (long)min(m0 + q, m - 1) * dim;
#pragma unroll 2
  for (int k = lane; k < ns; k += 64) {
    double2 a[MVR], b[MVM];
#pragma unroll
    for (int r = 0; r < MVR; ++r) a[r] = pr[r][k];
#pragma unroll
    for (int q = 0; q < MVM; ++q) b[q] = px[q][k];
#pragma unroll
    for (int r = 0; r < MVR; ++r)
#pragma unroll
      for (int q = 0; q < MVM; ++q) acc[r][q] = cadd(acc[r][q], cmul(a[r], b[q]));
  }
#pragma unroll
  for (int r = 0; r < MVR; ++r)
#pragma unroll
    for (int q = 0; q < MVM; ++q) {
      double2 v = acc[r][q];
      for (int off = 32; off > 0; off >>= 1) {
        v.x += __shfl_xor(v.x, off);
        v.y += __shfl_xor(v.y, off);
      }
      if (lane == 0 && row0 + r < ns && m0 + q < m) y[(long)(m0 + q) * dim + row0 + r] = v;
    }
}

// ---------------------------------------------------------------------------

adc2_status build_lvt(adc2_handle h, hipStream_t st) {
  const Dims& d = h->d;
  if (h->LoT) return ADC2_OK;
  ADC2_HIP(dmalloc(h, &h->LoT, sizeof(double2) * (long)d.o * d.nv * d.naux));
  h->LvT = h->LoT + (long)d.nc * d.nv * d.naux;
  const long nblk = (long)d.o * cdiv(d.nv, UT) * cdiv(d.naux, UT);
  k_lvo_transpose<<<(unsigned)nblk, 256, 0, st>>>(h->Lvo, d.nv, d.naux, h->LoT);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

adc2_status build_c64(adc2_handle h, hipStream_t st) {
  const Dims& d = h->d;
  if (h->Lv32 && h->LvT32) return ADC2_OK;
  const long nlv = (long)d.no * d.naux * d.nv;
  ADC2_HIP(dmalloc(h, &h->Lv32, sizeof(float2) * nlv));
  ADC2_HIP(dmalloc(h, &h->LvT32, sizeof(float2) * nlv));
  k_to_c64<<<grid_for(nlv), 256, 0, st>>>(h->Lvo + (long)d.nc * d.naux * d.nv, nlv, h->Lv32);
  ADC2_CHECK_LAUNCH();
  k_to_c64<<<grid_for(nlv), 256, 0, st>>>(h->LvT, nlv, h->LvT32);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// Split-BF16 copies of the two static operands (blocked split layout).
adc2_status build_b3(adc2_handle h, hipStream_t st) {
  adc2_status rc = build_c64(h, st);
  if (rc != ADC2_OK) return rc;
  if (h->LvB && h->LvTB) return ADC2_OK;
  const Dims& d = h->d;
  const long K1 = d.naux, R1 = (long)d.no * d.nv;   // sigma2 B: rows (j,b), K = P
  const long K2 = (long)d.no * d.nv, R2 = d.naux;   // Y-build A: rows P, K = (j,d)
  ADC2_HIP(dmalloc(h, &h->LvB, split_bytes(R1, K1)));
  ADC2_HIP(dmalloc(h, &h->LvTB, split_bytes(R2, K2)));
  if ((rc = split_pack(h->Lv32, (long)d.naux * d.nv, d.nv, d.nv, R1, K1, (__bf16*)h->LvB, st)) != ADC2_OK) return rc;
  return split_pack(h->LvT32, 0, d.naux, d.naux, R2, K2, (__bf16*)h->LvTB, st);
}

// Split-BF16 operands and GEMM of the Schur preconditioner's three-virtual
// column.  pack_valence_b3 writes the valence rows of L in the sigma2 B layout
// (rows (j,b), K = P; the same bits as the handle's LvB).  schur_gemm_b3
// packs, for virtuals c in [c0, c0 + nck), A rows (cc,a) with element
// L^P_{a,c0+cc} (from Lvv[P][a][c]) into Ab and forms
//   Z[cc][j][a][b] = sum_P L^P_{a,c0+cc} L^P_{b,j}     (all j, a, b)
// on the sigma2 split-BF16 kernel.
adc2_status pack_valence_b3(adc2_handle h, __bf16* dst, hipStream_t st) {
  const Dims& d = h->d;
  return split_pack(h->Lvo + (long)d.nc * d.naux * d.nv, (long)d.naux * d.nv, d.nv, d.nv, (long)d.no * d.nv, d.naux,
                    dst, st);
}

adc2_status schur_gemm_b3(adc2_handle h, int c0, int nck, const __bf16* LvB, __bf16* Ab, float2* Z,
                          hipStream_t st) {
  const Dims& d = h->d;
  const long R = (long)nck * d.nv;
  // row (cc, a): group cc (stride 1 in Lvv), position a (stride nv), k = P (stride nv^2)
  adc2_status rc = split_pack(h->Lvv + c0, 1, (long)d.nv * d.nv, d.nv, R, d.naux, Ab, st, (long)d.nv);
  if (rc != ADC2_OK) return rc;
  const long nblk = (long)cdiv(R, BT) * cdiv((long)d.no * d.nv, BT);
  k_zsig2_b3<<<(unsigned)nblk, 512, 0, st>>>(Ab, LvB, (int)R, d.no, d.nv, d.naux, Z);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

adc2_status ensure_ws_b3(adc2_handle h, int m) {
  if (h->wsb_m >= m) return ADC2_OK;
  dfree(h, h->XB);
  dfree(h, h->RB);
  h->XB = h->RB = nullptr;
  h->wsb_m = 0;
  const Dims& d = h->d;
  const long rows = (long)m * d.nc * d.nv;
  ADC2_HIP(dmalloc(h, &h->XB, split_bytes(rows, d.naux)));
  ADC2_HIP(dmalloc(h, &h->RB, split_bytes(rows, (long)d.no * d.nv)));
  h->wsb_m = m;
  return ADC2_OK;
}

// Sizes of the FP64 sigma work spaces for a block of m vectors and the two
// split counts that go with them.
struct WsPlan {
  int ysplit, nsplit;
  size_t x, y, zb, tp, part;   // bytes of h->X, h->Y, h->Zb, h->Tp, h->part
};

// ys, ns > 0 impose the split counts instead of choosing them.
// The Y-build's K-split count (1..8) whose tiles fill whole rounds of the
// engine's workgroup slots best (the last round of a launch runs partly
// empty), each further split charged 0.2% for its partial sum.
int ysplit_rule(adc2_handle h, int m) {
  const Dims& d = h->d;
  const long rows = (long)m * d.nc;
  const bool fp64 = h->prec == ADC2_FP64;
  const int tn = fp64 && h->zgemm != ZGEMM_BIG && h->zgemm != ZGEMM_WIDE ? BT3N : BT;
  const long slots = 256L * ((fp64 && h->zgemm != ZGEMM_MID) || h->prec == ADC2_BF16X3 ? 1 : 2);
  const long ytiles = (long)cdiv(d.naux, BT) * cdiv(rows * d.nv, tn);
  int ys = 1;
  double best = 0.0;
  for (int c = 1; c <= 8; ++c) {
    const double rounds = (double)(ytiles * c) / slots;
    const double cost = std::ceil(rounds) / rounds * (1.0 + 0.002 * (c - 1));
    if (c == 1 || cost < best) {
      best = cost;
      ys = c;
    }
  }
  return ys;
}

static WsPlan ws_plan(adc2_handle h, int m, int ys = 0, int ns = 0) {
  const Dims& d = h->d;
  WsPlan p;
  const long rows = (long)m * d.nc;
  if (ys <= 0) {
    ys = ysplit_rule(h, m);
    if (const char* v = getenv("ADC2_YSPLIT")) ys = std::max(1, std::min(16, atoi(v)));
    if (h->ysplit_tuned > 0) ys = h->ysplit_tuned;   // adc2_autotune's choice
  }
  p.ysplit = ys;
  if (ns <= 0) {
    const int nbi = cdiv(rows, TM), nba = cdiv(d.nv, TN);
    ns = std::max(1, std::min(256, 2048 / std::max(1, nbi * nba)));
    ns = std::min(ns, d.naux);
  }
  p.nsplit = ns;
  const int njg = (d.no + LJG - 1) / LJG;
  p.x = sizeof(double2) * rows * d.naux * d.nv;
  p.y = sizeof(double2) * rows * d.naux * d.nv * p.ysplit;
  p.zb = sizeof(double2) * rows * d.no * (long)d.nv * d.nv;
  p.tp = sizeof(double2) * rows * njg * d.nc * d.nv;
  p.part = sizeof(double2) * p.nsplit * rows * d.nv;
  return p;
}

adc2_status ensure_ws(adc2_handle h, int m, bool zb) {
  if (h->ws_m < m) {
    dfree(h, h->X);
    dfree(h, h->Y);
    dfree(h, h->part);
    dfree(h, h->Tp);
    h->X = h->Y = h->part = h->Tp = nullptr;
    h->ws_m = 0;
    const WsPlan p = ws_plan(h, m);
    h->ysplit = p.ysplit;
    h->nsplit = p.nsplit;
    ADC2_HIP(dmalloc(h, &h->X, p.x));
    ADC2_HIP(dmalloc(h, &h->Y, p.y));
    ADC2_HIP(dmalloc(h, &h->Tp, p.tp));
    ADC2_HIP(dmalloc(h, &h->part, p.part));
    h->ws_m = m;
  }
  if (zb && h->zb_m < m) {
    dfree(h, h->Zb);
    h->Zb = nullptr;
    h->zb_m = 0;
    ADC2_HIP(dmalloc(h, &h->Zb, ws_plan(h, m).zb));
    h->zb_m = m;
  }
  return ADC2_OK;
}

// ---------------------------------------------------------------------------
// The FP64 form on the residue engine (rns.h).  The doubles are unpacked,
// multiplied and packed again in chunks of (vector, core) rows, so that its
// work space is that of one chunk whatever m: the unpacked doubles or the
// sigma2 product of the chunk in FP64 (16 B an entry), the residues of the one
// operand or product (32 B), and the other, smaller, in residues.
// ---------------------------------------------------------------------------
constexpr size_t NOALLOC_SCRATCH_BYTES = size_t(128) << 20;   // adc2_sigma_noalloc's work space

// Products of a sigma of `rows` (vector, core) rows worth the conversions: the
// engine is the faster one from about 10^7 terms a product on, whatever the
// shape (FP64 MFMA against residues, us per sigma: nc=6 no=10 nv=40 naux=150, one
// vector 193 / 150, 16 vectors 264 / 245; nc=6 no=12 nv=100 naux=300, four 509 /
// 458; nc=6 no=15 nv=60 naux=200, eight 336 / 336; nc=6 no=20 nv=100 naux=400, three 692 /
// 536; nc=6 no=60 nv=300 naux=1500, one 14686 / 6267).
static bool rns_sized(const Dims& d, double rows) {
  const double kx = d.naux, ky = (double)d.no * d.nv;
  return kx <= RNS_KMAX && ky <= RNS_KMAX && kx >= 128 && ky >= 256 && rows * d.nv * kx * ky >= 1.2e7;
}

// Work space of a chunk of c (vector, core) rows, as offsets.
struct RnsPlan {
  int c;
  size_t f64, opnd, out, ex, norm, bytes;
};
static RnsPlan rns_plan(adc2_handle h, int rows, size_t target = 0, bool whole = false) {
  if (target == 0) target = h->rns_short ? h->rns_short : h->rns_target;
  const Dims& d = h->d;
  const long ky = (long)d.no * d.nv;
  auto at = [&](int c) {
    RnsPlan p;
    p.c = c;
    const long r = (long)c * d.nv;
    size_t q = 0;
    auto take = [&](size_t b) {
      const size_t o = q;
      q += (b + 255) & ~size_t(255);
      return o;
    };
    p.f64 = take(sizeof(double2) * r * ky);
    p.opnd = take(std::max(rns_op_bytes(r, ky), rns_op_bytes(r, d.naux)));
    p.out = take(std::max(rns_out_bytes(d.naux, r) * rns_long_splits(ky), rns_out_bytes(r, ky) * rns_long_splits(d.naux)));
    p.ex = take(rns_exp_bytes(r));
    p.norm = take(rns_norm_bytes(r));
    p.bytes = q;
    return p;
  };
  const double one = (double)at(1).bytes;
  const int most = (int)std::max(1.0, std::min((double)rows, std::floor((double)target / one)));
  return at(whole ? most : cdiv(rows, cdiv(rows, most)));   // equal chunks
}
// Bytes that serve every block of up to `rows` rows (equal chunks of fewer rows may be the
// longer ones): what a handle once had for m vectors is enough for fewer, so its buffers stay
// where captured graphs found them.
static size_t rns_most(adc2_handle h, int rows) { return rns_plan(h, rows, 0, true).bytes; }

// Valence rows of Lvo as an operand: rows (j, b), K = P.
static RnsSrc rns_lvo_rows(adc2_handle h) {
  const Dims& d = h->d;
  return RnsSrc{h->Lvo + (long)d.nc * d.naux * d.nv, d.nv, (long)d.naux * d.nv, 1, 1 << 30, 0, d.nv, false};
}

// Sigma work spaces besides the chunk's, with the most back-contraction splits.
static size_t rns_fixed_bytes(const Dims& d, int m) {
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t rows = (size_t)m * d.nc, xy = al(16 * rows * d.naux * d.nv);
  const size_t njg = (d.no + LJG - 1) / LJG;
  return 2 * xy + al(16 * rows * njg * d.nc * d.nv) + al(16 * rows * d.nv * std::min(256, d.naux));
}

// Systems whose sigmas of up to 16 vectors may run on the residue engine: they get its
// static operands with the FP64 form (at the setup, or when the form is set).
static bool rns_system(adc2_handle h) {
  const Dims& d = h->d;
  if (h->rns_mode == RNS_NEVER || d.naux > RNS_KMAX || (long)d.no * d.nv > RNS_KMAX) return false;
  return h->rns_mode == RNS_ALWAYS || rns_sized(d, 16.0 * d.nc);
}

// Whether a sigma of m vectors runs on the residue engine.  Where the MFMA
// engines' work spaces fit adc2_sigma_noalloc's array, that entry point has to give
// the same bits without allocating: there the engine is used only if its own fit as
// well and the system has its static operands from the start.  (A handle that had to
// give them back gets them again from its next adc2_sigma; adc2_sigma_noalloc does without till then.)
static bool rns_wanted(adc2_handle h, int m, bool noalloc = false) {
  const Dims& d = h->d;
  const double rows = (double)m * d.nc;
  if (h->prec != ADC2_FP64 || h->rns_off || h->rns_mode == RNS_NEVER || d.naux > RNS_KMAX ||
      (long)d.no * d.nv > RNS_KMAX)
    return false;
  if (h->rns_mode != RNS_ALWAYS && !rns_sized(d, rows)) return false;
  if (16.0 * rows * (2.0 * d.naux * d.nv + (double)d.no * d.nv * d.nv) > NOALLOC_SCRATCH_BYTES) return true;
  if (!rns_system(h) || rns_fixed_bytes(d, m) + rns_plan(h, m * d.nc, 1).bytes > NOALLOC_SCRATCH_BYTES) return false;
  return !noalloc || (h->rns_lvo && h->rns_lvt);
}

// (on the device of the handle's blocks: adc2_set_precision has no other use for it, so that another one may be current)
adc2_status rns_enter_fp64(adc2_handle h, hipStream_t st) {
  if (h->prec != ADC2_FP64 || !rns_system(h) || (h->rns_lvo && h->rns_lvt)) return ADC2_OK;
  int cur = 0;
  hipPointerAttribute_t at{};
  ADC2_HIP(hipGetDevice(&cur));
  ADC2_HIP(hipPointerGetAttributes(&at, h->Lvo));
  if (at.device != cur) ADC2_HIP(hipSetDevice(at.device));
  const adc2_status rc = rns_build_static(h, st);
  if (at.device != cur) ADC2_HIP(hipSetDevice(cur));
  return rc;
}

adc2_status rns_build_static(adc2_handle h, hipStream_t st) {
  const Dims& d = h->d;
  const long ky = (long)d.no * d.nv;
  if (h->rns_lvo && h->rns_lvt) return ADC2_OK;
  if (h->rns_off || d.naux > RNS_KMAX || ky > RNS_KMAX) return ADC2_OK;
  double* norm = nullptr;
  hipError_t e = dmalloc_try(h, (void**)&norm, std::max(rns_norm_bytes(ky), rns_norm_bytes(d.naux)));
  if (e == hipSuccess) e = dmalloc_try(h, (void**)&h->rns_lvo, rns_op_bytes(ky, d.naux) + rns_exp_bytes(ky));
  if (e == hipSuccess)
    e = dmalloc_try(h, (void**)&h->rns_lvt, rns_op_bytes(d.naux, ky) + rns_exp_bytes(d.naux));
  adc2_status rc = ADC2_OK;
  if (e != hipSuccess) {   // without the memory: none of it
    (void)hipGetLastError();
    rns_release(h);
  } else {
    RnsMat t;
    rc = rns_pack(rns_lvo_rows(h), (int)ky, d.naux, (int8_t*)h->rns_lvo,
                  (int*)(h->rns_lvo + rns_op_bytes(ky, d.naux)), norm, &t, st);
    if (rc == ADC2_OK)
      rc = rns_pack(rns_kmajor(h->LvT, d.naux, (int)ky), d.naux, (int)ky, (int8_t*)h->rns_lvt,
                    (int*)(h->rns_lvt + rns_op_bytes(d.naux, ky)), norm, &t, st);
    if (hipStreamSynchronize(st) != hipSuccess && rc == ADC2_OK) {   // later calls may use other streams
      set_error("residue operands: stream synchronisation failed");
      rc = ADC2_ERR_HIP;
    }
    if (rc != ADC2_OK) rns_release(h);
  }
  dfree(h, norm);
  return rc;
}

// Terms of a product up to which the two halves of a sigma run side by side (sigma_overlapped), us
// one after the other / side by side: no=12 nv=100 naux=300, one vector (2e8) 201 / 158, four (9e8)
// 364 / 329; no=20 nv=200 naux=800, two (8e9) 1363 / 1303, four (1.5e10) 2285 / 2293; no=45
// nv=310 naux=1240, one (3e10), 4240 / 4470.
constexpr double OVERLAP_TERMS = 1e10;
static bool overlap_sized(const Dims& d, double rows) { return rows * d.nv * d.naux * d.no * d.nv <= OVERLAP_TERMS; }
static size_t overlap_base(adc2_handle h, int rows) { return (rns_plan(h, rows).bytes + 255) & ~size_t(255); }

// The residue engine's buffers for m vectors; *ok = false (and the MFMA engines)
// where the memory is not to be had.  Where it is short, first the
// scratch of the MFMA engines and of the split-BF16 form goes (it is allocated again when
// used: a two-stage solve at nc=6 no=120 nv=600 naux=3000 leaves 60 GB of it beside
// a search space of 153 GB, and its FP64 stage took 1.9 s a sigma of ten vectors
// on the MFMA engines, 0.63 s here), then chunks get smaller.  What was short is
// asked for again after RNS_WAIT sigmas of the handle (a request that fails and the
// buffers freed and taken around it: some ms).
constexpr int RNS_WAIT = 64;
static void rns_tick(adc2_handle h, hipStream_t st) {
  if (h->rns_wait == 0) return;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess) (void)hipGetLastError();
  if (cs != hipStreamCaptureStatusNone || --h->rns_wait > 0) return;
  h->rns_short = 0;
  h->rns_off = false;
}

static adc2_status rns_ready(adc2_handle h, int m, hipStream_t st, bool* ok) {
  *ok = false;
  const Dims& d = h->d;
  auto spare = [&]() {
    if (!h->Zb && !h->XB && !h->RB) return false;
    dfree(h, h->Zb);
    dfree(h, h->XB);
    dfree(h, h->RB);
    h->Zb = nullptr;
    h->XB = h->RB = nullptr;
    h->zb_m = h->wsb_m = 0;
    return true;
  };
  // blocks of up to m vectors whose halves run side by side
  const int side_m = (int)std::min<double>(m, OVERLAP_TERMS / ((double)d.nc * d.nv * d.naux * d.no * d.nv));
  for (;;) {
    const adc2_status rc = rns_build_static(h, st);
    if (rc != ADC2_OK) return rc;
    if (h->rns_lvo && h->rns_lvt) {
      if (h->side && !h->rns_lent && h->rns_wait == 0 && side_m > 0) {
        if (rns_reserve(h, std::max(rns_most(h, m * d.nc), 2 * ((rns_most(h, side_m * d.nc) + 255) & ~size_t(255))))) break;
        h->rns_wait = RNS_WAIT;
      }
      if (rns_reserve(h, rns_most(h, m * d.nc))) break;
    }
    if (h->rns_lent) return ADC2_OK;   // (sized before the array was lent)
    if (spare()) continue;
    h->rns_wait = RNS_WAIT;
    if (!h->rns_lvo || !h->rns_lvt || rns_plan(h, m * d.nc).c <= 1) {
      rns_release(h);
      h->rns_off = true;
      return ADC2_OK;
    }
    h->rns_short = (h->rns_short ? h->rns_short : h->rns_target) / 2;
  }
  *ok = true;
  return ADC2_OK;
}

static RnsMat rns_static(char* mem, long rows, long K, const RnsSrc& src) {
  RnsMat a;
  a.src = src;
  a.p = (int8_t*)mem;
  a.e = (int*)(mem + rns_op_bytes(rows, K));
  a.rows = (int)rows;
  a.K = (int)K;
  a.nrt = cdiv(rows, RNS_RT);
  a.nkc = cdiv(K, RNS_KC);
  return a;
}

// Event pairs around the launches of a kernel class, summed at the end.
struct RnsProf {
  bool on;
  hipStream_t st;
  struct Seg {
    int slot;
    hipEvent_t a, b;
  };
  std::vector<Seg> segs;
  template <class F>
  adc2_status run(int slot, F&& f) {
    if (!on) return f();
    Seg s{slot, nullptr, nullptr};
    ADC2_HIP(hipEventCreate(&s.a));
    ADC2_HIP(hipEventCreate(&s.b));
    segs.push_back(s);
    ADC2_HIP(hipEventRecord(s.a, st));
    const adc2_status rc = f();
    ADC2_HIP(hipEventRecord(s.b, st));
    return rc;
  }
  // ms of a slot (the stream has been waited for)
  double ms(int slot) const {
    double t = 0.0;
    for (const Seg& s : segs) {
      float x = 0.f;
      if (s.slot == slot && hipEventElapsedTime(&x, s.a, s.b) == hipSuccess) t += x;
    }
    return t;
  }
  ~RnsProf() {
    for (const Seg& s : segs) {
      if (s.a) (void)hipEventDestroy(s.a);
      if (s.b) (void)hipEventDestroy(s.b);
    }
  }
};

// Y of the doubles input (and the light partials Tp), chunk by chunk.
static adc2_status rns_doubles_in(adc2_handle h, const SigReq& rq, RnsProf& pf, hipStream_t st) {
  const Dims& d = h->d;
  const int rows = rq.m * d.nc, K = d.no * d.nv;
  const RnsPlan p = rns_plan(h, rows);
  double2* R = (double2*)(h->rns_ws + p.f64);
  int8_t* out = (int8_t*)(h->rns_ws + p.out);
  const RnsMat L = rns_static(h->rns_lvt, d.naux, K, rns_kmajor(h->LvT, d.naux, K));
  const int nb = cdiv(d.nv, UT);
  for (int r0 = 0; r0 < rows; r0 += p.c) {
    const int c = std::min(p.c, rows - r0);
    adc2_status rc = pf.run(0, [&]() -> adc2_status {
      k_unpack<double2, false><<<(unsigned)((long)c * d.no * (nb * (nb + 1) / 2)), 256, 0, st>>>(
          rq.xin, d.dim, r0, c, d.nc, d.no, d.nv, R, nullptr);
      ADC2_CHECK_LAUNCH();
      return ADC2_OK;
    });
    if (rc != ADC2_OK) return rc;
    rc = pf.run(2, [&]() -> adc2_status {
      light1_launch(R, h->Vt, r0, c, d, h->Tp, st);
      ADC2_CHECK_LAUNCH();
      return ADC2_OK;
    });
    if (rc != ADC2_OK) return rc;
    rc = pf.run(1, [&]() -> adc2_status {
      RnsMat B;
      const int ncol = c * d.nv;
      adc2_status r = rns_pack(rns_kmajor(R, ncol, K), ncol, K, (int8_t*)(h->rns_ws + p.opnd), (int*)(h->rns_ws + p.ex),
                               (double*)(h->rns_ws + p.norm), &B, st);
      const int ns = rns_long_splits(K);
      if (r == ADC2_OK) r = rns_gemm(L, B, 0, ncol, ns, out, st);
      // Y[mI][P][c], columns (mI, c)
      const RnsDst y{h->Y + (long)r0 * d.naux * d.nv, 1 << 30, 0, d.nv, d.nv, (long)d.naux * d.nv, 1, 1.0, false};
      if (r == ADC2_OK) r = rns_join(L, B, 0, ncol, ns, out, y, st);
      return r;
    });
    if (rc != ADC2_OK) return rc;
  }
  return ADC2_OK;
}

// sigma2 of the singles input (X built), chunk by chunk.
static adc2_status rns_singles_in(adc2_handle h, const SigReq& rq, int with_d, RnsProf& pf, char* ws, hipStream_t st) {
  const Dims& d = h->d;
  const int rows = rq.m * d.nc, N = d.no * d.nv;
  const RnsPlan p = rns_plan(h, rows);
  double2* Z = (double2*)(ws + p.f64);
  int8_t* out = (int8_t*)(ws + p.out);
  const RnsMat L = rns_static(h->rns_lvo, N, d.naux, rns_lvo_rows(h));
  const int nb = cdiv(d.nv, PT);
  for (int r0 = 0; r0 < rows; r0 += p.c) {
    const int c = std::min(p.c, rows - r0);
    adc2_status rc = pf.run(4, [&]() -> adc2_status {
      RnsMat A;
      const RnsSrc x{h->X + (long)r0 * d.naux * d.nv, d.nv, (long)d.naux * d.nv, 1, 1 << 30, 0, d.nv, false};
      adc2_status r = rns_pack(x, c * d.nv, d.naux, (int8_t*)(ws + p.opnd), (int*)(ws + p.ex),
                               (double*)(ws + p.norm), &A, st);
      const int ns = rns_long_splits(d.naux);
      if (r == ADC2_OK) r = rns_gemm(A, L, 0, N, ns, out, st);
      // Z[mI][j][a][b], rows (mI, a), columns (j, b)
      const RnsDst z{Z, d.nv, (long)d.no * d.nv * d.nv, d.nv, d.nv, (long)d.nv * d.nv, 1, 1.0, false};
      if (r == ADC2_OK) r = rns_join(A, L, 0, N, ns, out, z, st);
      return r;
    });
    if (rc != ADC2_OK) return rc;
    rc = pf.run(5, [&]() -> adc2_status {
      k_pack2<double2><<<(unsigned)((long)c * d.no * (nb * (nb + 1) / 2)), 256, 0, st>>>(
          Z, rq.xin, rq.sout, d.dim, h->Vt, h->eps, r0, d.nc, d.no, d.nv, with_d);
      ADC2_CHECK_LAUNCH();
      return ADC2_OK;
    });
    if (rc != ADC2_OK) return rc;
  }
  return ADC2_OK;
}

// Weighted unpack Rt[(j,d)][(mI,c)] = w_m R_{mIj}[c][d] into h->Zb, and the
// FP64 Y-build on it into h->Y (split partials summed); used by the adjoint.
adc2_status unpack_weighted(adc2_handle h, int m, const double2* xin, const double* wts, hipStream_t st) {
  const Dims& d = h->d;
  const int nb = cdiv(d.nv, UT);
  const long nblk = (long)m * d.nc * d.no * (nb * (nb + 1) / 2);
  k_unpack<double2, true><<<(unsigned)nblk, 256, 0, st>>>(xin, d.dim, 0, m * d.nc, d.nc, d.no, d.nv, h->Zb, wts);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

adc2_status ybuild_fp64(adc2_handle h, int m, hipStream_t st) {
  const Dims& d = h->d;
  const int rows = m * d.nc;
  const long nblk = (long)cdiv(d.naux, BT) * cdiv((long)rows * d.nv, BT);
  dim3 grid((unsigned)nblk, h->ysplit);
  k_ygemm<false><<<grid, 256, 0, st>>>(h->LvT, h->Zb, rows, d.nc, d.no, d.nv, d.naux, h->Y);
  ADC2_CHECK_LAUNCH();
  if (h->ysplit > 1) {
    const long len = (long)rows * d.naux * d.nv;
    k_ysum<<<grid_for(len), 256, 0, st>>>(h->Y, len, h->ysplit);
    ADC2_CHECK_LAUNCH();
  }
  return ADC2_OK;
}

adc2_status sigma_fp64(adc2_handle h, int m, const double2* xin, double2* sout, hipStream_t st) {
  return sigma_parts(h, m, xin, sout, SIGMA_SINGLES_IN | SIGMA_DOUBLES_IN, st);
}

// zero the singles block of m vectors
__global__ void k_zero_singles(double2* __restrict__ s, long dim, long ns, int m) {
  const long total = ns * m;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total; e += (long)gridDim.x * blockDim.x)
    s[(e / ns) * dim + e % ns] = make_double2(0.0, 0.0);
}

// parts = SIGMA_SINGLES_IN: sigma of (r1, 0):  s1 = M11 r1, s2 = M21 r1 (doubles of xin not read)
// parts = SIGMA_DOUBLES_IN: singles of the sigma of (0, r2): s1 = M12 r2 (singles of xin not read,
//                           doubles of sout not written)
// both: the full sigma.
adc2_status sigma_parts(adc2_handle h, int m, const double2* xin, double2* sout, int parts, hipStream_t st) {
  const SigReq r{h, m, xin, sout, parts};
  return sigma_multi(1, &r, st);
}

adc2_status sigma_call(adc2_handle h, int m, const double2* xin, double2* sout, int parts, hipStream_t st) {
  if (h->sigma_hook) return h->sigma_hook(m, xin, sout, parts, st);
  return sigma_parts(h, m, xin, sout, parts, st);
}

// The Y-build GEMM of one request (m vectors) in the handle's precision form,
// h->ysplit K-split partials into h->Y.
adc2_status ybuild_launch(adc2_handle h, int m, hipStream_t st) {
  const Dims& d = h->d;
  const int rows = m * d.nc;
  const int ys = h->ysplit;
  if (h->prec != ADC2_FP64) {
    const long nblk = (long)cdiv(d.naux, BT) * cdiv((long)rows * d.nv, BT);
    dim3 grid((unsigned)nblk, ys);
    if (h->prec == ADC2_BF16X3)
      k_ygemm_b3<<<grid, 512, 0, st>>>((const __bf16*)h->LvTB, (const __bf16*)h->RB, rows, d.no, d.nv, d.naux, h->Y);
    else
      k_ygemm_c64<<<grid, 256, 0, st>>>(h->LvT32, (const float2*)h->Zb, rows, d.no, d.nv, d.naux, h->Y);
  } else {
    const bool wide_tile = h->zgemm == ZGEMM_BIG || h->zgemm == ZGEMM_WIDE;
    const long nblk = (long)cdiv(d.naux, BT) * cdiv((long)rows * d.nv, wide_tile ? BT : BT3N);
    dim3 grid((unsigned)nblk, ys);
    if (h->zgemm == ZGEMM_WIDE)
      k_ygemm_wide<<<grid, 512, 0, st>>>(h->LvT, h->Zb, rows, d.no, d.nv, d.naux, h->Y);
    else if (h->zgemm == ZGEMM_MID)
      k_ygemm_mid<<<grid, 256, 0, st>>>(h->LvT, h->Zb, rows, d.no, d.nv, d.naux, h->Y);
    else if (h->zgemm == ZGEMM_3M)
      k_ygemm<true><<<grid, 256, 0, st>>>(h->LvT, h->Zb, rows, d.nc, d.no, d.nv, d.naux, h->Y);
    else
      k_ygemm<false><<<grid, 256, 0, st>>>(h->LvT, h->Zb, rows, d.nc, d.no, d.nv, d.naux, h->Y);
  }
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// Sum of the Y-build's K-split partials into the first one.
adc2_status ybuild_sum(adc2_handle h, int m, hipStream_t st) {
  const Dims& d = h->d;
  if (h->ysplit > 1) {
    const long len = (long)m * d.nc * d.naux * d.nv;
    k_ysum<<<grid_for(len), 256, 0, st>>>(h->Y, len, h->ysplit);
    ADC2_CHECK_LAUNCH();
  }
  return ADC2_OK;
}

// Launch the grouped heavy GEMM (Y-build if ybuild, else sigma2) of the
// requests selected by use[] whose handles share the precision form prec
// (complex64 or split-BF16), GMAX systems per launch.
static adc2_status grouped_gemm(int nreq, const SigReq* rq, const std::vector<char>& use, int prec, bool ybuild,
                                hipStream_t st) {
  GemmJobs J;
  J.n = 0;
  J.total = 0;
  auto flush = [&]() -> adc2_status {
    if (J.n == 0) return ADC2_OK;
    const unsigned grid = (unsigned)std::min<long>(J.total, 1L << 20);   // both multiples of 8
    if (prec == ADC2_BF16X3) {
      if (ybuild) k_gemm_b3_grouped<true><<<grid, 512, 0, st>>>(J);
      else k_gemm_b3_grouped<false><<<grid, 512, 0, st>>>(J);
    } else {
      if (ybuild) k_gemm_c64_grouped<true><<<grid, 256, 0, st>>>(J);
      else k_gemm_c64_grouped<false><<<grid, 256, 0, st>>>(J);
    }
    ADC2_CHECK_LAUNCH();
    J.n = 0;
    J.total = 0;
    return ADC2_OK;
  };
  // requests of this form, by decreasing K per item (ties: request order)
  std::vector<std::pair<long, int>> order;
  for (int q = 0; q < nreq; ++q) {
    if (!use[q] || rq[q].h->prec != prec) continue;
    const Dims& d = rq[q].h->d;
    const long kpi = ybuild ? (long)d.no * d.nv / std::max(1, rq[q].h->ysplit) : (long)d.naux;
    order.push_back({-kpi, q});
  }
  std::stable_sort(order.begin(), order.end(),
                   [](const std::pair<long, int>& a, const std::pair<long, int>& b) { return a.first < b.first; });
  for (const auto& oq : order) {
    const int q = oq.second;
    adc2_handle h = rq[q].h;
    const Dims& d = h->d;
    const int rows = rq[q].m * d.nc;
    GemmJob& g = J.j[J.n];
    g.rows = ybuild ? rows : rows * d.nv;
    g.no = d.no;
    g.nv = d.nv;
    g.naux = d.naux;
    const bool split = prec == ADC2_BF16X3;
    if (ybuild) {
      g.A = split ? h->LvTB : (const void*)h->LvT32;
      g.B = split ? h->RB : (const void*)h->Zb;
      g.C = h->Y;
      g.nsplit = h->ysplit;
      g.ntile = (long)cdiv(d.naux, BT) * cdiv((long)rows * d.nv, BT);
    } else {
      g.A = split ? h->XB : (const void*)h->X;
      g.B = split ? h->LvB : (const void*)h->Lv32;
      g.C = h->Zb;
      g.nsplit = 1;
      g.ntile = (long)cdiv((long)rows * d.nv, BT) * cdiv((long)d.no * d.nv, BT);
    }
    g.w0 = J.total;
    J.total += (g.ntile * g.nsplit + 7) & ~7L;
    if (++J.n == GMAX) {
      adc2_status r = flush();
      if (r != ADC2_OK) return r;
    }
  }
  return flush();
}

static adc2_status backc_launch(adc2_handle h, int m, hipStream_t st) {
  const Dims& d = h->d;
  const int rows = m * d.nc;
  const int mr = thin_rows(d, rows) ? 0 : row_tile(rows);
  const unsigned nblk = (unsigned)((long)(mr ? cdiv(rows, mr) : 1) * cdiv(d.nv, TN) * h->nsplit);
  if (mr == 0) k_backc_thin<<<nblk, 256, 0, st>>>(h->Y, h->Lvv, rows, d.nv, d.naux, h->nsplit, h->part);
  else if (mr == 32) k_backc<32><<<nblk, 256, 0, st>>>(h->Y, h->Lvv, rows, d.nv, d.naux, h->nsplit, h->part);
  else if (mr == 48) k_backc<48><<<nblk, 256, 0, st>>>(h->Y, h->Lvv, rows, d.nv, d.naux, h->nsplit, h->part);
  else k_backc<64><<<nblk, 256, 0, st>>>(h->Y, h->Lvv, rows, d.nv, d.naux, h->nsplit, h->part);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

static adc2_status m11_launch(adc2_handle h, const SigReq& rq, hipStream_t st) {
  const Dims& d = h->d;
  k_m11_mv<<<dim3(cdiv(d.ns, 4 * MVR), cdiv(rq.m, MVM)), 256, 0, st>>>(h->M11, (int)d.ns, rq.xin, d.dim, rq.m, rq.sout);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

static adc2_status finish_launch(adc2_handle h, const SigReq& rq, hipStream_t st) {
  const Dims& d = h->d;
  k_sigma1_finish<<<cdiv((long)rq.m * d.nc * d.nv, 64), 64 * FW, 0, st>>>(h->part, h->nsplit, h->Tp, rq.m, d.nc, d.no,
                                                                          d.nv, d.dim, rq.sout);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// Small sigmas on the residue engine run their two halves side by side: the
// doubles-in chain on the caller's stream, the singles-in chain on the handle's own,
// between two events on the caller's stream, in two halves of the work space.  Each
// chain is eight or nine launches that fill a part of the chip each.  Not under
// capture and not while the kernels are timed.
// Whether requests may use the first handle's second stream.
static bool side_free(adc2_handle h, hipStream_t st) {
  if (!h->side || h->rns_lent || h->profiling) return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return cs == hipStreamCaptureStatusNone;
}

static adc2_status sigma_overlapped(adc2_handle h, const SigReq& rq, RnsProf& rp, hipStream_t st) {
  const int rows = rq.m * h->d.nc;
  ADC2_HIP(hipEventRecord(h->side_fork, st));
  ADC2_HIP(hipStreamWaitEvent(h->side, h->side_fork, 0));
  adc2_status rc = rns_doubles_in(h, rq, rp, st);
  if (rc == ADC2_OK) rc = backc_launch(h, rq.m, st);
  if (rc == ADC2_OK) rc = xbuild_launch(rq.xin, h->d, rows, h->Lvv, h->X, h->side);
  if (rc == ADC2_OK) rc = rns_singles_in(h, rq, 1, rp, h->rns_ws + overlap_base(h, rows), h->side);
  if (rc == ADC2_OK) rc = m11_launch(h, rq, h->side);
  // joined whatever happened
  if (hipEventRecord(h->side_join, h->side) != hipSuccess || hipStreamWaitEvent(st, h->side_join, 0) != hipSuccess) {
    (void)hipStreamSynchronize(h->side);
    set_error("adc2_sigma: the two halves could not be joined");
    if (rc == ADC2_OK) rc = ADC2_ERR_HIP;
  }
  return rc == ADC2_OK ? finish_launch(h, rq, st) : rc;
}

// Several sigma requests (possibly of different systems) on one stream.  Each
// phase runs for every request before the next phase; with more than one
// request the two heavy GEMMs of the requests in the complex64 and split-BF16
// forms are one grouped launch per form.  Per-kernel profiling (adc2_profile)
// is recorded for single requests only.
adc2_status sigma_multi(int nreq, const SigReq* rq, hipStream_t st, bool allow_rns) {
  adc2_status rc;
  std::vector<char> rns(nreq, 0);   // requests on the residue engine
  for (int q = 0; q < nreq; ++q) {
    adc2_handle h = rq[q].h;
    if (!h->rns_lent) rns_tick(h, st);
    if (allow_rns && rns_wanted(h, rq[q].m)) {
      bool ok = false;
      if ((rc = ensure_ws(h, rq[q].m, false)) != ADC2_OK || (rc = rns_ready(h, rq[q].m, st, &ok)) != ADC2_OK) return rc;
      rns[q] = ok;
    }
    if ((rc = ensure_ws(h, rq[q].m, !rns[q])) != ADC2_OK) return rc;
    const bool b3 = h->prec == ADC2_BF16X3;
    const bool c64 = h->prec == ADC2_C64 || b3;   // complex64 operand copies
    if (c64 && (rc = build_c64(h, st)) != ADC2_OK) return rc;
    if (b3 && ((rc = build_b3(h, st)) != ADC2_OK || (rc = ensure_ws_b3(h, rq[q].m)) != ADC2_OK)) return rc;
  }
  adc2_handle h0 = rq[0].h;
  const bool prof = nreq == 1 && h0->profiling != 0;
  RnsProf rp{prof && rns[0], st, {}};
  auto mark = [&](int i) -> adc2_status {
    if (prof) ADC2_HIP(hipEventRecord(h0->kev[i], st));
    return ADC2_OK;
  };
  std::vector<char> sgl(nreq), dbl(nreq);
  for (int q = 0; q < nreq; ++q) {
    sgl[q] = (rq[q].parts & SIGMA_SINGLES_IN) != 0;
    dbl[q] = (rq[q].parts & SIGMA_DOUBLES_IN) != 0;
  }
  const bool side = side_free(h0, st), whole = nreq == 1 && sgl[0] && dbl[0];
  if (side && whole && rns[0] && overlap_sized(h0->d, rq[0].m * h0->d.nc) &&
      h0->rns_ws_bytes >= 2 * overlap_base(h0, rq[0].m * h0->d.nc)) {
    if ((rc = sigma_overlapped(h0, rq[0], rp, st)) != ADC2_OK) return rc;
    return h0->method == ADC2_METHOD_ADC2X ? adc2x_apply(h0, rq[0].m, rq[0].xin, rq[0].sout, st) : ADC2_OK;
  }
  // precision forms that have a grouped GEMM and more than one request
  auto grouped = [&](const std::vector<char>& use, int prec) {
    if (nreq < 2) return false;
    int n = 0;
    for (int q = 0; q < nreq; ++q) n += use[q] && rq[q].h->prec == prec;
    return n > 0;
  };
  auto is_grouped = [&](int q) { return nreq > 1 && rq[q].h->prec != ADC2_FP64; };

  // X-build and back-contraction on the first handle's stream.  ASIDE (one whole request): beside the
  // products of the other half (no=45 nv=310, seven vectors: 24.0 -> 23.5 ms; split-BF16, no=60
  // nv=300, ten: 25.1 -> 24.1).  BESIDE (complex64, whose products leave the matrix cores no room:
  // 24.8 -> 25.1 aside; and batches of the precision forms): only beside the unpacking and the
  // packing (eight systems at once: 19.9 -> 19.5 ms; one: 24.8 -> 24.7).
  bool prec_all = true;
  for (int q = 0; q < nreq; ++q) prec_all = prec_all && rq[q].h->prec != ADC2_FP64;
  enum { SERIAL, ASIDE, BESIDE };
  const int how = !side ? SERIAL
                  : whole && h0->prec != ADC2_C64 ? ASIDE
                  : (whole || nreq > 1) && prec_all ? BESIDE : SERIAL;
  struct Joined {   // an error between fork and join: waited for before the caller's vectors go
    hipStream_t s;
    ~Joined() {
      if (s) (void)hipStreamSynchronize(s);
    }
  } joined{how != SERIAL ? h0->side : nullptr};
  auto xbuild_all = [&](hipStream_t on) -> adc2_status {
    for (int q = 0; q < nreq; ++q) {
      if (!sgl[q]) continue;
      adc2_handle h = rq[q].h;
      const int rows = rq[q].m * h->d.nc;
      const adc2_status r = h->prec != ADC2_FP64 ? xbuild_launch(rq[q].xin, h->d, rows, h->Lvv, (float2*)h->X, on)
                                                 : xbuild_launch(rq[q].xin, h->d, rows, h->Lvv, h->X, on);
      if (r != ADC2_OK) return r;
    }
    return ADC2_OK;
  };
  auto backc_all = [&](hipStream_t on) -> adc2_status {
    for (int q = 0; q < nreq; ++q)
      if (dbl[q]) {
        const adc2_status r = backc_launch(rq[q].h, rq[q].m, on);
        if (r != ADC2_OK) return r;
      }
    return ADC2_OK;
  };
  auto fork = [&](auto&& work) -> adc2_status {   // after what the stream holds so far
    ADC2_HIP(hipEventRecord(h0->side_fork, st));
    ADC2_HIP(hipStreamWaitEvent(h0->side, h0->side_fork, 0));
    const adc2_status r = work(h0->side);
    ADC2_HIP(hipEventRecord(h0->side_join, h0->side));
    return r;
  };
  auto join = [&]() -> adc2_status {
    ADC2_HIP(hipStreamWaitEvent(st, h0->side_join, 0));
    return ADC2_OK;
  };
  if (how != SERIAL && (rc = fork(xbuild_all)) != ADC2_OK) return rc;
  // kernel order (profiling slots): unpack, ygemm, light1, xbuild, zsig2, pack2, backc, m11mv+finish
  for (int q = 0; q < nreq; ++q)
    if (rns[q] && dbl[q] && (rc = rns_doubles_in(rq[q].h, rq[q], rp, st)) != ADC2_OK) return rc;
  if ((rc = mark(0)) != ADC2_OK) return rc;
  for (int q = 0; q < nreq; ++q) {
    if (!dbl[q] || rns[q]) continue;
    adc2_handle h = rq[q].h;
    const Dims& d = h->d;
    const bool c64 = h->prec != ADC2_FP64;
    const int nb = cdiv(d.nv, UT);
    const long nblk = (long)rq[q].m * d.nc * d.no * (nb * (nb + 1) / 2);
    if (c64)
      k_unpack<float2, false><<<(unsigned)nblk, 256, 0, st>>>(rq[q].xin, d.dim, 0, rq[q].m * d.nc, d.nc, d.no,
                                                               d.nv, (float2*)h->Zb, nullptr);
    else
      k_unpack<double2, false><<<(unsigned)nblk, 256, 0, st>>>(rq[q].xin, d.dim, 0, rq[q].m * d.nc, d.nc, d.no,
                                                                d.nv, h->Zb, nullptr);
    ADC2_CHECK_LAUNCH();
  }
  for (int q = 0; q < nreq; ++q) {   // split-BF16: the unpacked doubles into the blocked split layout
    adc2_handle h = rq[q].h;
    if (!dbl[q] || h->prec != ADC2_BF16X3) continue;
    const Dims& d = h->d;
    const long ncols = (long)rq[q].m * d.nc * d.nv;
    if ((rc = split_pack((const float2*)h->Zb, 0, ncols, (int)ncols, ncols, (long)d.no * d.nv, (__bf16*)h->RB, st)) !=
        ADC2_OK)
      return rc;
  }
  if (how == BESIDE && (rc = join()) != ADC2_OK) return rc;
  if ((rc = mark(1)) != ADC2_OK) return rc;
  for (int prec : {ADC2_C64, ADC2_BF16X3})
    if (grouped(dbl, prec) && (rc = grouped_gemm(nreq, rq, dbl, prec, true, st)) != ADC2_OK) return rc;
  for (int q = 0; q < nreq; ++q) {
    if (!dbl[q] || rns[q]) continue;
    adc2_handle h = rq[q].h;
    if (!is_grouped(q) && (rc = ybuild_launch(h, rq[q].m, st)) != ADC2_OK) return rc;
    if ((rc = ybuild_sum(h, rq[q].m, st)) != ADC2_OK) return rc;
  }
  if ((rc = mark(2)) != ADC2_OK) return rc;
  for (int q = 0; q < nreq; ++q) {
    if (!dbl[q] || rns[q]) continue;
    adc2_handle h = rq[q].h;
    const Dims& d = h->d;
    const int rows = rq[q].m * d.nc;
    if (h->prec != ADC2_FP64) light1_launch((const float2*)h->Zb, h->Vt, 0, rows, d, h->Tp, st);
    else light1_launch(h->Zb, h->Vt, 0, rows, d, h->Tp, st);
    ADC2_CHECK_LAUNCH();
  }
  if ((rc = mark(3)) != ADC2_OK) return rc;
  if (how == ASIDE && ((rc = join()) != ADC2_OK || (rc = fork(backc_all)) != ADC2_OK)) return rc;
  if (how == SERIAL && (rc = xbuild_all(st)) != ADC2_OK) return rc;
  for (int q = 0; q < nreq; ++q) {   // split-BF16: X into the blocked split layout
    adc2_handle h = rq[q].h;
    if (!sgl[q] || h->prec != ADC2_BF16X3) continue;
    const Dims& d = h->d;
    if ((rc = split_pack((const float2*)h->X, (long)d.naux * d.nv, d.nv, d.nv, (long)rq[q].m * d.nc * d.nv, d.naux,
                         (__bf16*)h->XB, st)) != ADC2_OK)
      return rc;
  }
  if ((rc = mark(4)) != ADC2_OK) return rc;
  for (int prec : {ADC2_C64, ADC2_BF16X3})
    if (grouped(sgl, prec) && (rc = grouped_gemm(nreq, rq, sgl, prec, false, st)) != ADC2_OK) return rc;
  for (int q = 0; q < nreq; ++q) {
    if (!sgl[q] || is_grouped(q)) continue;
    adc2_handle h = rq[q].h;
    const Dims& d = h->d;
    const int rows = rq[q].m * d.nc;
    if (rns[q]) {
      if ((rc = rns_singles_in(h, rq[q], dbl[q] ? 1 : 0, rp, h->rns_ws, st)) != ADC2_OK) return rc;
      continue;
    }
    if (h->prec != ADC2_FP64) {
      const long nblk = (long)cdiv((long)rows * d.nv, BT) * cdiv((long)d.no * d.nv, BT);
      if (h->prec == ADC2_BF16X3)
        k_zsig2_b3<<<(unsigned)nblk, 512, 0, st>>>((const __bf16*)h->XB, (const __bf16*)h->LvB, rows * d.nv, d.no,
                                                     d.nv, d.naux, (float2*)h->Zb);
      else
        k_zsig2_c64<<<(unsigned)nblk, 256, 0, st>>>((const float2*)h->X, h->Lv32, rows * d.nv, d.no, d.nv, d.naux,
                                                      (float2*)h->Zb);
    } else if (h->zgemm == ZGEMM_WIDE) {
      const long nblk = (long)cdiv((long)rows * d.nv, BT) * cdiv((long)d.no * d.nv, BT);
      k_zsig2_wide<<<(unsigned)nblk, 512, 0, st>>>(h->X, h->Lvo, rows * d.nv, d.nc, d.no, d.nv, d.naux, h->Zb);
    } else if (h->zgemm == ZGEMM_MID) {
      const long nblk = (long)cdiv((long)rows * d.nv, BT) * cdiv((long)d.no * d.nv, MTN);
      k_zsig2_mid<<<(unsigned)nblk, 256, 0, st>>>(h->X, h->Lvo, rows * d.nv, d.nc, d.no, d.nv, d.naux, h->Zb);
    } else if (h->zgemm == ZGEMM_3M) {
      const long nblk = (long)cdiv((long)rows * d.nv, BT) * cdiv((long)d.no * d.nv, BT3N);
      k_zsig2<true><<<(unsigned)nblk, 256, 0, st>>>(h->X, h->Lvo, rows * d.nv, d.nc, d.no, d.nv, d.naux, h->Zb);
    } else {
      const long nblk = (long)cdiv((long)rows * d.nv, BT) * cdiv((long)d.no * d.nv, BT);
      k_zsig2<false><<<(unsigned)nblk, 256, 0, st>>>(h->X, h->Lvo, rows * d.nv, d.nc, d.no, d.nv, d.naux, h->Zb);
    }
    ADC2_CHECK_LAUNCH();
  }
  if (how == BESIDE && (rc = fork(backc_all)) != ADC2_OK) return rc;
  if ((rc = mark(5)) != ADC2_OK) return rc;
  for (int q = 0; q < nreq; ++q) {
    if (!sgl[q] || rns[q]) continue;
    adc2_handle h = rq[q].h;
    const Dims& d = h->d;
    const int m = rq[q].m;
    const int with_d = dbl[q] ? 1 : 0;
    const int nb = cdiv(d.nv, PT);
    const long nblk = (long)m * d.nc * d.no * (nb * (nb + 1) / 2);
    if (h->prec != ADC2_FP64)
      k_pack2<float2><<<(unsigned)nblk, 256, 0, st>>>((const float2*)h->Zb, rq[q].xin, rq[q].sout, d.dim, h->Vt,
                                                      h->eps, 0, d.nc, d.no, d.nv, with_d);
    else
      k_pack2<double2><<<(unsigned)nblk, 256, 0, st>>>(h->Zb, rq[q].xin, rq[q].sout, d.dim, h->Vt, h->eps, 0, d.nc,
                                                       d.no, d.nv, with_d);
    ADC2_CHECK_LAUNCH();
  }
  if ((rc = mark(6)) != ADC2_OK) return rc;
  if ((rc = how == SERIAL ? backc_all(st) : join()) != ADC2_OK) return rc;
  joined.s = nullptr;
  if ((rc = mark(7)) != ADC2_OK) return rc;
  for (int q = 0; q < nreq; ++q) {
    adc2_handle h = rq[q].h;
    const Dims& d = h->d;
    const int m = rq[q].m;
    if (sgl[q]) {
      if ((rc = m11_launch(h, rq[q], st)) != ADC2_OK) return rc;
    } else {
      k_zero_singles<<<grid_for(d.ns * m), 256, 0, st>>>(rq[q].sout, d.dim, d.ns, m);
      ADC2_CHECK_LAUNCH();
    }
    if (dbl[q] && (rc = finish_launch(h, rq[q], st)) != ADC2_OK) return rc;
  }
  if ((rc = mark(8)) != ADC2_OK) return rc;
  // ADC(2)-x: the first-order doubles block (FP64), on whole sigma requests only
  for (int q = 0; q < nreq; ++q) {
    adc2_handle h = rq[q].h;
    if (h->method != ADC2_METHOD_ADC2X) continue;
    if (!sgl[q] || !dbl[q]) {
      set_error("sigma: ADC(2)-x needs whole sigma products (partial products assume a diagonal doubles block)");
      return ADC2_ERR_ARG;
    }
    if ((rc = adc2x_apply(h, rq[q].m, rq[q].xin, rq[q].sout, st)) != ADC2_OK) return rc;
  }
  if (prof) {
    adc2_handle h = h0;
    const Dims& d = h->d;
    ADC2_HIP(hipEventSynchronize(h->kev[8]));
    const double nc_ = d.nc, no_ = d.no, nv_ = d.nv, na_ = d.naux, m_ = rq[0].m;
    const double heavy = 8.0 * m_ * nc_ * no_ * nv_ * nv_ * na_;
    const double fs = sgl[0] ? 1.0 : 0.0, fd = dbl[0] ? 1.0 : 0.0;
    const double fl[adc2_handle_s::NK] = {
        0.0,                                             // unpack (data movement)
        fd * heavy,                                      // Y-build GEMM
        fd * 8.0 * m_ * nc_ * no_ * nv_ * nv_ * nc_,     // light sigma1 core term
        fs * 8.0 * m_ * nc_ * nv_ * nv_ * na_,           // X-build
        fs * heavy,                                      // sigma2 GEMM
        fs * 8.0 * m_ * nc_ * no_ * nv_ * nv_ * nc_,     // pack + light sigma2 core term
        fd * 8.0 * m_ * nc_ * nv_ * nv_ * na_,           // back-contraction
        fs * 8.0 * m_ * (nc_ * nv_) * (nc_ * nv_)};      // M11 r1 + finish
    const bool ran[adc2_handle_s::NK] = {(bool)dbl[0], (bool)dbl[0], (bool)dbl[0], (bool)sgl[0],
                                          (bool)sgl[0], (bool)sgl[0], (bool)dbl[0], true};
    for (int i = 0; i < adc2_handle_s::NK; ++i) {
      if (!ran[i]) continue;
      float ms = 0.f;
      ADC2_HIP(hipEventElapsedTime(&ms, h->kev[i], h->kev[i + 1]));
      if (rns[0] && i != 3 && i < 6) ms = (float)rp.ms(i);   // its chunks' launches
      h->k_ms[i] += ms;
      h->k_launches[i] += 1;
      h->k_flops[i] += fl[i];
    }
  }
  return ADC2_OK;
}

}  // namespace adc2

// ---------------------------------------------------------------------------
// Sigma without device allocation: the FP64 sigma build of adc2_sigma with its
// work spaces (X, Y, unpacked doubles, light partials, back-contraction
// partials) carved from one static device array instead of the handle's
// buffers.  The array is a fixed part of the code object, so each device the
// library runs on holds one copy until the process ends; the host reaches it
// only through the address hipGetSymbolAddress returns for the current
// device (the array's own name is a host-side stand-in).
// ---------------------------------------------------------------------------
namespace adc2 {
namespace {
constexpr int NOALLOC_MAX_DEVICES = 64;
}  // namespace
}  // namespace adc2

static __device__ __align__(256) unsigned char scratch[adc2::NOALLOC_SCRATCH_BYTES];

namespace adc2 {

static std::mutex g_scratch_mu;
static void* g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

// Device address of `scratch` on the current device, looked up once per device.
static adc2_status scratch_address(void** out) {
  int dev = 0;
  ADC2_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) {
    set_error("adc2_sigma_noalloc: device index out of range");
    return ADC2_ERR_ARG;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    ADC2_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) {
      set_error("adc2_sigma_noalloc: hipGetSymbolAddress returned NULL");
      return ADC2_ERR_HIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return ADC2_OK;
}

// The plan of a no-allocation sigma: the split counts adc2_sigma would use
// on this handle now (those of its current work spaces when they already
// hold m vectors), so that both give the same result.
static WsPlan noalloc_plan(adc2_handle h, int m) {
  return h->ws_m >= m ? ws_plan(h, m, h->ysplit, h->nsplit) : ws_plan(h, m);
}

static size_t plan_bytes(const WsPlan& p) {
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  return al(p.x) + al(p.y) + al(p.zb) + al(p.tp) + al(p.part);
}

}  // namespace adc2

extern "C" adc2_status adc2_sigma_noalloc(adc2_handle h, int m, const void* X, void* S, void* stream) {
  using namespace adc2;
  if (!h || !X || !S || m <= 0) {
    set_error("adc2_sigma_noalloc: bad arguments");
    return ADC2_ERR_ARG;
  }
  if (X == S) {
    set_error("adc2_sigma_noalloc: S must not alias X");
    return ADC2_ERR_ARG;
  }
  if (h->prec != ADC2_FP64) {
    set_error("adc2_sigma_noalloc: only the FP64 form (the handle is in a precision form)");
    return ADC2_ERR_ARG;
  }
  if (h->method != ADC2_METHOD_ADC2) {
    set_error("adc2_sigma_noalloc: only the ADC(2) matrix (the handle is set to ADC(2)-x)");
    return ADC2_ERR_ARG;
  }
  const WsPlan p = noalloc_plan(h, m);
  const size_t need = plan_bytes(p);
  if (need > NOALLOC_SCRATCH_BYTES) {
    char buf[256];
    snprintf(buf, sizeof buf,
             "adc2_sigma_noalloc: m=%d needs %zu bytes of scratch, above its maximum of %zu bytes "
             "(use adc2_sigma)",
             m, need, NOALLOC_SCRATCH_BYTES);
    set_error(buf);
    return ADC2_ERR_ARG;
  }
  void* base = nullptr;
  adc2_status rc = scratch_address(&base);
  if (rc != ADC2_OK) return rc;
  // point the handle's work spaces into the scratch for this call only; the
  // kernels take these addresses as arguments at launch
  double2 *sX = h->X, *sY = h->Y, *sZb = h->Zb, *sTp = h->Tp, *spart = h->part;
  const int sws = h->ws_m, szb = h->zb_m, sys = h->ysplit, sns = h->nsplit;
  unsigned char* q = static_cast<unsigned char*>(base);
  auto take = [&](size_t b) {
    double2* r = reinterpret_cast<double2*>(q);
    q += (b + 255) & ~size_t(255);
    return r;
  };
  const bool rns = rns_wanted(h, m, true);   // then its own work spaces instead of Zb, in smaller chunks
  char* sws_rns = h->rns_ws;
  const size_t swsb = h->rns_ws_bytes, starget = h->rns_target, sshort = h->rns_short;
  h->X = take(p.x);
  h->Y = take(rns ? p.x : p.y);
  h->Zb = rns ? nullptr : take(p.zb);
  h->Tp = take(p.tp);
  h->part = take(p.part);
  if (rns) {
    h->rns_ws = reinterpret_cast<char*>(q);
    h->rns_lent = true;
    h->rns_short = 0;
    h->rns_target = h->rns_ws_bytes = NOALLOC_SCRATCH_BYTES - (size_t)(q - static_cast<unsigned char*>(base));
  }
  h->ws_m = h->zb_m = m;
  h->ysplit = p.ysplit;
  h->nsplit = p.nsplit;
  const SigReq rq{h, m, static_cast<const double2*>(X), static_cast<double2*>(S), SIGMA_SINGLES_IN | SIGMA_DOUBLES_IN};
  rc = sigma_multi(1, &rq, static_cast<hipStream_t>(stream), rns);
  h->rns_lent = false;
  h->rns_ws = sws_rns;
  h->rns_ws_bytes = swsb;
  h->rns_target = starget;
  h->rns_short = sshort;
  h->X = sX;
  h->Y = sY;
  h->Zb = sZb;
  h->Tp = sTp;
  h->part = spart;
  h->ws_m = sws;
  h->zb_m = szb;
  h->ysplit = sys;
  h->nsplit = sns;
  return rc;
}

