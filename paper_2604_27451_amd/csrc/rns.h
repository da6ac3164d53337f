// rns.h -- complex FP64 matrix products on the INT8 matrix cores of gfx950,
// through residues modulo 16 small moduli.
//
// C[i][j] = sum_k A(k, i) B(k, j) for complex128 A, B.  Each operand row is
// scaled by a power of two, 2^e with ||row|| 2^e <= 2^58.33, and rounded to
// Gaussian integers; the product of two such rows is then a Gaussian integer z
// with |z| <= 2^116.66 (Cauchy-Schwarz), which its residues modulo
// M = prod p_i > 2^117.6 determine.  Every p_i is a product of primes = 1 mod 4,
// so -1 has a square root s_i modulo p_i and the map
//   x + iy -> (x + s_i y, x - s_i y) mod p_i
// turns one complex product into two real ones: 32 real INT8 products
// ("planes") per complex product, exact in INT32 (|residue| <= 121, K <= 2^17).
// The Chinese remainder theorem recovers z.  INT8 MFMA runs at 64 times the
// FP64 MFMA rate, and 32 / 4 = 8 INT8 multiply-adds replace each FP64 one.
//
// Precision.  The integer products are exact.  The errors are the rounding of
// the operands, at most 2^-58.33 ||row|| in the real and the imaginary part of an
// entry (||row|| 2^e lies in (2^57.33, 2^58.33], e being whole), that is about
// 2^-59 ||a|| ||b|| rms in a product whatever K; the FP64 sum of the parts below
// 2^-34 in the recombination, at most 2^-60 ||a|| ||b|| for each K-run; and the final
// rounding to FP64.
//
// A rounding set by the norm of the row is a loss where the large entries of one
// row meet small ones of the other (rows that are graded, or that share only their
// small entries): the FP64 sum is off by about 0.2 2^-53 sqrt(N sum |a_k|^2 |b_k|^2), N
// common terms, which may be far below ||a|| ||b||.  So one more plane holds a code
// of each entry's squared magnitude, 0 for an exact zero, and two products of it, the common
// terms and the sum of the codes' products, bound that from below (rnsconst.h).
// Entries that the integers would hold less well than the FP64 sum, and those of
// rows that are not finite, are formed in FP64 by k_rns_fp64 (which ends at once
// where there are none); which they are depends on the two rows
// and the K-splits alone, not on tiles or chunks.  Rows of like entries are known for that by the
// counts of their codes (rns_class), and tiles of such rows need no product of codes.  What the
// codes cost there: nc=6 no=60 nv=300 naux=1500, ten vectors, 46.1 -> 46.7 ms; the smallest sigma
// 98 -> 108 us.  Cholesky entries spread by a log-normal of half a decade at nc=6 no=45 nv=310 naux=1240,
// seven vectors: 31 ms (even ones 24, the FP64 MFMA engine 59); of a whole decade, where most entries of the product
// need the FP64 sum: 143.
//
// Measured against long double (nc=6 no=60 nv=300 naux=1500, a unit vector on a
// singles entry, so that every doubles entry is one K = 1500 product): rms error
// 1.2e-16 of the rms entry, 2.1e-15 on the FP64 MFMA engine; singles from random
// doubles at nc=6 no=20 nv=100 naux=400: 8.8e-16 against 1.2e-15.
//
// What bounds it.  The product of M=3072, N=9000, K=18000 runs at 2338 TOPS, as 292 TFLOP/s of
// complex products (the FP64 MFMA engine reaches 67); a loop of v_mfma_i32_16x16x64_i8 alone on
// random bytes at 4085, at the power limit (4850 on zeros).  The matrix cores are 60% busy at the clock
// that the limit leaves; what idles them in the rest is not shown.  LDS is the first suspect: four waves
// read 12 KB of fragments each per 32 instructions.
//
// Rows with NaN or Inf give what the FP64 sum gives (NaN against rows of zeros);
// rows of zeros give exact zeros.
#pragma once
#include "internal.h"
#include "rnsconst.h"

namespace adc2 {

constexpr int RNS_PL = 2 * RNS_NM;      // residue planes
constexpr int RNS_NP = RNS_PL + 1;      // planes of an operand: the last one the magnitude codes
constexpr int RNS_OP = RNS_PL + 2;      // planes of a product: the last two of the codes
constexpr int RNS_RT = 128;             // rows per operand block
constexpr int RNS_KC = 64;              // k per operand block
constexpr int RNS_BLK = RNS_RT * RNS_KC;
constexpr long RNS_KMAX = 131072;       // K 121^2 and K 126^2 < 2^31

constexpr int RNS_NAN = 1 << 20;

constexpr int RNS_SPLITS = 32;          // most K-splits of a product

size_t rns_op_bytes(long rows, long K);                 // planes of an operand
size_t rns_exp_bytes(long rows);                        // its exponents, code scales and counts
size_t rns_norm_bytes(long rows);                       // work space of rns_pack
size_t rns_out_bytes(long rows, long cols);             // planes of a product (one K-split)

// Element (row, k) of a strided complex128 operand, conjugated if conj:
//   p[(r / ri) * rg + (r % ri) * rx + (k / ki) * kg + (k % ki) * kx],  r = r0 + row
struct RnsSrc {
  const double2* p;
  int ri;
  long rg, rx;
  int ki;
  long kg, kx;
  bool conj;
  int r0 = 0;
};

// An operand in residues.  Plane q (modulus q / 2, sign q % 2; q = RNS_PL the
// codes), row block rt, k block kc is the 8 KB run at
// ((q * nrt + rt) * nkc + kc) * RNS_BLK, laid out
// [row / 16][k / 16][row % 16][k % 16]: the LDS image of the GEMM, in which a
// 16 x 64 fragment is 1 KB in lane order.
struct RnsMat {
  int8_t* p = nullptr;
  int* e = nullptr;        // row exponents (RNS_NAN: a row that is not finite), then the rows' code scales and counts
  RnsSrc src{};            // the FP64 entries, for what the integers do not serve
  int rows = 0, K = 0, nrt = 0, nkc = 0;
};
// rows x K with unit stride along the rows, k stride ld
inline RnsSrc rns_kmajor(const double2* p, long ld, int K, bool conj = false) {
  return RnsSrc{p, 1 << 30, 0, 1, 1 << 30, 0, ld, conj};
}
// rows x K with unit stride along k, row stride ld
inline RnsSrc rns_rmajor(const double2* p, long ld, bool conj = false) {
  return RnsSrc{p, 1 << 30, 0, ld, 1 << 30, 0, 1, conj};
}
// Where entry (i, j) of a product goes:
//   C[(i' / ii) * ig + (i' % ii) * ix + (j' / ji) * jg + (j' % ji) * jx] = (or +=) alpha v,
// i' = i0 + i, j' = j0 + j
struct RnsDst {
  double2* C;
  int ii;
  long ig, ix;
  int ji;
  long jg, jx;
  double alpha;
  bool add;
  int i0 = 0, j0 = 0;
};
inline RnsDst rns_rows(double2* C, long ldc, double alpha = 1.0, bool add = false) {
  return RnsDst{C, 1 << 30, 0, ldc, 1 << 30, 0, 1, alpha, add};
}

// K-splits of a long product: workgroups that walk 10^5 terms drift apart and lose
// each other's panels in L2; runs of about 9000 keep them together (M=3072, N=1280, K=72000:
// 2074 TOPS in one run, 2282 in eight; no difference at K = 18000).
// (The number of runs decides which residues stand for a sum, and through the FP64 sums of the
// low parts the last bits: it must not depend on the rows and columns of a chunk.  This one
// and that of rns_product come from K, and from the whole M, N and K, so results are the same bits in
// whatever chunks and tiles.)
inline int rns_long_splits(long K) { return K > 20480 ? (int)((K + 9215) / 9216) : 1; }

// Residues of an operand; buf, ebuf and nbuf hold the sizes above.
adc2_status rns_pack(const RnsSrc& src, int rows, int K, int8_t* buf, int* ebuf, double* nbuf, RnsMat* out,
                     hipStream_t st);

// out = residues of the products of the rows of A with the rows [col0,
// col0 + ncols) of B (col0 a multiple of 128) over nsplit runs of K: split s, plane
// q, 32 x 32 block (rb, cb) as a 1 KB run at
// (((s * RNS_OP + q) * nrb + rb) * ncb + cb) * 1024, in MFMA register order.
adc2_status rns_gemm(const RnsMat& A, const RnsMat& B, int col0, int ncols, int nsplit, int8_t* out, hipStream_t st);
// The products themselves out of those residues, and in FP64 from A.src and B.src
// those entries that the integers do not hold well enough, after the others: dst must not overlap
// what A.src and B.src read.
adc2_status rns_join(const RnsMat& A, const RnsMat& B, int col0, int ncols, int nsplit, int8_t* out, const RnsDst& dst,
                     hipStream_t st);

// dst(i, j) = sum_k A(i, k) B(j, k), i < M, j < N, in chunks of rows whose work
// space is at most h->rns_target (or that of one 256 x 128 tile); the entry points
// that use it give that back at their end (rns_tmp_release).  *done = false (nothing written, no error)
// where the caller's own FP64 MFMA kernel, of `rate` flop/s at such sizes, is the
// faster one (rate 0: the caller has asked rns_pays itself) or the memory is
// not to be had: the caller then uses that.
constexpr double RNS_VS_BIG = 60e12;    // 128 x 128 tiles (k_bgemm)
// 64 x 64 tiles (gemm_rr): 25 TFLOP/s from two tiles a CU on, in proportion
// below (0.32 measured on 4 tiles)
inline double rns_vs_tile(long M, long N) {
  const double tiles = (double)((M + 63) / 64) * ((N + 63) / 64);
  return 25e12 * (tiles < 512.0 ? tiles / 512.0 : 1.0);
}
adc2_status rns_product(adc2_handle h, const RnsSrc& A, int M, const RnsSrc& B, int N, int K, const RnsDst& dst,
                        double rate, bool* done, hipStream_t st);
// The size rule of rns_product
bool rns_pays(adc2_handle h, long M, long N, long K, double rate);
// At least `bytes` of the handle's sigma work space, contents undefined; false
// where it is not to be had.
bool rns_reserve(adc2_handle h, size_t bytes);

}  // namespace adc2
