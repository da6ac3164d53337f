// rns.h -- complex FP64 matrix products on the INT8 matrix cores of gfx950,
// through residues modulo 16 small moduli.
//
// C[i][j] = sum_k A(k, i) B(k, j) for complex128 A, B.  Each operand row is
// scaled by a power of two, 2^e with ||row|| 2^e <= 2^58, and rounded to
// Gaussian integers; the product of two such rows is then a Gaussian integer z
// with |z| <= 2^116 (Cauchy-Schwarz), which its residues modulo
// M = prod p_i > 2^117 determine.  Every p_i is a product of primes = 1 mod 4,
// so -1 has a square root s_i modulo p_i and the map
//   x + iy -> (x + s_i y, x - s_i y) mod p_i
// turns one complex product into two real ones: 32 real INT8 products
// ("planes") per complex product, exact in INT32 (|residue| <= 121, K <= 2^17).
// The Chinese remainder theorem recovers z.  INT8 MFMA runs at 64 times the
// FP64 MFMA rate, and 32 / 4 = 8 INT8 multiply-adds replace each FP64 one.
//
// Precision.  The integer products are exact, so the only errors are the
// rounding of the operands, at most 2^-58 ||row|| sqrt(1/2) per entry (for rows
// of K like entries 2^-58 sqrt(2K) of an entry), and the final rounding to
// FP64.  Normwise this is below the accumulation error of the FP64 matrix
// cores at every K (the error per product is sqrt(K) 2^-58 ||a|| ||b||, that
// of a K-term FP64 sum of random signs about 0.2 sqrt(K) 2^-53 |a.b|).  The
// result does not depend on tiles, chunks or the order of summation.
//
// Measured against long double (nc=6 no=60 nv=300 naux=1500, a unit vector on a
// singles entry, so that every doubles entry is one K = 1500 product): rms error
// 1.2e-16 of the rms entry, 2.1e-15 on the FP64 MFMA engine; singles from random
// doubles at nc=6 no=20 nv=100 naux=400: 8.8e-16 against 1.2e-15.
//
// What bounds it.  The INT8 products draw the card to its power limit: a
// loop of v_mfma_i32_32x32x32_i8 on random bytes alone runs at 3047 TOPS (4320 on
// zeros), the product of M=1500, N=K=18000 at 1914 (2800 on zeros), as 239
// TFLOP/s of complex products; the FP64 MFMA engine reaches 67.
// One 10-vector sigma at nc=6 no=60 nv=300 naux=1500: 124.8 ms before, 56.5 ms so.
//
// Rows with NaN or Inf give NaN in every product with them; rows of zeros
// give exact zeros.
#pragma once
#include "internal.h"

namespace adc2 {

constexpr int RNS_NM = 16;              // moduli
constexpr int RNS_PL = 2 * RNS_NM;      // planes
constexpr int RNS_RT = 128;             // rows per operand block
constexpr int RNS_KC = 64;              // k per operand block
constexpr int RNS_BLK = RNS_RT * RNS_KC;
constexpr long RNS_KMAX = 131072;       // K 121^2 < 2^31

// An operand in residues.  Plane q (modulus q / 2, sign q % 2), row block rt,
// k block kc is the 8 KB run at ((q * nrt + rt) * nkc + kc) * RNS_BLK, laid
// out [k / 16][row][k % 16], which is both the LDS image of the GEMM and
// conflict-free for its 16-byte fragment reads.
struct RnsMat {
  int8_t* p = nullptr;
  int* e = nullptr;        // row exponents (RNS_NAN: a row that is not finite)
  int rows = 0, K = 0, nrt = 0, nkc = 0;
};
constexpr int RNS_NAN = 1 << 20;

size_t rns_op_bytes(long rows, long K);                 // planes of an operand
size_t rns_exp_bytes(long rows);                        // its exponents
size_t rns_norm_bytes(long rows);                       // work space of rns_pack
size_t rns_out_bytes(long rows, long cols);             // planes of a product

// Residues of the K-major operand with element (k, row) at
// src[(row / inner) * gstride + (row % inner) + k * ld]; conj negates the
// imaginary parts.  buf, ebuf and nbuf hold the sizes above.
adc2_status rns_pack(const double2* src, long gstride, long ld, int inner, int rows, int K, bool conj,
                     int8_t* buf, int* ebuf, double* nbuf, RnsMat* out, hipStream_t st);

// out = residues of A^T B for the rows [col0, col0 + ncols) of B (col0 a
// multiple of 128): plane q, 32 x 32 block (rb, cb) as a 1 KB run at
// ((q * nrb + rb) * ncb + cb) * 1024, in MFMA register order.
adc2_status rns_gemm(const RnsMat& A, const RnsMat& B, int col0, int ncols, int8_t* out, hipStream_t st);

// The sigma build's two products out of those residues, rows x cols of out
//   Z: rows (g, a), a < nv, columns (j, b), b < nv:  Z[((g * no + j) * nv + a) * nv + b]
//   Y: rows P, columns (g, c):                        Y[(g * naux + P) * nv + c]
adc2_status rns_to_z(const RnsMat& A, const RnsMat& B, const int8_t* out, int no, int nv, double2* Z, hipStream_t st);
adc2_status rns_to_y(const RnsMat& A, const RnsMat& B, const int8_t* out, int naux, int nv, double2* Y,
                     hipStream_t st);
// Row-major C[i * ldc + j]
adc2_status rns_to_rows(const RnsMat& A, const RnsMat& B, int col0, int ncols, const int8_t* out, double2* C, long ldc,
                        hipStream_t st);

}  // namespace adc2
