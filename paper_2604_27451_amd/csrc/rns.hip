// rns.hip -- residue engine of the large complex FP64 products (rns.h).
#include <algorithm>
#include <cmath>

#include "rns.h"
#include "tile.h"

namespace adc2 {

typedef int i4v __attribute__((ext_vector_type(4)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));

static inline int rcdiv(long a, long b) { return (int)((a + b - 1) / b); }

__constant__ const RnsConst RNS_C = make_const();

// 2^(2 G) <= M / 2: scaled rows of norm at most 2^G.  G = (log2 M - 1) / 2 less a margin
// for the rounding of the entries (sqrt(2K) / 2 <= 2^8 against 2^58).
constexpr double RNS_G = 58.33;
static_assert(rns_m() > 2.0 * (double)(1L << 58) * (double)(1L << 58) * 1.58, "2 RNS_G = 116.66 bits");

// ---------------------------------------------------------------------------
// sizes
// ---------------------------------------------------------------------------
constexpr int NORM_SPLIT = 64;
constexpr size_t RNS_ROW = sizeof(int) + sizeof(float) + sizeof(unsigned long long);   // e, code scale, code counts of a row
size_t rns_op_bytes(long rows, long K) { return (size_t)RNS_NP * rcdiv(rows, RNS_RT) * rcdiv(K, RNS_KC) * RNS_BLK; }
size_t rns_exp_bytes(long rows) { return RNS_ROW * (size_t)rcdiv(rows, RNS_RT) * RNS_RT; }
size_t rns_norm_bytes(long rows) { return sizeof(double) * 3 * NORM_SPLIT * (size_t)rows; }
// (three bytes a 32 x 32 block more: two for k_rns_join to say whether k_rns_fp64 has entries in it, one for
// k_rns_gemm, of which it uses one a tile, to say whether the tile's rows are flat)
size_t rns_out_bytes(long rows, long cols) { return (size_t)(RNS_OP * 1024 + 3) * rcdiv(rows, 32) * rcdiv(cols, 32); }

// ---------------------------------------------------------------------------
// row exponents
// ---------------------------------------------------------------------------
__device__ __forceinline__ long rns_row(const RnsSrc& s, int row) {
  row += s.r0;
  const int g = row / s.ri;
  return (long)g * s.rg + (long)(row - g * s.ri) * s.rx;
}
__device__ __forceinline__ long rns_k(const RnsSrc& s, int k) {
  const int g = k / s.ki;
  return (long)g * s.kg + (long)(k - g * s.ki) * s.kx;
}

// Three sums of squares, of x, 2^-540 x and 2^540 x, so that no row of finite
// entries overflows or underflows.
struct RnsSums {
  double s[3];
  __device__ __forceinline__ void add(double x) {
    const double b = x * 0x1p-540, t = x * 0x1p540;
    s[0] = fma(x, x, s[0]);
    s[1] = fma(b, b, s[1]);
    s[2] = fma(t, t, s[2]);
  }
};

// Partial sums of squares of the rows, K split over blockIdx.y.  HBM-bound (one
// read of the operand): lane = row where rows are contiguous, a wave per row
// where k is.
// The largest e with ||row|| 2^e <= 2^RNS_G from the row's three sums
// (and the scale of its squared magnitudes in units of 2^64 of the scaled integers', -1 for a zero row and
// 0 for one that is not finite; the counts of its codes start at 0)
__device__ __forceinline__ void rns_exponent(double s0, double s1, double s2, int K, int padded, int row, int* e) {
  double l2;   // log2 of the norm
  if (s0 >= 0x1p-900 && s0 <= 0x1p1000) l2 = 0.5 * log2(s0);
  else if (s0 > 1.0) l2 = 0.5 * log2(s1) + 540.0;   // above 2^500 (Inf where a row is not finite)
  else if (s2 > 0.0) l2 = 0.5 * log2(s2) - 540.0;   // below 2^-450
  else if (s0 == 0.0) l2 = RNS_G;                   // zero row: e = 0
  else l2 = s0;                                     // NaN
  const int ex = isfinite(l2) ? (int)floor(RNS_G - 1e-9 - l2) : RNS_NAN;
  e[row] = ex;
  ((float*)(e + padded))[row] = ex == RNS_NAN ? 0.0f
                                : s0 == 0.0 && s2 == 0.0 ? -1.0f
                                                         : RNS_QMEAN * (float)K * exp2f(64.0f - 2.0f * (float)(l2 + ex));
  ((unsigned long long*)(e + 2 * padded))[row] = 0;
}
// (rows past the end: as zero rows)
__device__ __forceinline__ void rns_no_row(int padded, int row, int* e) {
  e[row] = 0;
  ((float*)(e + padded))[row] = -1.0f;
  ((unsigned long long*)(e + 2 * padded))[row] = 0;
}

__global__ __launch_bounds__(256) void k_rns_norm(const RnsSrc src, int rows, int K, double* __restrict__ part) {
  __shared__ double red[4][3][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = blockIdx.x * 64 + lane;
  const bool ok = row < rows;
  const double2* p = src.p + rns_row(src, ok ? row : 0);
  const int per = (K + gridDim.y - 1) / gridDim.y;
  const int k0 = blockIdx.y * per, k1 = min(K, k0 + per);
  RnsSums t{{0.0, 0.0, 0.0}};
  int k = k0 + w;
  for (; k + 12 < k1; k += 16) {
    double2 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = p[rns_k(src, k + 4 * u)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      t.add(v[u].x);
      t.add(v[u].y);
    }
  }
  for (; k < k1; k += 4) {
    const double2 v = p[rns_k(src, k)];
    t.add(v.x);
    t.add(v.y);
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) red[w][q][lane] = t.s[q];
  __syncthreads();
  if (w < 3 && ok) {
    const double v = (red[0][w][lane] + red[1][w][lane]) + (red[2][w][lane] + red[3][w][lane]);
    part[((long)blockIdx.y * 3 + w) * rows + row] = v;
  }
}

// (one slice: the exponents themselves)
__global__ __launch_bounds__(256) void k_rns_norm_k(const RnsSrc src, int rows, int K, int padded,
                                                    double* __restrict__ part, int* __restrict__ e) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) {
    if (gridDim.y == 1 && lane == 0 && row < padded) rns_no_row(padded, row, e);
    return;
  }
  const double2* p = src.p + rns_row(src, row);
  const int per = (K + gridDim.y - 1) / gridDim.y;
  const int k0 = blockIdx.y * per, k1 = min(K, k0 + per);
  RnsSums t{{0.0, 0.0, 0.0}};
  int k = k0 + lane;
  for (; k + 192 < k1; k += 256) {
    double2 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = p[rns_k(src, k + 64 * u)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      t.add(v[u].x);
      t.add(v[u].y);
    }
  }
  for (; k < k1; k += 64) {
    const double2 v = p[rns_k(src, k)];
    t.add(v.x);
    t.add(v.y);
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    double v = t.s[q];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    t.s[q] = v;
  }
  if (lane != 0) return;
  if (gridDim.y == 1) rns_exponent(t.s[0], t.s[1], t.s[2], K, padded, row, e);
  else
#pragma unroll
    for (int q = 0; q < 3; ++q) part[((long)blockIdx.y * 3 + q) * rows + row] = t.s[q];
}

// e[row]: the largest e with ||row|| 2^e <= 2^RNS_G; rows past the end 0.  A workgroup
// owns 64 rows, its 16 waves share the slices of the norm (one thread a row read up to
// 192 values in turn: 22 us).
__global__ __launch_bounds__(1024) void k_rns_expo(const double* __restrict__ part, int nsplit, int rows, int K,
                                                   int padded, int* __restrict__ e) {
  __shared__ double red[16][3][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int row = blockIdx.x * 64 + lane;
  double s[3] = {0.0, 0.0, 0.0};
  if (row < rows)
#pragma unroll 4
    for (int t = w; t < nsplit; t += 16)
#pragma unroll
      for (int q = 0; q < 3; ++q) s[q] += part[((long)t * 3 + q) * rows + row];
#pragma unroll
  for (int q = 0; q < 3; ++q) red[w][q][lane] = s[q];
  __syncthreads();
  if (w != 0 || row >= padded) return;
  const int nw = nsplit < 16 ? nsplit : 16;
  for (int t = 1; t < nw; ++t)
#pragma unroll
    for (int q = 0; q < 3; ++q) s[q] += red[t][q][lane];
  if (row < rows) rns_exponent(s[0], s[1], s[2], K, padded, row, e);
  else rns_no_row(padded, row, e);
}

// ---------------------------------------------------------------------------
// residues of an operand
// ---------------------------------------------------------------------------
// A thread owns 16 consecutive k of one row: it rounds them to 59-bit signed
// integers, splits these into signed bytes once, and forms both residues for
// each modulus from four 4-byte dot products and a float reduction, and the codes of the
// magnitudes from the upper four bytes; the 16 bytes of a plane are one store, so a wave writes 1 KB runs.  Bound by its
// vector instructions (about 250 per entry) and its 32-byte writes per entry:
// 0.29 ms for the 27 M entries of a 18000 x 1500 operand, 4 TB/s.  Operands
// contiguous along k go through LDS, so that both their reads and the writes
// are whole lines: in two halves of 33 KB, so that four workgroups share a
// compute unit (in one of 66 KB, two of them: 1.84 ms for 128 M entries against
// 1.27 ms).  Grids too short for the chip are split over the moduli
// (blockIdx.y), each part rounding the entries again.
constexpr int RNS_MAGIC = 0x4B400000;   // 1.5 * 2^23 as a float: float(MAGIC + x) = 1.5 * 2^23 + x
template <bool KLANE>
__global__ __launch_bounds__(256, KLANE ? 3 : 5) void k_rns_pack(const RnsSrc src, int rows, int K,
                                                                 int* __restrict__ e, int nrt, int nkc,
                                                                 int8_t* __restrict__ dst) {
  // codes of at least 1, 2 and 3, a byte each here and 21 bits in the row's count (the first to run over,
  // by rows of more than 2^21 terms, is then below its RNS_FLAT: such rows are looked at by their codes)
  __shared__ unsigned cnt[4][64];
  const int lane = threadIdx.x & 63, kg = threadIdx.x >> 6;
  const int rb = blockIdx.x % (2 * nrt), kc = blockIdx.x / (2 * nrt);
  const int row = rb * 64 + lane;
  const int k0 = kc * RNS_KC + kg * 16;
  i4v d[16];   // re lo, re hi, im lo, im hi
  const bool ok = row < rows;
  if constexpr (KLANE) {
    __shared__ double2 t[32][65];
    const int k = kc * RNS_KC + lane;
    const double2* p = src.p + (k < K ? rns_k(src, k) : 0);
    double2 v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = rb * 64 + kg * 16 + r;
      v[r] = (rr < rows && k < K) ? p[rns_row(src, rr)] : make_double2(0.0, 0.0);
    }
    // rows 16 g + r with r < 8, then those with r >= 8
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half) __syncthreads();
#pragma unroll
      for (int r = 0; r < 8; ++r) t[kg * 8 + r][lane] = v[half * 8 + r];
      __syncthreads();
      if (((lane >> 3) & 1) == half)
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const double2 x = t[(lane >> 4) * 8 + (lane & 7)][kg * 16 + u];
          d[u].x = __double2loint(x.x);
          d[u].y = __double2hiint(x.x);
          d[u].z = __double2loint(x.y);
          d[u].w = __double2hiint(x.y);
        }
    }
  } else {
    const double2* p = src.p + rns_row(src, ok ? row : 0);
    int q = k0 / src.ki, r = k0 - q * src.ki;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      double2 v = make_double2(0.0, 0.0);
      if (ok && k0 + u < K) v = p[(long)q * src.kg + (long)r * src.kx];
      if (++r == src.ki) {
        r = 0;
        ++q;
      }
      d[u].x = __double2loint(v.x);
      d[u].y = __double2hiint(v.x);
      d[u].z = __double2loint(v.y);
      d[u].w = __double2hiint(v.y);
    }
  }
  const double cs = src.conj ? -1.0 : 1.0;
  int ex = e[ok ? row : 0];
  if (ex == RNS_NAN) ex = 0;
  const float cw = ((const float*)(e + nrt * RNS_RT))[ok ? row : 0];
  auto digits = [&](double x, int& lo, int& hi) {
    x = rint(ldexp(x, ex));
    // x = h 2^32 + l, |x| < 2^59: exact
    const double h = floor(x * 0x1p-32);
    const double l = fma(h, -0x1p32, x);
    const unsigned long long v = ((unsigned long long)(unsigned)(int)h << 32 | (unsigned)l) + 0x8080808080808080ull;
    lo = (int)((unsigned)v ^ 0x80808080u);
    hi = (int)((unsigned)(v >> 32) ^ 0x80808080u);
  };
  auto top = [](int x) { return (float)(int)(((unsigned)x ^ 0x80808080u) - 0x80808080u); };   // the upper four bytes
  int8_t* out = dst + ((long)(rb >> 1) * nkc + kc) * RNS_BLK + ((rb & 1) * 4 + (lane >> 4)) * 1024 + kg * 256 + (lane & 15) * 16;
  const long ps = (long)nrt * nkc * RNS_BLK;
  int n1 = 0, n2 = 0, n3 = 0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    bool zero[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int u = 4 * t + q;
      const double re = __hiloint2double(d[u].y, d[u].x), im = cs * __hiloint2double(d[u].w, d[u].z);
      zero[q] = (d[u].x | d[u].z | ((d[u].y | d[u].w) & 0x7fffffff)) == 0;
      int a, b;
      digits(re, a, b);
      d[u].x = a;
      d[u].y = b;
      digits(im, a, b);
      d[u].z = a;
      d[u].w = b;
    }
    int cc = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float hr = top(d[4 * t + q].y), hi = top(d[4 * t + q].w);
      const int c = zero[q] ? 0 : 1 + (int)fminf(fmaxf(cw * fmaf(hr, hr, hi * hi), 0.0f), 126.0f);   // NaN: 1
      cc |= c << (8 * q);
    }
    n1 += __popc((cc + 0x7f7f7f7f) & 0x80808080);   // (codes are at most 127: no carry)
    n2 += __popc((cc + 0x7e7e7e7e) & 0x80808080);
    n3 += __popc((cc + 0x7d7d7d7d) & 0x80808080);
    if (blockIdx.y == 0) *(int*)(out + RNS_PL * ps + 4 * t) = cc;
    __builtin_amdgcn_sched_barrier(0);   // (all entries interleaved: 50 registers more)
  }
  const float magic = 12582912.0f;
  cnt[kg][lane] = n1 | n2 << 8 | n3 << 16;
  __syncthreads();
  if (blockIdx.y == 0 && kg == 0 && ok) {
    const unsigned n = cnt[0][lane] + cnt[1][lane] + cnt[2][lane] + cnt[3][lane];   // at most 64 each
    if (n)
      atomicAdd((unsigned long long*)(e + 2 * nrt * RNS_RT) + row,
                (unsigned long long)(n & 255) | (unsigned long long)(n >> 8 & 255) << 21 | (unsigned long long)(n >> 16) << 42);
  }
  const int nq = RNS_NM / gridDim.y;
  for (int q = blockIdx.y * nq; q < (int)(blockIdx.y + 1) * nq; ++q) {
    const RnsSplit c = RNS_C.split[q];
    i4v o0, o1;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      int r0[4], r1[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const i4v x = d[4 * t + u];
        const int tr = __builtin_amdgcn_sdot4(x.x, c.re_lo, __builtin_amdgcn_sdot4(x.y, c.re_hi, RNS_MAGIC, false), false);
        const int ti = __builtin_amdgcn_sdot4(x.z, c.im_lo, __builtin_amdgcn_sdot4(x.w, c.im_hi, 0, false), false);
        const float f0 = __int_as_float(tr + ti), f1 = __int_as_float(tr - ti);
        const float q0 = fmaf(f0 - magic, c.inv, magic) - magic;
        const float q1 = fmaf(f1 - magic, c.inv, magic) - magic;
        r0[u] = __float_as_int(fmaf(-q0, c.p, f0));   // low byte: the balanced residue
        r1[u] = __float_as_int(fmaf(-q1, c.p, f1));
      }
      o0[t] = (int)__builtin_amdgcn_perm(__builtin_amdgcn_perm(r0[3], r0[2], 0x0c0c0400),
                                         __builtin_amdgcn_perm(r0[1], r0[0], 0x0c0c0400), 0x05040100);
      o1[t] = (int)__builtin_amdgcn_perm(__builtin_amdgcn_perm(r1[3], r1[2], 0x0c0c0400),
                                         __builtin_amdgcn_perm(r1[1], r1[0], 0x0c0c0400), 0x05040100);
    }
    *(i4v*)(out + (2 * q) * ps) = o0;
    *(i4v*)(out + (2 * q + 1) * ps) = o1;
  }
}

adc2_status rns_pack(const RnsSrc& src, int rows, int K, int8_t* buf, int* ebuf, double* nbuf, RnsMat* out,
                     hipStream_t st) {
  out->p = buf;
  out->e = ebuf;
  out->src = src;
  out->rows = rows;
  out->K = K;
  out->nrt = rcdiv(rows, RNS_RT);
  out->nkc = rcdiv(K, RNS_KC);
  const bool klane = src.rx != 1 && src.kx == 1;
  // enough blocks to fill the chip, at least 16 (64) k a block
  const int nrow = rcdiv(rows, klane ? 4 : 64);
  const int ns = std::max(1, std::min({NORM_SPLIT, rcdiv(4096, nrow), rcdiv(K, klane ? 64 : 16)}));
  const int padded = out->nrt * RNS_RT;
  if (klane) {
    k_rns_norm_k<<<dim3((unsigned)rcdiv(padded, 4), (unsigned)ns), 256, 0, st>>>(src, rows, K, padded, nbuf, ebuf);
  } else {
    k_rns_norm<<<dim3((unsigned)nrow, (unsigned)ns), 256, 0, st>>>(src, rows, K, nbuf);
  }
  ADC2_CHECK_LAUNCH();
  if (!klane || ns > 1) {
    k_rns_expo<<<rcdiv(padded, 64), 1024, 0, st>>>(nbuf, ns, rows, K, padded, ebuf);
    ADC2_CHECK_LAUNCH();
  }
  const long nblk = (long)2 * out->nrt * out->nkc;
  // a block alone on its compute unit takes 15 us for the 16 moduli, 7 us for 4 of them
  const dim3 grid((unsigned)nblk, nblk <= 256 ? 4 : (nblk <= 512 ? 2 : 1));
  if (klane) k_rns_pack<true><<<grid, 256, 0, st>>>(src, rows, K, ebuf, out->nrt, out->nkc, buf);
  else k_rns_pack<false><<<grid, 256, 0, st>>>(src, rows, K, ebuf, out->nrt, out->nkc, buf);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// ---------------------------------------------------------------------------
// which entries the integers serve (the rule: rnsconst.h)
// ---------------------------------------------------------------------------
struct RnsRows {
  const int* e;      // exponents, then code scales and counts
  int padded, n1, n2, n3;
};
// What is known of a row by the counts of its codes
enum RnsClass { ROW_OTHER, ROW_FULL, ROW_FLAT, ROW_ZERO };   // (full: at least RNS_FLAT[0] of it not zero)
__device__ __forceinline__ int rns_class(const RnsRows& r, int row) {
  const float w = ((const float*)(r.e + r.padded))[row];
  const unsigned long long n = ((const unsigned long long*)(r.e + 2 * r.padded))[row];
  if (w < 0.0f) return ROW_ZERO;
  if (!(w > 0.0f) || (int)(n & 0x1fffff) < r.n1) return ROW_OTHER;
  return (int)(n >> 21 & 0x1fffff) >= r.n2 && (int)(n >> 42) >= r.n3 ? ROW_FLAT : ROW_FULL;
}
static RnsRows rns_rows_of(const RnsMat& m) {
  return RnsRows{m.e, m.nrt * RNS_RT, (int)std::ceil(RNS_FLAT[0] * m.K), (int)std::ceil(RNS_FLAT[1] * m.K),
                 (int)std::ceil(RNS_FLAT[2] * m.K)};
}

// Sums over an entry's K-runs of the two bytes that k_rns_gemm keeps of its code products
struct RnsSpread {
  int terms = 0, part = 0, weight = 0;   // whether there are common terms; their number and sum in units of the bytes
  __device__ __forceinline__ void add(int n, int s) {
    terms |= n;
    part += n ? n - 1 : 0;
    weight += s;
  }
};
__device__ __forceinline__ bool rns_serves(const RnsSpread& s, int a, int b) {
  if (a == ROW_ZERO || b == ROW_ZERO || (a == ROW_FLAT && b == ROW_FLAT)) return true;
  if (a >= ROW_FULL && b >= ROW_FULL) return rns_spread_serves(1, RNS_FULL_PART, s.weight);
  return rns_spread_serves(s.terms, s.part, s.weight);
}
// Of a tile: no code products needed, no count of the common terms needed
constexpr int TILE_FLAT = 1, TILE_FULL = 2;

// ---------------------------------------------------------------------------
// the product of one plane:  C[i][j] = sum_k A[i][k] B[j][k] mod p
// ---------------------------------------------------------------------------
// Tiles of 128 WM x 64 WN on WM WN waves of 128 x 64 (v_mfma_i32_16x16x64_i8,
// 8 x 4 blocks, 128 accumulators a lane).  Chunks of 64 k go from global
// memory straight into an LDS ring of NB stages (the operand layout is the
// LDS image, and a fragment is 1 KB of it in lane order), NB - 1 chunks ahead;
// one barrier a chunk.  On random bytes a loop of this instruction alone runs at 4085 TOPS, of
// 32x32x32 at 3498 (both about 4850 on zeros: there the power limit sets the rate), and the whole product
// at 2240 to 2340 against 1950 to 2050 at K = 18000, 1960 to 1990 against 1710 to 1840 at K = 1500
// (rns.h: what bounds it).  Two workgroups a CU, so that one's reduction runs under the other's products.
template <int WM, int WN, int NB>
__global__ __launch_bounds__(64 * WM * WN, WM * WN == 4 ? 2 : 1) void k_rns_gemm(
    const int8_t* __restrict__ A, const int8_t* __restrict__ B, int nrtA, int nrtB, int brt0, int nkca, int nkcs, int nbm,
    int nbn, int nrb, int ncb, float qs, const RnsRows ra, const RnsRows rb_, int8_t* __restrict__ C) {
  constexpr int BM = 128 * WM, BN = 64 * WN, T = 64 * WM * WN;
  constexpr int SB = (BM + BN) * RNS_KC, NL = SB / (T * 16), NLA = BM * RNS_KC / (T * 16);
  __shared__ __align__(16) int8_t s[NB][SB];
  const long nt = (long)nbm * nbn;
  // planes in order, so that each XCD works on the tiles of few planes, the code products of
  // all splits after them (34 planes in order straddle the XCDs: 1% slower); tiles in
  // groups of 8 row panels
  const long ncode = gridDim.x / RNS_OP * 2, nres = gridDim.x - ncode;
  const bool codes = (long)blockIdx.x >= nres;
  const long lid = codes ? xcd_remap(blockIdx.x - nres, ncode) : xcd_remap(blockIdx.x, nres);
  const int g = (int)(lid / nt);                      // K-split * RNS_PL + plane, 2 * K-split + product of codes
  const int t0 = (int)(lid - (long)g * nt);
  const int po = codes ? RNS_PL + (g & 1) : g % RNS_PL, split = codes ? g >> 1 : g / RNS_PL;
  const int pl = codes ? RNS_PL : po;
  const int sp = split * RNS_OP + po, kc0 = split * nkcs;
  const int nkc = min(nkcs, nkca - kc0);              // chunks of this split
  const int per = 8 * nbn, grp = t0 / per, gm = min(8, nbm - grp * 8), r = t0 - grp * per;
  const int bm = grp * 8 + r % gm, bn = r / gm;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  if (codes) {   // (every wave looks: an LDS reduction beside the ring would have the compiler wait for all
                 // loads before each fragment read)
    int least = ROW_ZERO;
    for (int r = lane; r < BM + BN; r += 64) {
      const bool isa = r < BM;
      const int row = isa ? bm * BM + r : brt0 * RNS_RT + bn * BN + r - BM;
      if (row < (isa ? ra.padded : rb_.padded)) least = min(least, rns_class(isa ? ra : rb_, row));
    }
    const int of = (__ballot(least < ROW_FLAT) == 0 ? TILE_FLAT : 0) | (__ballot(least < ROW_FULL) == 0 ? TILE_FULL : 0);
    if (tid == 0) C[(long)(gridDim.x / nt) * nrb * ncb * 1024 + 2L * nrb * ncb + bm * nbn + bn] = of;
    if (of & (po == RNS_PL ? TILE_FULL : TILE_FLAT)) return;
  }
  // global address of each of this thread's NL pieces of a stage (chunk 0)
  const int8_t* src[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    const int off = (q * T + tid) * 16;
    if (q < NLA) {
      const int rt = min(bm * (BM / RNS_RT) + (off >> 13), nrtA - 1);   // past the end: discarded rows
      src[q] = A + (((long)pl * nrtA + rt) * nkca + kc0) * RNS_BLK + (off & (RNS_BLK - 1));
    } else {
      const int ob = off - BM * RNS_KC;
      const int rt = min(brt0 + bn * (BN / RNS_RT) + (ob >> 13), nrtB - 1);
      src[q] = B + (((long)pl * nrtB + rt) * nkca + kc0) * RNS_BLK + (ob & (RNS_BLK - 1));
    }
  }
  auto load = [&](int t) {
    const long tc = (long)min(t, nkc - 1) * RNS_BLK;
    int8_t* d = s[t % NB];
#pragma unroll
    for (int q = 0; q < NL; ++q)
      __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)(src[q] + tc),
                                       (__attribute__((address_space(3))) void*)(d + (q * T + w * 64) * 16), 16, 0, 0);
  };
  i4v acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = i4v{0, 0, 0, 0};
  const int wm = w % WM, wn = w / WM;
#pragma unroll
  for (int t = 0; t < NB - 1; ++t) load(t);
  auto sweep = [&](auto&& op) {
    for (int t = 0; t < nkc; ++t) {
      // chunk t has landed when at most the NB - 2 later ones are outstanding;
      // the barrier also ends every wave's reads of the stage that load() refills, so
      // these have to have returned (lgkmcnt 0: the products before them need not stay before the barrier)
      constexpr int V = (NB - 2) * NL;
      __builtin_amdgcn_s_waitcnt(0x0070 | (V & 15) | ((V >> 4) << 14));
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      load(t + NB - 1);
      const int8_t* p = s[t % NB];
      const int8_t* pa = p + wm * RNS_BLK + lane * 16;
      const int8_t* pb = p + BM * RNS_KC + (wn >> 1) * RNS_BLK + (wn & 1) * (RNS_BLK / 2) + lane * 16;
      i4v a[8], b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = op(*(const i4v*)(pb + j * 1024));
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] = op(*(const i4v*)(pa + i * 1024));
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };
  // code products: common terms, or codes less one
  auto ones = [](i4v q) { return (i4v)((((u4v)q + 0x7f7f7f7fu) & 0x80808080u) >> 7); };   // (codes are at most 127)
  if (!codes) sweep([](i4v q) { return q; });
  else if (po == RNS_PL) sweep(ones);
  else sweep([&](i4v q) { return q - ones(q); });
  __builtin_amdgcn_s_waitcnt(0x0f70);
  auto each = [&](auto&& byte) {   // the low byte of byte(acc) of every entry
#pragma unroll
    for (int i = 0; i < 4; ++i)   // 32 x 32 blocks: two row blocks, two column blocks
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        i4v o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          int rr[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) rr[x] = byte(acc[2 * i + (q & 1)][2 * j + (q >> 1)][x]);
          o[q] = (int)__builtin_amdgcn_perm(__builtin_amdgcn_perm(rr[3], rr[2], 0x0c0c0400),
                                            __builtin_amdgcn_perm(rr[1], rr[0], 0x0c0c0400), 0x05040100);
        }
        const int rb = (bm * BM + wm * 128) / 32 + i, cb = (bn * BN + wn * 64) / 32 + j;
        if (rb < nrb && cb < ncb) *(i4v*)(C + (((long)sp * nrb + rb) * ncb + cb) * 1024 + lane * 16) = o;
      }
  };
  if (codes) {
    if (po == RNS_PL) each([&](int v) { return rns_terms_byte(v, qs); });
    else each([&](int v) { return rns_weight_byte(v, qs); });
    return;
  }
  const RnsSplit c = RNS_C.split[pl >> 1];
  const int pi = (int)c.p;
  const float magic = 12582912.0f;
  // |acc| <= K 121^2.  Above 4096 k a first step takes off multiples of 1024 p
  // (the float image of acc is then off by up to 64, its quotient by less than
  // one), leaving |x| < 2^18, which the second step reduces to |x| <= p / 2 + 1;
  // up to 4096 k the second step alone ends within 126.
  const bool far = nkc > 64;
  const float invf = c.inv * (1.0f / 1024.0f);
  each([&](int v) {
    if (far) {
      const float t = fmaf((float)v, invf, magic);
      v -= __mul24(__float_as_int(t) - RNS_MAGIC, pi * 1024);
    }
    const float t = fmaf((float)v, c.inv, magic);
    return v - __mul24(__float_as_int(t) - RNS_MAGIC, pi);
  });
}

// 256 x 128 tiles rather than 128 x 256
static bool rns_tall(const RnsMat& A, int ncols, int nsplit) {
  // 256 x 128 or 128 x 256 tiles: the one that pads less, weighed by its rate (256 x
  // 128 is 2% the faster one at K = 1500, the other 1 to 4% from K = 3000 on)
  const double tall = 256.0 * rcdiv(A.rows, 256) * 128.0 * rcdiv(ncols, 128);
  const double flat = 128.0 * rcdiv(A.rows, 128) * 256.0 * rcdiv(ncols, 256) * (rcdiv(A.nkc, nsplit) < 40 ? 1.02 : 0.98);
  return tall <= flat;
}

adc2_status rns_gemm(const RnsMat& A, const RnsMat& B, int col0, int ncols, int nsplit, int8_t* out, hipStream_t st) {
  const int nrb = rcdiv(A.rows, 32), ncb = rcdiv(ncols, 32), nkcs = rcdiv(A.nkc, nsplit);
  const float qs = 1.0f / (float)A.K;
  const RnsRows ra = rns_rows_of(A), rb = rns_rows_of(B);
  if (rns_tall(A, ncols, nsplit)) {
    const int nbm = rcdiv(A.rows, 256), nbn = rcdiv(ncols, 128);
    k_rns_gemm<2, 2, 3><<<(unsigned)((long)nsplit * RNS_OP * nbm * nbn), 256, 0, st>>>(
        A.p, B.p, A.nrt, B.nrt, col0 / RNS_RT, A.nkc, nkcs, nbm, nbn, nrb, ncb, qs, ra, rb, out);
  } else {
    const int nbm = rcdiv(A.rows, 128), nbn = rcdiv(ncols, 256);
    k_rns_gemm<1, 4, 3><<<(unsigned)((long)nsplit * RNS_OP * nbm * nbn), 256, 0, st>>>(
        A.p, B.p, A.nrt, B.nrt, col0 / RNS_RT, A.nkc, nkcs, nbm, nbn, nrb, ncb, qs, ra, rb, out);
  }
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// ---------------------------------------------------------------------------
// recombination
// ---------------------------------------------------------------------------
// A thread recombines 8 entries of one column (two runs of 4 rows): 32 loads
// of 8 bytes, each a 512-byte run of the wave.  Per entry and pair of moduli
// the two weighted residue sums (over the K-splits, at most RNS_SPLITS) are
// exact integers; their multiples of hi are summed exactly in FP64 and reduced
// modulo 1, those of lo added after.  Bound by the 32 bytes read and 16 written
// per entry.
template <bool SPLIT>
__global__ __launch_bounds__(256) void k_rns_join(int8_t* __restrict__ R, int nrb, int ncb, int rows, int cols,
                                                   int nsplit, const RnsRows ra, const RnsRows rb_, int col0,
                                                   int tr, int tc, int nbn, const RnsDst dst) {
  const int ncp = (ncb + 1) >> 1;
  const int rb = blockIdx.x / ncp;
  const int cb = 2 * (blockIdx.x % ncp) + (threadIdx.x >> 7);
  if (cb >= ncb) return;
  const int item = threadIdx.x & 127, lane = item >> 1, half = item & 1;
  const int col = cb * 32 + 16 * half + (lane & 15);
  const int row0 = rb * 32 + 4 * (lane >> 4);   // rows row0 + {0..3} and row0 + 16 + {0..3}
  const long ps = (long)nrb * ncb * 1024;
  const int8_t* src = R + ((long)rb * ncb + cb) * 1024 + item * 8;
  if (col >= cols) return;
  // which entries the integers serve: all of them in a tile of flat rows (tiles of 2^tr x 2^tc blocks)
  const int8_t* fl = R + (long)nsplit * RNS_OP * ps;
  const int of = fl[2L * nrb * ncb + (rb >> tr) * nbn + (cb >> tc)];
  unsigned serve = 255;
  if (!(of & TILE_FLAT)) {
    serve = 0;
    RnsSpread spread[8];
    for (int s = 0; s < nsplit; ++s) {
      int2 n = make_int2(0, 0);
      if (!(of & TILE_FULL)) n = *(const int2*)(src + ((long)s * RNS_OP + RNS_PL) * ps);
      const int2 v = *(const int2*)(src + ((long)s * RNS_OP + RNS_PL + 1) * ps);
#pragma unroll
      for (int x = 0; x < 8; ++x)
        spread[x].add(((x < 4 ? n.x : n.y) >> (8 * (x & 3))) & 255, ((x < 4 ? v.x : v.y) >> (8 * (x & 3))) & 255);
    }
    const int cclass = rns_class(rb_, col0 + col);
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int row = row0 + (x >> 2) * 16 + (x & 3);
      serve |= (unsigned)(row >= rows || rns_serves(spread[x], rns_class(ra, row), cclass)) << x;
    }
  }
  // (lane 0 has the block's first column, which is there)
  const bool any = __ballot(serve != 255) != 0;
  if ((threadIdx.x & 63) == 0)
    R[(long)nsplit * RNS_OP * ps + ((long)rb * ncb + cb) * 2 + (item >> 6)] = any;
  double fr[8], fi[8], gr[8], gi[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) fr[x] = fi[x] = gr[x] = gi[x] = 0.0;
#pragma unroll 2
  for (int t = 0; t < RNS_NM / 2; ++t) {
    int u[4][8];   // residues c+, c- of the two moduli, summed over the splits
    {
      int2 v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = *(const int2*)(src + (4 * t + q) * ps);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int x = 0; x < 8; ++x) u[q][x] = (int)(int8_t)((x < 4 ? v[q].x : v[q].y) >> (8 * (x & 3)));
    }
    if constexpr (SPLIT) {
      for (int s = 1; s < nsplit; ++s) {
        int2 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = *(const int2*)(src + ((long)s * RNS_OP + 4 * t + q) * ps);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int x = 0; x < 8; ++x) u[q][x] += (int)(int8_t)((x < 4 ? v[q].x : v[q].y) >> (8 * (x & 3)));
      }
    }
    const RnsJoin c = RNS_C.join[t];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int yr = __mul24(u[0][x] + u[1][x], c.kre1) + __mul24(u[2][x] + u[3][x], c.kre2);
      const int yi = __mul24(u[0][x] - u[1][x], c.kim1) + __mul24(u[2][x] - u[3][x], c.kim2);
      const double dr = (double)yr, di = (double)yi;
      fr[x] = fma(dr, c.hi, fr[x]);
      gr[x] = fma(dr, c.lo, gr[x]);
      fi[x] = fma(di, c.hi, fi[x]);
      gi[x] = fma(di, c.lo, gi[x]);
    }
  }
  const int* ea = ra.e;
  const int ec = rb_.e[col0 + col];
  constexpr double M = rns_m();
  const int jj = dst.j0 + col, cg = jj / dst.ji;
  double2* pc = dst.C + (long)cg * dst.jg + (long)(jj - cg * dst.ji) * dst.jx;
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int row = row0 + (x >> 2) * 16 + (x & 3);
    if (row >= rows || !(serve >> x & 1)) continue;
    const int er = ea[row];
    double re = M * rns_frac(fr[x], gr[x]), im = M * rns_frac(fi[x], gi[x]);
    if (er == RNS_NAN || ec == RNS_NAN) {
      re = im = __builtin_nan("");
    } else {
      re = ldexp(re, -(er + ec));
      im = ldexp(im, -(er + ec));
    }
    const int i = dst.i0 + row, rg = i / dst.ii;
    double2* o = pc + (long)rg * dst.ig + (long)(i - rg * dst.ii) * dst.ix;
    double2 v = make_double2(dst.alpha * re, dst.alpha * im);
    if (dst.add) v = cadd(*o, v);
    *o = v;
  }
}

// The entries that the integers do not serve, as FP64 sums of the operands' own
// entries, in 64 x 64 tiles on the tile engine of tile.h.  Two workgroups a compute unit take
// them; where the join found none the launch ends after the read of eight bytes a tile (3 us).
// K is not split, so that the sums do not depend on the rows and columns of a call.
template <int MAP_>
struct SrcRns {
  static constexpr int MAP = MAP_;
  RnsSrc s;
  int row0, rows, K;
  __device__ __forceinline__ double2 get(int k, int i) const {
    if (k >= K || row0 + i >= rows) return czero();
    const double2 v = s.p[rns_row(s, row0 + i) + rns_k(s, k)];
    return make_double2(v.x, s.conj ? -v.y : v.y);
  }
};

constexpr int FSEG = 4096;   // chunks looked at together
template <int MAPA, int MAPB>
__global__ __launch_bounds__(256) void k_rns_fp64(const RnsSrc A, const RnsSrc B, int col0, int rows, int cols, int K,
                                                   const int8_t* __restrict__ R, int nrb, int ncb, int nsplit,
                                                   const RnsRows ra, const RnsRows rb_, const int8_t* __restrict__ qa,
                                                   const int8_t* __restrict__ qb, int nkc, int tr, int tc, int nbn,
                                                   const RnsDst dst) {
  __shared__ TileSmem s;
  __shared__ unsigned char own[64][64];
  __shared__ unsigned long long need[FSEG / 64];   // chunks of 16 terms in which both operands have some
  __shared__ unsigned long long todo[4];   // the tiles that have such entries
  const int nct = (ncb + 1) >> 1, ntile = ((nrb + 1) >> 1) * nct;
  const int tid = threadIdx.x, lane = tid & 63;
  const int br = (tid >> 6) & 1, bc = tid >> 7;   // a wave per 32 x 32 block
  const unsigned short* left = (const unsigned short*)(R + (long)nsplit * RNS_OP * nrb * ncb * 1024);
  for (int t0 = blockIdx.x; t0 < ntile; t0 += 256 * gridDim.x) {   // a thread looks at one tile of up to 256
    const int tt = t0 + tid * gridDim.x, b0 = (tt / nct) * 2, c0 = (tt % nct) * 2;
    unsigned any = 0;
    if (tt < ntile)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (b0 + (q & 1) < nrb && c0 + (q >> 1) < ncb) any |= left[(b0 + (q & 1)) * (long)ncb + c0 + (q >> 1)];
    const unsigned long long m = __ballot(any != 0);
    if (lane == 0) todo[tid >> 6] = m;
    __syncthreads();
    for (int w = 0; w < 4; ++w)
      for (unsigned long long t = todo[w]; t; t &= t - 1) {
        const int tile = t0 + (w * 64 + __builtin_ctzll(t)) * gridDim.x;
        const int i0 = (tile / nct) * 64, j0 = (tile % nct) * 64, rb = i0 / 32 + br, cb = j0 / 32 + bc;
        RnsSpread spread[16];
        if (rb < nrb && cb < ncb) {
          const bool full = (((const int8_t*)left)[2L * nrb * ncb + (rb >> tr) * nbn + (cb >> tc)] & TILE_FULL) != 0;
          for (int q = 0; q < nsplit; ++q) {
            const int8_t* c = R + ((((long)q * RNS_OP + RNS_PL) * nrb + rb) * ncb + cb) * 1024 + lane * 16;
            const i4v n = full ? i4v{0, 0, 0, 0} : *(const i4v*)c, v = *(const i4v*)(c + (long)nrb * ncb * 1024);
#pragma unroll
            for (int x = 0; x < 16; ++x) spread[x].add((n[x >> 2] >> (8 * (x & 3))) & 255, (v[x >> 2] >> (8 * (x & 3))) & 255);
          }
        }
#pragma unroll
        for (int x = 0; x < 16; ++x) {   // register order of the 16 x 16 blocks of k_rns_gemm
          const int q = x >> 2, r = 32 * br + 16 * (q & 1) + 4 * (lane >> 4) + (x & 3);
          const int c = 32 * bc + 16 * (q >> 1) + (lane & 15);
          own[r][c] = (unsigned char)(i0 + r < rows && j0 + c < cols &&
                                      !rns_serves(spread[x], rns_class(ra, i0 + r), rns_class(rb_, col0 + j0 + c)));
        }
        // Chunks in which one operand has no term of the tile are left out: they add exact zeros, unless a row is
        // not finite (nc=6 no=60 nv=300, a folded solve from singles guesses: 128 -> 81 ms of 2.6 s, its first
        // products being of rows with 60 terms in 18000).
        const int ja = i0 + tid, jb = col0 + j0 + tid - 64;
        const bool bad = tid < 64 ? ja < rows && ra.e[ja] == RNS_NAN : tid < 128 && jb < col0 + cols && rb_.e[jb] == RNS_NAN;
        const bool all = __syncthreads_or(bad) != 0;
        const SrcRns<MAPA> sa{A, i0, rows, K};
        const SrcRns<MAPB> sb{B, col0 + j0, col0 + cols, K};
        Acc acc;
        acc.zero();
        const int nch = (K + TK - 1) / TK;
        for (int h0 = 0; h0 < nch; h0 += FSEG) {
          const int nh = min(FSEG, nch - h0);
          for (int h = (tid >> 6) * 64; h < nh; h += 256) {   // a wave per 64 chunks
            unsigned long long bits = 0;
            if (all) bits = ~0ull;
            else
#pragma unroll 4
              for (int c = 0; c < 64; ++c) {
                const int ch = min(h0 + h + c, 4 * nkc - 1);
                const long o = (long)(ch >> 2) * RNS_BLK + (lane >> 4) * 1024 + (ch & 3) * 256 + (lane & 15) * 16;
                const i4v x = *(const i4v*)(qa + ((long)(i0 >> 7) * nkc) * RNS_BLK + ((i0 >> 6) & 1) * 4096 + o);
                const i4v y = *(const i4v*)(qb + ((long)((col0 + j0) >> 7) * nkc) * RNS_BLK + (((col0 + j0) >> 6) & 1) * 4096 + o);
                const bool both = __ballot((x[0] | x[1] | x[2] | x[3]) != 0) && __ballot((y[0] | y[1] | y[2] | y[3]) != 0);
                bits |= (unsigned long long)both << c;
              }
            if (nh - h < 64) bits &= (1ull << (nh - h)) - 1;
            if (lane == 0) need[h >> 6] = bits;
          }
          __syncthreads();
          int wd = 0;
          unsigned long long bits = need[0];
          auto next = [&]() {   // the next such chunk, or -1 (the same in every thread)
            while (bits == 0) {
              if (++wd >= (nh + 63) >> 6) return -1;
              bits = need[wd];
            }
            const int c = __builtin_ctzll(bits);
            bits &= bits - 1;
            return h0 + wd * 64 + c;
          };
          Regs va, vb;
          int ch = next();
          if (ch >= 0) {
            fetch(sa, ch * TK, va, tid);
            fetch(sb, ch * TK, vb, tid);
          }
          while (ch >= 0) {
            __syncthreads();
            stash<MAPA>(s.a_re, s.a_im, va, tid);
            stash<MAPB>(s.b_re, s.b_im, vb, tid);
            __syncthreads();
            ch = next();
            if (ch >= 0) {
              fetch(sa, ch * TK, va, tid);
              fetch(sb, ch * TK, vb, tid);
            }
            mma_chunk(s, acc, Acc::row0(tid >> 6), Acc::col0(tid >> 6), lane);
          }
          __syncthreads();   // need is free
        }
        for_each_acc(acc, [&](int r, int c, double2 v) {
          if (!own[r][c]) return;
          const int i = dst.i0 + i0 + r, rg = i / dst.ii, j = dst.j0 + j0 + c, cg = j / dst.ji;
          double2* o = dst.C + (long)rg * dst.ig + (long)(i - rg * dst.ii) * dst.ix + (long)cg * dst.jg +
                       (long)(j - cg * dst.ji) * dst.jx;
          double2 u = cscale(v, dst.alpha);
          if (dst.add) u = cadd(*o, u);
          *o = u;
        });
        __syncthreads();   // own and s are free
      }
    __syncthreads();   // todo is free
  }
}

adc2_status rns_join(const RnsMat& A, const RnsMat& B, int col0, int ncols, int nsplit, int8_t* out, const RnsDst& dst,
                     hipStream_t st) {
  const int nrb = rcdiv(A.rows, 32), ncb = rcdiv(ncols, 32);
  const unsigned nblk = (unsigned)((long)nrb * ((ncb + 1) / 2));
  const RnsRows ra = rns_rows_of(A), rb = rns_rows_of(B);
  const bool tall = rns_tall(A, ncols, nsplit);
  const int tr = tall ? 3 : 2, tc = tall ? 2 : 3, nbn = rcdiv(ncols, tall ? 128 : 256);
  if (nsplit > 1)
    k_rns_join<true><<<nblk, 256, 0, st>>>(out, nrb, ncb, A.rows, ncols, nsplit, ra, rb, col0, tr, tc, nbn, dst);
  else
    k_rns_join<false><<<nblk, 256, 0, st>>>(out, nrb, ncb, A.rows, ncols, 1, ra, rb, col0, tr, tc, nbn, dst);
  ADC2_CHECK_LAUNCH();
  const unsigned ntile = (unsigned)std::min<long>(512, (long)((nrb + 1) / 2) * ((ncb + 1) / 2));
  const int8_t *qa = A.p + (long)RNS_PL * A.nrt * A.nkc * RNS_BLK, *qb = B.p + (long)RNS_PL * B.nrt * B.nkc * RNS_BLK;
#define RNS_FP64(MA_, MB_)                                                                                        \
  k_rns_fp64<MA_, MB_><<<ntile, 256, 0, st>>>(A.src, B.src, col0, A.rows, ncols, A.K, out, nrb, ncb, nsplit, ra, rb, qa, \
                                              qb, A.nkc, tr, tc, nbn, dst)
  const bool ak = A.src.rx == 1, bk = B.src.rx == 1;   // contiguous along the rows
  if (ak && bk) RNS_FP64(KMAJOR, KMAJOR);
  else if (ak) RNS_FP64(KMAJOR, RMAJOR);
  else if (bk) RNS_FP64(RMAJOR, KMAJOR);
  else RNS_FP64(RMAJOR, RMAJOR);
#undef RNS_FP64
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// ---------------------------------------------------------------------------
// general products
// ---------------------------------------------------------------------------
// Where the conversions pay: per term of the product 8 / 225e12 s against 8 / rate
// on the FP64 MFMA kernel, per operand entry 1.25e-11 s (norm and residues), per
// output entry 1e-11 s; about 60 us of
// launches and part-filled rounds.
bool rns_pays(adc2_handle h, long M, long N, long K, double rate) {
  if (h->rns_mode == RNS_ALWAYS) return K <= RNS_KMAX * RNS_SPLITS;
  if (h->rns_mode == RNS_NEVER || K > RNS_KMAX * RNS_SPLITS) return false;
  const double terms = (double)M * N * K;
  const double padded = 256.0 * rcdiv(M, 256) * 128.0 * rcdiv(N, 128) * K;
  const double rns = 6e-5 + padded * 8 / 225e12 + 1.25e-11 * ((double)M * K + (double)N * K) + 1e-11 * (double)M * N;
  return rns < 0.85 * terms * 8 / rate;
}

static bool rns_grow(adc2_handle h, char** buf, size_t* have, size_t bytes) {
  if (*have >= bytes) return true;
  if (h->rns_lent) return false;
  if (bytes > (size_t(256) << 20)) bytes = (bytes + (size_t(512) << 20) - 1) >> 29 << 29;   // few sizes: blocks are reused
  char* old = *buf;
  *buf = nullptr;
  *have = 0;
  dfree(h, old);
  const hipError_t e = dmalloc_try(h, reinterpret_cast<void**>(buf), bytes);
  if (e == hipSuccess) {
    *have = bytes;
    return true;
  }
  (void)hipGetLastError();
  return false;
}

bool rns_reserve(adc2_handle h, size_t bytes) {
  return rns_grow(h, &h->rns_ws, &h->rns_ws_bytes, bytes);
}

void rns_tmp_release(adc2_handle h) {
  char* t = h->rns_tmp;
  h->rns_tmp = nullptr;
  h->rns_tmp_bytes = 0;
  dfree(h, t);
}

void rns_scratch_release(adc2_handle h) {
  char* c = h->rns_ws;
  h->rns_ws = nullptr;
  h->rns_ws_bytes = 0;
  dfree(h, c);
  rns_tmp_release(h);
}

void rns_release(adc2_handle h) {
  char *a = h->rns_lvo, *b = h->rns_lvt;
  h->rns_lvo = h->rns_lvt = nullptr;
  dfree(h, a);
  dfree(h, b);
  rns_scratch_release(h);
}

adc2_status rns_product(adc2_handle h, const RnsSrc& A, int M, const RnsSrc& B, int N, int K, const RnsDst& dst,
                        double rate, bool* done, hipStream_t st) {
  *done = false;
  if (M <= 0 || N <= 0 || K <= 0 || (rate > 0.0 && !rns_pays(h, M, N, K, rate))) return ADC2_OK;
  // K-splits: within the INT32 range (RNS_KMAX a split), and enough tiles for two a CU
  const long tiles = (long)RNS_PL * rcdiv(M, 256) * rcdiv(N, 128);
  const int nkc = rcdiv(K, RNS_KC);
  int ns = std::max(std::max(rcdiv(K, RNS_KMAX), std::min(rns_long_splits(K), RNS_SPLITS)), (int)std::min<long>({(long)RNS_SPLITS, (1024 + tiles - 1) / tiles, std::max(1, nkc / 8)}));
  ns = rcdiv(nkc, rcdiv(nkc, ns));   // no empty split
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  auto need = [&](long m, long n) {
    return al(rns_op_bytes(m, K)) + al(rns_op_bytes(n, K)) + al(rns_out_bytes(m, n) * ns) + al(rns_exp_bytes(m)) +
           al(rns_exp_bytes(n)) + al(rns_norm_bytes(std::max(m, n)));
  };
  long mc = M, nc = N;
  while (need(mc, nc) > h->rns_target && (mc > 256 || nc > 128)) {
    if (mc > 256 && (mc >= nc || nc <= 128)) mc = (mc / 2 + 255) / 256 * 256;
    else nc = (nc / 2 + 127) / 128 * 128;
  }
  if (!rns_grow(h, &h->rns_tmp, &h->rns_tmp_bytes, need(mc, nc))) return ADC2_OK;
  char* q = h->rns_tmp;
  auto take = [&](size_t b) {
    char* r = q;
    q += al(b);
    return r;
  };
  int8_t* ap = (int8_t*)take(rns_op_bytes(mc, K));
  int8_t* bp = (int8_t*)take(rns_op_bytes(nc, K));
  int8_t* out = (int8_t*)take(rns_out_bytes(mc, nc) * ns);
  int* ae = (int*)take(rns_exp_bytes(mc));
  int* be = (int*)take(rns_exp_bytes(nc));
  double* nrm = (double*)take(rns_norm_bytes(std::max(mc, nc)));
  auto rows_from = [](RnsSrc s, long r0) {   // the operand from row r0 on
    s.r0 += (int)r0;
    return s;
  };
  *done = true;
  RnsMat am, bm;
  adc2_status rc;
  for (long n0 = 0; n0 < N; n0 += nc) {
    const int n = (int)std::min<long>(nc, N - n0);
    if ((rc = rns_pack(rows_from(B, n0), n, K, bp, be, nrm, &bm, st)) != ADC2_OK) return rc;
    for (long m0 = 0; m0 < M; m0 += mc) {
      const int m = (int)std::min<long>(mc, M - m0);
      if ((n0 == 0 || mc < M) && (rc = rns_pack(rows_from(A, m0), m, K, ap, ae, nrm, &am, st)) != ADC2_OK) return rc;
      RnsDst o = dst;
      o.i0 += (int)m0;
      o.j0 += (int)n0;
      if ((rc = rns_gemm(am, bm, 0, n, ns, out, st)) != ADC2_OK) return rc;
      if ((rc = rns_join(am, bm, 0, n, ns, out, o, st)) != ADC2_OK) return rc;
    }
  }
  return ADC2_OK;
}

}  // namespace adc2
