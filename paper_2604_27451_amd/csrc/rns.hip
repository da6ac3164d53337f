// rns.hip -- residue engine of the large complex FP64 products (rns.h).
#include <algorithm>
#include <cmath>

#include "rns.h"
#include "tile.h"

namespace adc2 {

typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i16v __attribute__((ext_vector_type(16)));

static inline int rcdiv(long a, long b) { return (int)((a + b - 1) / b); }

// ---------------------------------------------------------------------------
// constants of the moduli
// ---------------------------------------------------------------------------
// Pairwise coprime products of primes = 1 mod 4 below 2^8 (221 = 13 * 17,
// 205 = 5 * 41): the sixteen of largest product, log2 M = 117.7.
constexpr int RNS_P[RNS_NM] = {241, 233, 229, 221, 205, 197, 193, 181, 173, 157, 149, 137, 113, 109, 101, 97};

constexpr int cmod(long a, int p) { return (int)(((a % p) + p) % p); }
constexpr int balanced(long a, int p) {
  const int r = cmod(a, p);
  return r > p / 2 ? r - p : r;
}
constexpr int inverse(long a, int p) {
  for (int x = 1; x < p; ++x)
    if (cmod(a * x, p) == 1) return x;
  return 0;
}
constexpr int sqrt_m1(int p) {
  for (int x = 1; x < p; ++x)
    if (cmod((long)x * x, p) == p - 1) return x;
  return 0;
}

// Split of an operand's scaled integers: v = sum_k d_k 256^k with signed bytes
// d_k, so v mod p = sum_k d_k (256^k mod p): two 4-byte dot products.
struct RnsSplit {
  int re_lo, re_hi;    // bytes 256^k mod p
  int im_lo, im_hi;    // bytes s 256^k mod p
  float p, inv;
};
// Recombination of the moduli 2t and 2t + 1: with u = c+ + c- and w = c+ - c-,
//   re / M = sum (u_1 kre1 + u_2 kre2) / (p1 p2) mod 1,  im / M the same with w, kim.
struct RnsJoin {
  int kre1, kre2, kim1, kim2;
  double hi, lo;       // 1 / (p1 p2) = hi + lo, hi a multiple of 2^-38
};
struct RnsConst {
  RnsSplit split[RNS_NM];
  RnsJoin join[RNS_NM / 2];
};

constexpr RnsConst make_const() {
  RnsConst c{};
  for (int q = 0; q < RNS_NM; ++q) {
    const int p = RNS_P[q], s = sqrt_m1(p);
    unsigned r[2] = {0, 0}, m[2] = {0, 0};
    long w = 1;
    for (int k = 0; k < 8; ++k) {
      r[k / 4] |= (unsigned)(balanced(w, p) & 255) << (8 * (k % 4));
      m[k / 4] |= (unsigned)(balanced(w * s, p) & 255) << (8 * (k % 4));
      w = (w * 256) % p;
    }
    c.split[q].re_lo = (int)r[0];
    c.split[q].re_hi = (int)r[1];
    c.split[q].im_lo = (int)m[0];
    c.split[q].im_hi = (int)m[1];
    c.split[q].p = (float)p;
    c.split[q].inv = 1.0f / (float)p;
  }
  for (int t = 0; t < RNS_NM / 2; ++t) {
    int kre[2] = {0, 0}, kim[2] = {0, 0};
    for (int h = 0; h < 2; ++h) {
      const int q = 2 * t + h, p = RNS_P[q], s = sqrt_m1(p);
      long mp = 1;     // M / p mod p
      for (int j = 0; j < RNS_NM; ++j)
        if (j != q) mp = (mp * RNS_P[j]) % p;
      const long ti = inverse(mp, p);
      kre[h] = balanced(ti * inverse(2, p), p);
      kim[h] = balanced(ti * inverse(2 * s, p), p);
    }
    const int p1 = RNS_P[2 * t], p2 = RNS_P[2 * t + 1];
    const long pp = (long)p1 * p2, one = 1L << 38;
    const long n = (one + pp / 2) / pp;
    c.join[t].kre1 = kre[0] * p2;
    c.join[t].kre2 = kre[1] * p1;
    c.join[t].kim1 = kim[0] * p2;
    c.join[t].kim2 = kim[1] * p1;
    c.join[t].hi = (double)n / (double)one;
    c.join[t].lo = (double)(one - n * pp) / (double)pp / (double)one;
  }
  return c;
}
__constant__ const RnsConst RNS_C = make_const();

constexpr double rns_m() {
  double m = 1.0;
  for (int q = 0; q < RNS_NM; ++q) m *= RNS_P[q];
  return m;
}
// 2^(2 G) <= M / 2: scaled rows of norm at most 2^G.  G = (log2 M - 1) / 2 less a margin
// for the rounding of the entries (sqrt(2K) / 2 <= 2^8 against 2^58).
constexpr double RNS_G = 58.33;
static_assert(rns_m() > 2.0 * (double)(1L << 58) * (double)(1L << 58) * 1.58, "2 RNS_G = 116.66 bits");

// ---------------------------------------------------------------------------
// sizes
// ---------------------------------------------------------------------------
constexpr int NORM_SPLIT = 64;
size_t rns_op_bytes(long rows, long K) { return (size_t)RNS_PL * rcdiv(rows, RNS_RT) * rcdiv(K, RNS_KC) * RNS_BLK; }
size_t rns_exp_bytes(long rows) { return sizeof(int) * (size_t)rcdiv(rows, RNS_RT) * RNS_RT; }
size_t rns_norm_bytes(long rows) { return sizeof(double) * 3 * NORM_SPLIT * (size_t)rows; }
size_t rns_out_bytes(long rows, long cols) { return (size_t)RNS_PL * rcdiv(rows, 32) * rcdiv(cols, 32) * 1024; }

// ---------------------------------------------------------------------------
// row exponents
// ---------------------------------------------------------------------------
// Partial sums of squares of the rows, lane = row (coalesced), K split over
// blockIdx.y.  Three sums, of x, 2^-540 x and 2^540 x, so that no row of
// finite entries overflows or underflows.  HBM-bound (one read of the operand).
__global__ __launch_bounds__(256) void k_rns_norm(const double2* __restrict__ src, long gstride, long ld, int inner,
                                                   int rows, int K, double* __restrict__ part) {
  __shared__ double red[4][3][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int row = blockIdx.x * 64 + lane;
  const bool ok = row < rows;
  const int rr = ok ? row : 0;
  const int g = rr / inner;
  const double2* p = src + (long)g * gstride + (rr - g * inner);
  const int per = (K + gridDim.y - 1) / gridDim.y;
  const int k0 = blockIdx.y * per, k1 = min(K, k0 + per);
  const double big = 0x1p-540, small = 0x1p540;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  auto add = [&](double x) {
    s0 = fma(x, x, s0);
    const double b = x * big, t = x * small;
    s1 = fma(b, b, s1);
    s2 = fma(t, t, s2);
  };
  int k = k0 + w;
  for (; k + 12 < k1; k += 16) {
    double2 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = p[(long)(k + 4 * u) * ld];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      add(v[u].x);
      add(v[u].y);
    }
  }
  for (; k < k1; k += 4) {
    const double2 v = p[(long)k * ld];
    add(v.x);
    add(v.y);
  }
  red[w][0][lane] = s0;
  red[w][1][lane] = s1;
  red[w][2][lane] = s2;
  __syncthreads();
  if (w < 3 && ok) {
    const double t = (red[0][w][lane] + red[1][w][lane]) + (red[2][w][lane] + red[3][w][lane]);
    part[((long)blockIdx.y * 3 + w) * rows + row] = t;
  }
}

// e[row]: the largest e with ||row|| 2^e <= 2^RNS_G; rows past the end 0.
__global__ void k_rns_expo(const double* __restrict__ part, int nsplit, int rows, int padded, int* __restrict__ e) {
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= padded) return;
  int ex = 0;
  if (row < rows) {
    double s[3] = {0.0, 0.0, 0.0};
    for (int t = 0; t < nsplit; ++t)
      for (int q = 0; q < 3; ++q) s[q] += part[((long)t * 3 + q) * rows + row];
    double l2;   // log2 of the norm
    if (s[0] >= 0x1p-900 && s[0] <= 0x1p1000) l2 = 0.5 * log2(s[0]);
    else if (s[0] > 1.0) l2 = 0.5 * log2(s[1]) + 540.0;   // above 2^500 (Inf where a row is not finite)
    else if (s[2] > 0.0) l2 = 0.5 * log2(s[2]) - 540.0;   // below 2^-450
    else if (s[0] == 0.0) l2 = RNS_G;                      // zero row: e = 0
    else l2 = s[0];                                        // NaN
    ex = isfinite(l2) ? (int)floor(RNS_G - 1e-9 - l2) : RNS_NAN;
  }
  e[row] = ex;
}

// ---------------------------------------------------------------------------
// residues of an operand
// ---------------------------------------------------------------------------
// A thread owns 16 consecutive k of one row: it rounds them to 59-bit signed
// integers, splits these into signed bytes once, and forms both residues for
// each modulus from four 4-byte dot products and a float reduction; the 16
// bytes of a plane are one store, so a wave writes 1 KB runs.  Bound by its
// vector instructions (about 250 per entry) and its 32-byte writes per entry.
constexpr int RNS_MAGIC = 0x4B400000;   // 1.5 * 2^23 as a float: float(MAGIC + x) = 1.5 * 2^23 + x
__global__ __launch_bounds__(256) void k_rns_pack(const double2* __restrict__ src, long gstride, long ld, int inner,
                                                   int rows, int K, double cs, const int* __restrict__ e, int nrt,
                                                   int nkc, int8_t* __restrict__ dst) {
  const int lane = threadIdx.x & 63, kg = threadIdx.x >> 6;
  const int rb = blockIdx.x % (2 * nrt), kc = blockIdx.x / (2 * nrt);
  const int row = rb * 64 + lane;
  const int k0 = kc * RNS_KC + kg * 16;
  i4v d[16];   // re lo, re hi, im lo, im hi
  const bool ok = row < rows;
  const int rr = ok ? row : 0;
  const int g = rr / inner;
  const double2* p = src + (long)g * gstride + (rr - g * inner);
  int ex = e[rr];
  if (ex == RNS_NAN) ex = 0;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    double2 v = make_double2(0.0, 0.0);
    if (ok && k0 + u < K) v = p[(long)(k0 + u) * ld];
    d[u].x = __double2loint(v.x);
    d[u].y = __double2hiint(v.x);
    d[u].z = __double2loint(v.y);
    d[u].w = __double2hiint(v.y);
  }
  auto digits = [&](double x, int& lo, int& hi) {
    x = rint(ldexp(x, ex));
    // x = h 2^32 + l, |x| < 2^59: exact
    const double h = floor(x * 0x1p-32);
    const double l = fma(h, -0x1p32, x);
    const unsigned long long v = ((unsigned long long)(unsigned)(int)h << 32 | (unsigned)l) + 0x8080808080808080ull;
    lo = (int)((unsigned)v ^ 0x80808080u);
    hi = (int)((unsigned)(v >> 32) ^ 0x80808080u);
  };
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const double re = __hiloint2double(d[u].y, d[u].x), im = cs * __hiloint2double(d[u].w, d[u].z);
    int a, b;
    digits(re, a, b);
    d[u].x = a;
    d[u].y = b;
    digits(im, a, b);
    d[u].z = a;
    d[u].w = b;
  }
  const float magic = 12582912.0f;
  int8_t* out = dst + ((long)(rb >> 1) * nkc + kc) * RNS_BLK + kg * (RNS_RT * 16) + ((rb & 1) * 64 + lane) * 16;
  const long ps = (long)nrt * nkc * RNS_BLK;
  for (int q = 0; q < RNS_NM; ++q) {
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

adc2_status rns_pack(const double2* src, long gstride, long ld, int inner, int rows, int K, bool conj, int8_t* buf,
                     int* ebuf, double* nbuf, RnsMat* out, hipStream_t st) {
  out->p = buf;
  out->e = ebuf;
  out->rows = rows;
  out->K = K;
  out->nrt = rcdiv(rows, RNS_RT);
  out->nkc = rcdiv(K, RNS_KC);
  const int nrow64 = rcdiv(rows, 64);
  // enough blocks to fill the chip, at least 16 k a block
  const int ns = std::max(1, std::min({NORM_SPLIT, rcdiv(4096, nrow64), rcdiv(K, 16)}));
  k_rns_norm<<<dim3((unsigned)nrow64, (unsigned)ns), 256, 0, st>>>(src, gstride, ld, inner, rows, K, nbuf);
  ADC2_CHECK_LAUNCH();
  const int padded = out->nrt * RNS_RT;
  k_rns_expo<<<rcdiv(padded, 256), 256, 0, st>>>(nbuf, ns, rows, padded, ebuf);
  ADC2_CHECK_LAUNCH();
  k_rns_pack<<<(unsigned)((long)2 * out->nrt * out->nkc), 256, 0, st>>>(src, gstride, ld, inner, rows, K,
                                                                       conj ? -1.0 : 1.0, ebuf, out->nrt, out->nkc, buf);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// ---------------------------------------------------------------------------
// the product of one plane:  C[i][j] = sum_k A[i][k] B[j][k] mod p
// ---------------------------------------------------------------------------
// Tiles of 128 WM x 64 WN on WM WN waves of 128 x 64 (v_mfma_i32_32x32x32_i8,
// 4 x 2 blocks, 128 accumulators a lane).  Chunks of 64 k go from global
// memory straight into an LDS ring of NB stages (the operand layout is the
// LDS image), NB - 1 chunks ahead; one barrier a chunk.
template <int WM, int WN, int NB>
__global__ __launch_bounds__(64 * WM * WN, WM * WN == 4 ? 2 : 1) void k_rns_gemm(
    const int8_t* __restrict__ A, const int8_t* __restrict__ B, int nrtA, int nrtB, int brt0, int nkc, int nbm, int nbn,
    int nrb, int ncb, int8_t* __restrict__ C) {
  constexpr int BM = 128 * WM, BN = 64 * WN, T = 64 * WM * WN;
  constexpr int SB = (BM + BN) * RNS_KC, NL = SB / (T * 16), NLA = BM * RNS_KC / (T * 16);
  __shared__ __align__(16) int8_t s[NB][SB];
  const long nt = (long)nbm * nbn;
  // planes in order, so that each XCD works on the tiles of few planes; tiles
  // in groups of 8 row panels
  const long lid = xcd_remap(blockIdx.x, gridDim.x);
  const int pl = (int)(lid / nt);
  const int t0 = (int)(lid - (long)pl * nt);
  const int per = 8 * nbn, grp = t0 / per, gm = min(8, nbm - grp * 8), r = t0 - grp * per;
  const int bm = grp * 8 + r % gm, bn = r / gm;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  // global address of each of this thread's NL pieces of a stage (chunk 0)
  const int8_t* src[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    const int off = (q * T + tid) * 16;
    if (q < NLA) {
      const int rt = min(bm * (BM / RNS_RT) + (off >> 13), nrtA - 1);   // past the end: discarded rows
      src[q] = A + ((long)pl * nrtA + rt) * nkc * RNS_BLK + (off & (RNS_BLK - 1));
    } else {
      const int ob = off - BM * RNS_KC;
      const int rt = min(brt0 + bn * (BN / RNS_RT) + (ob >> 13), nrtB - 1);
      src[q] = B + ((long)pl * nrtB + rt) * nkc * RNS_BLK + (ob & (RNS_BLK - 1));
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
  i16v acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int x = 0; x < 16; ++x) acc[i][j][x] = 0;
  const int wm = w % WM, wn = w / WM;
#pragma unroll
  for (int t = 0; t < NB - 1; ++t) load(t);
  for (int t = 0; t < nkc; ++t) {
    // chunk t has landed when at most the NB - 2 later ones are outstanding;
    // the barrier also ends every wave's reads of the stage that load() refills
    constexpr int V = (NB - 2) * NL;
    __builtin_amdgcn_s_waitcnt(0x0f70 | (V & 15) | ((V >> 4) << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    load(t + NB - 1);
    const int8_t* p = s[t % NB];
    const int8_t* pa = p + wm * RNS_BLK + (lane >> 5) * (RNS_RT * 16) + (lane & 31) * 16;
    const int8_t* pb = p + BM * RNS_KC + (wn >> 1) * RNS_BLK + (lane >> 5) * (RNS_RT * 16) +
                       ((wn & 1) * 64 + (lane & 31)) * 16;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      i4v a[4], b[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = *(const i4v*)(pb + k2 * (2 * RNS_RT * 16) + j * 512);
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = *(const i4v*)(pa + k2 * (2 * RNS_RT * 16) + i * 512);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);
  const RnsSplit c = RNS_C.split[pl >> 1];
  const int pi = (int)c.p;
  const float magic = 12582912.0f;
  // |acc| <= K 121^2.  Above 4096 k a first step takes off multiples of 1024 p
  // (the float image of acc is then off by up to 64, its quotient by less than
  // one), leaving |x| < 2^18, which the second step reduces to |x| <= p / 2 + 1;
  // up to 4096 k the second step alone ends within 126.
  const bool far = nkc > 64;
  const float invf = c.inv * (1.0f / 1024.0f);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      i4v o;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        int rr[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          int v = acc[i][j][q * 4 + x];
          if (far) {
            const float t = fmaf((float)v, invf, magic);
            v -= __mul24(__float_as_int(t) - RNS_MAGIC, pi * 1024);
          }
          const float t = fmaf((float)v, c.inv, magic);
          rr[x] = v - __mul24(__float_as_int(t) - RNS_MAGIC, pi);
        }
        o[q] = (int)__builtin_amdgcn_perm(__builtin_amdgcn_perm(rr[3], rr[2], 0x0c0c0400),
                                          __builtin_amdgcn_perm(rr[1], rr[0], 0x0c0c0400), 0x05040100);
      }
      const int rb = (bm * BM + wm * 128) / 32 + i, cb = (bn * BN + wn * 64) / 32 + j;
      if (rb < nrb && cb < ncb) *(i4v*)(C + (((long)pl * nrb + rb) * ncb + cb) * 1024 + lane * 16) = o;
    }
}

adc2_status rns_gemm(const RnsMat& A, const RnsMat& B, int col0, int ncols, int8_t* out, hipStream_t st) {
  const int nrb = rcdiv(A.rows, 32), ncb = rcdiv(ncols, 32);
  const int nbm = rcdiv(A.rows, 256), nbn = rcdiv(ncols, 128);
  k_rns_gemm<2, 2, 3><<<(unsigned)((long)RNS_PL * nbm * nbn), 256, 0, st>>>(
      A.p, B.p, A.nrt, B.nrt, col0 / RNS_RT, A.nkc, nbm, nbn, nrb, ncb, out);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

// ---------------------------------------------------------------------------
// recombination
// ---------------------------------------------------------------------------
// A thread recombines 8 entries of one column (two runs of 4 rows): 32 loads
// of 8 bytes, each a 512-byte run of the wave.  Per entry and pair of moduli
// the two weighted residue sums are exact 24-bit integers; their multiples of
// hi are summed exactly in FP64 and reduced modulo 1, those of lo added after.
// Bound by the 32 bytes read and 16 written per entry.
template <class ST>
__global__ __launch_bounds__(256) void k_rns_join(const int8_t* __restrict__ R, int nrb, int ncb, int rows, int cols,
                                                   const int* __restrict__ ea, const int* __restrict__ eb, ST store) {
  const int ncp = (ncb + 1) >> 1;
  const int rb = blockIdx.x / ncp;
  const int cb = 2 * (blockIdx.x % ncp) + (threadIdx.x >> 7);
  if (cb >= ncb) return;
  const int item = threadIdx.x & 127, lane = item >> 1, half = item & 1;
  const int col = cb * 32 + (lane & 31);
  const int row0 = rb * 32 + 16 * half + 4 * (lane >> 5);   // rows row0 + {0..3} and row0 + 8 + {0..3}
  const long ps = (long)nrb * ncb * 1024;
  const int8_t* src = R + ((long)rb * ncb + cb) * 1024 + item * 8;
  double fr[8], fi[8], gr[8], gi[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) fr[x] = fi[x] = gr[x] = gi[x] = 0.0;
#pragma unroll 2
  for (int t = 0; t < RNS_NM / 2; ++t) {
    int2 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = *(const int2*)(src + (4 * t + q) * ps);
    const RnsJoin c = RNS_C.join[t];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      int b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = (int)(int8_t)((x < 4 ? v[q].x : v[q].y) >> (8 * (x & 3)));
      const int yr = __mul24(b[0] + b[1], c.kre1) + __mul24(b[2] + b[3], c.kre2);
      const int yi = __mul24(b[0] - b[1], c.kim1) + __mul24(b[2] - b[3], c.kim2);
      const double dr = (double)yr, di = (double)yi;
      fr[x] = fma(dr, c.hi, fr[x]);
      gr[x] = fma(dr, c.lo, gr[x]);
      fi[x] = fma(di, c.hi, fi[x]);
      gi[x] = fma(di, c.lo, gi[x]);
    }
  }
  if (col >= cols) return;
  const int ec = eb[col];
  constexpr double M = rns_m();
  store.column(col);
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int row = row0 + (x >> 2) * 8 + (x & 3);
    if (row >= rows) continue;
    const int er = ea[row];
    double re = M * ((fr[x] - rint(fr[x])) + gr[x]), im = M * ((fi[x] - rint(fi[x])) + gi[x]);
    if (er == RNS_NAN || ec == RNS_NAN) {
      re = im = __builtin_nan("");
    } else {
      re = ldexp(re, -(er + ec));
      im = ldexp(im, -(er + ec));
    }
    store.put(row, make_double2(re, im));
  }
}

struct StoreZ {
  double2* Z;
  int no, nv;
  double2* p;
  int b;
  __device__ __forceinline__ void column(int col) {
    const int j = col / nv;
    b = col - j * nv;
    p = Z + (long)j * nv * nv;
  }
  __device__ __forceinline__ void put(int row, double2 v) const {
    const int g = row / nv, a = row - g * nv;
    p[(long)g * no * nv * nv + (long)a * nv + b] = v;
  }
};

struct StoreY {
  double2* Y;
  int naux, nv;
  double2* p;
  __device__ __forceinline__ void column(int col) {
    const int g = col / nv;
    p = Y + (long)g * naux * nv + (col - g * nv);
  }
  __device__ __forceinline__ void put(int row, double2 v) const { p[(long)row * nv] = v; }
};

struct StoreRows {
  double2* C;
  long ldc;
  int c;
  __device__ __forceinline__ void column(int col) { c = col; }
  __device__ __forceinline__ void put(int row, double2 v) const { C[(long)row * ldc + c] = v; }
};

template <class ST>
static adc2_status join(const RnsMat& A, const int* eb, int ncols, const int8_t* out, const ST& s, hipStream_t st) {
  const int nrb = rcdiv(A.rows, 32), ncb = rcdiv(ncols, 32);
  k_rns_join<ST><<<(unsigned)((long)nrb * ((ncb + 1) / 2)), 256, 0, st>>>(out, nrb, ncb, A.rows, ncols, A.e, eb, s);
  ADC2_CHECK_LAUNCH();
  return ADC2_OK;
}

adc2_status rns_to_z(const RnsMat& A, const RnsMat& B, const int8_t* out, int no, int nv, double2* Z, hipStream_t st) {
  return join(A, B.e, no * nv, out, StoreZ{Z, no, nv, nullptr, 0}, st);
}
adc2_status rns_to_y(const RnsMat& A, const RnsMat& B, const int8_t* out, int naux, int nv, double2* Y,
                     hipStream_t st) {
  return join(A, B.e, B.rows, out, StoreY{Y, naux, nv, nullptr}, st);
}
adc2_status rns_to_rows(const RnsMat& A, const RnsMat& B, int col0, int ncols, const int8_t* out, double2* C, long ldc,
                        hipStream_t st) {
  return join(A, B.e + col0, ncols, out, StoreRows{C, ldc, 0}, st);
}

}  // namespace adc2
