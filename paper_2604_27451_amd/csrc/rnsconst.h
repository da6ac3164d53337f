// rnsconst.h -- the moduli of the residue engine (rns.h) and the arithmetic of its
// recombination, plain C++ (constexpr: host and device).
#pragma once

namespace adc2 {

constexpr int RNS_NM = 16;   // moduli
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
  double hi, lo;       // 1 / (p1 p2) = hi + lo, hi a multiple of 2^-34
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
    const long pp = (long)p1 * p2, one = 1L << 34;
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
constexpr double rns_m() {
  double m = 1.0;
  for (int q = 0; q < RNS_NM; ++q) m *= RNS_P[q];
  return m;
}
// Which entries of a product the integers serve.  Code of an entry a_k of an operand's row: 0 for an exact
// zero, else 1 + q, q = |a_k|^2 in units of a quarter of the row's mean (RNS_QMEAN), rounded down, at most 126.
// Two sums over the terms of an entry: N, the common terms that are not zero, and S = sum q_k(a) q_k(b), at
// most 16 K^2 sum |a_k|^2 |b_k|^2 / (||a||^2 ||b||^2).  The entry is served if N = 0 (an exact zero on either engine)
// or N S >= K^2 / 4, that is
//   N sum |a_k|^2 |b_k|^2 >= ||a||^2 ||b||^2 / 64.
// A FP64 sum of N terms in any order that knows nothing of them is off by about
// 0.2 2^-53 sqrt(N sum |a_k|^2 |b_k|^2) rms (0.29 2^-53 of each partial sum), then 0.025 2^-53 ||a|| ||b||; the
// integers by 2^-59 ||a|| ||b|| = 0.015 2^-53.
// A flat row has at least RNS_FLAT K codes of 1, 2 and 3 and more (1, 0.78 and 0.61 of normal complex entries):
// two of them have N >= 0.8 K and, the smaller codes of each against the larger of the other, S >= 0.32 K.
constexpr float RNS_QMEAN = 4.0f;
constexpr double RNS_FLAT[3] = {0.90, 0.60, 0.46};
// The two sums of a run of terms as bytes (rk = 1 / K): N in units of K / 254, 0 for none, and S in units of K / 8
constexpr int rns_terms_byte(int n, float rk) { return n == 0 ? 0 : 1 + (int)((float)n * (254.0f * rk) < 254.0f ? (float)n * (254.0f * rk) : 254.0f); }
constexpr int rns_weight_byte(int s, float rk) { return (int)((float)s * (8.0f * rk) < 255.0f ? (float)s * (8.0f * rk) : 255.0f); }
// ... N of two rows of which at least RNS_FLAT[0] is not zero, and the rule on the sums over the runs
constexpr int RNS_FULL_PART = 203;   // 254 (2 * 0.90 - 1), rounded down
constexpr bool rns_spread_serves(int terms, int part, int weight) { return terms == 0 || part * weight >= 254 * 8 / 4; }

// hi + lo modulo 1, in [-1/2, 1/2]; |hi| < 2^50.  hi comes as an exact sum, so its whole part goes
// first; lo may carry the rest past 1/2 (0.018 at 32 K-runs, against 0.0106 between the largest
// |z| / M and 1/2), so it is reduced as well.
constexpr double rns_whole(double x) { return (x + 0x1.8p52) - 0x1.8p52; }
constexpr double rns_frac(double hi, double lo) {
  const double t = (hi - rns_whole(hi)) + lo;
  return t - rns_whole(t);
}

}  // namespace adc2
