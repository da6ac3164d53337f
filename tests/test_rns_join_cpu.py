"""Recombination of the residue engine (csrc/rnsconst.h, rns.h) against whole-number arithmetic: the
fraction z / M from residue sums of up to 32 K-runs, in the order of k_rns_join.

Tolerance: the parts of hi are exact; the parts of lo are at most 0.018 (32 runs) and summed in eight
FP64 fma, so the fraction is off by less than 8 * 0.018 * 2^-53 + 2^-54."""
import ctypes
import os
import random
import shutil
import subprocess
from fractions import Fraction

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2604_27451_amd", "csrc")
SHIM = r'''
#include <cmath>
#include "rnsconst.h"
static constexpr adc2::RnsConst C = adc2::make_const();
extern "C" void rule(double* r) {
  r[0] = adc2::RNS_QMEAN;
  for (int i = 0; i < 3; ++i) r[1 + i] = adc2::RNS_FLAT[i];
}
extern "C" int serves(int runs, const int* n, const int* s, int K) {   // of an entry's sums by K-runs
  int terms = 0, part = 0, weight = 0;
  for (int i = 0; i < runs; ++i) {
    const int b = adc2::rns_terms_byte(n[i], 1.0f / (float)K);
    terms |= b;
    part += b ? b - 1 : 0;
    weight += adc2::rns_weight_byte(s[i], 1.0f / (float)K);
  }
  return adc2::rns_spread_serves(terms, part, weight);
}
extern "C" int serves_full(int runs, const int* s, int K) {   // ... of two rows that are known to be full
  int weight = 0;
  for (int i = 0; i < runs; ++i) weight += adc2::rns_weight_byte(s[i], 1.0f / (float)K);
  return adc2::rns_spread_serves(1, adc2::RNS_FULL_PART, weight);
}
extern "C" int full_part() { return adc2::RNS_FULL_PART; }
extern "C" void moduli(int* p) { for (int q = 0; q < adc2::RNS_NM; ++q) p[q] = adc2::RNS_P[q]; }
extern "C" void join(const int* u, double* out) {   // u[2 q], u[2 q + 1]: sums of c+, c- of modulus q
  double fr = 0, fi = 0, gr = 0, gi = 0;
  for (int t = 0; t < adc2::RNS_NM / 2; ++t) {
    const adc2::RnsJoin c = C.join[t];
    const int* v = u + 4 * t;
    const int yr = (v[0] + v[1]) * c.kre1 + (v[2] + v[3]) * c.kre2;
    const int yi = (v[0] - v[1]) * c.kim1 + (v[2] - v[3]) * c.kim2;
    fr = std::fma((double)yr, c.hi, fr);
    gr = std::fma((double)yr, c.lo, gr);
    fi = std::fma((double)yi, c.hi, fi);
    gi = std::fma((double)yi, c.lo, gi);
  }
  out[0] = adc2::rns_frac(fr, gr);
  out[1] = adc2::rns_frac(fi, gi);
  out[2] = gr;
  out[3] = gi;
}
'''
G2 = 2.0 ** 116.66


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("rnsjoin")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o",
                    str(d / "lib.so")], check=True)
    return ctypes.CDLL(str(d / "lib.so"))


def join(lib, u):
    a, out = (ctypes.c_int * 32)(*u), (ctypes.c_double * 4)()
    lib.join(a, out)
    return list(out)


def moduli(lib):
    p = (ctypes.c_int * 16)()
    lib.moduli(p)
    return list(p)


class Crt:
    def __init__(self, P):
        self.P, self.M = P, 1
        for p in P:
            self.M *= p
        self.s = [next(x for x in range(1, p) if (x * x + 1) % p == 0) for p in P]
        self.w = [self.M // p * pow(self.M // p, -1, p) for p in P]

    def value(self, u):
        """(re, im) in (-M/2, M/2] of the sums u of residues x + s y, x - s y."""
        re = im = 0
        for q, p in enumerate(self.P):
            a, b = u[2 * q], u[2 * q + 1]
            re += self.w[q] * ((a + b) * pow(2, -1, p) % p)
            im += self.w[q] * ((a - b) * pow(2 * self.s[q], -1, p) % p)
        half = self.M // 2
        return tuple((v % self.M) - (self.M if v % self.M > half else 0) for v in (re, im))

    def residues(self, re, im):
        out = []
        for q, p in enumerate(self.P):
            for sg in (1, -1):
                r = (re + sg * self.s[q] * im) % p
                out.append(r - p if r > p // 2 else r)
        return out


TOL = 8 * 0.0185 * 2.0 ** -53 + 2.0 ** -54


def check(lib, crt, u):
    got = join(lib, u)
    for g, z in zip(got, crt.value(u)):
        if abs(z) > G2:
            continue    # beyond what rows of norm 2^58.33 give
        assert abs(Fraction(g) - Fraction(z, crt.M)) < TOL, (u, g, float(Fraction(z, crt.M)))
    return got


def test_products_of_one_and_more_runs(lib):
    crt, rng = Crt(moduli(lib)), random.Random(5)
    lim = int(G2)
    for runs in (1, 2, 8, 32):
        for _ in range(200):
            re, im = rng.randint(-lim, lim), rng.randint(-lim, lim)
            parts = [[rng.randint(-lim // runs, lim // runs) for _ in range(2)] for _ in range(runs - 1)]
            parts.append([re - sum(p[0] for p in parts), im - sum(p[1] for p in parts)])
            u = [sum(v) for v in zip(*(crt.residues(*p) for p in parts))]
            assert crt.value(u) == (re, im)
            check(lib, crt, u)


def test_largest_low_parts(lib):
    """Residue sums of 32 runs with every low part as large as it can be and of one sign, and z next to
    the largest: the low parts take the fraction of the high ones past 1/2."""
    crt, rng = Crt(moduli(lib)), random.Random(6)
    P = crt.P
    one = [join(lib, [1 if i == q else 0 for i in range(32)])[2:] for q in range(32)]   # low parts of each residue
    past = 0
    for part in (0, 1):
        for sign in (1, -1):
            for _ in range(6000):
                u = []
                for q in range(32):
                    top = 32 * (P[q // 2] // 2)
                    u.append((top if one[q][part] * sign > 0 else -top) if q < 28 else rng.randint(-top, top))
                z = crt.value(u)[part]
                got = check(lib, crt, u)
                high = Fraction(z, crt.M) - Fraction(got[2 + part])
                past += abs(z) <= G2 and abs(high) > Fraction(1, 2)
    assert past > 0


# ---- which entries the integers serve: N sum |a|^2 |b|^2 >= ||a||^2 ||b||^2 / 64, or N = 0 (csrc/rnsconst.h) ----
def rule(lib):
    r = (ctypes.c_double * 4)()
    lib.rule(r)
    return list(r)


def codes(a, qmean):
    import numpy as np
    q = np.floor(qmean * len(a) * np.abs(a) ** 2 / (np.abs(a) ** 2).sum())
    return np.where(a == 0, 0, 1 + np.clip(q, 0, 126)).astype(int)


def rows(K):
    """Rows of many kinds: like entries, real ones, spread over decades, blocks, few large ones."""
    import numpy as np
    rng = np.random.default_rng(K)
    g = lambda: rng.standard_normal(K) + 1j * rng.standard_normal(K)
    out = [g(), rng.standard_normal(K) + 0j, np.ones(K) + 0j]
    out += [g() * 10.0 ** (s * rng.standard_normal(K)) for s in (0.3, 0.6, 1.0, 2.0)]
    out += [g() * np.where(np.arange(K) < f * K, 1.0, t) for f in (0.02, 0.3, 0.5, 0.8) for t in (0.0, 1e-8, 0.05, 0.3)]
    out += [g() * np.where(np.arange(K) >= f * K, 1.0, t) for f in (0.1, 0.5, 0.7) for t in (0.0, 1e-8, 0.05, 0.3)]
    out += [g() * 10.0 ** (-6.0 * np.arange(K) / K), g() * 10.0 ** (-6.0 * (K - np.arange(K)) / K)]
    return out


@pytest.mark.parametrize("K", [37, 150, 1500])
@pytest.mark.parametrize("runs", [1, 8, 32])
def test_rows_that_the_integers_serve(lib, K, runs):
    import numpy as np
    qmean, *flat = rule(lib)
    rs = rows(K)
    qs = [codes(r, qmean) for r in rs]
    fl = [all((q > i).sum() >= np.ceil(f * K) for i, f in enumerate(flat)) for q in qs]
    full = [(q > 0).sum() >= np.ceil(flat[0] * K) for q in qs]
    cut = [K * i // runs for i in range(runs + 1)]
    served = refused = 0
    for a, qa, fa, ga in zip(rs, qs, fl, full):
        for b, qb, fb, gb in zip(rs, qs, fl, full):
            n = (qa > 0) & (qb > 0)
            s = np.maximum(qa - 1, 0) * np.maximum(qb - 1, 0)
            sums = [(ctypes.c_int * runs)(*(int(v[i:j].sum()) for i, j in zip(cut, cut[1:]))) for v in (n, s)]
            assert not (ga and gb) or n.sum() >= lib.full_part() * K / 254.0
            if (fa and fb) or (lib.serves_full(runs, sums[1], K) if ga and gb else lib.serves(runs, *sums, K)):
                served += 1
                d = n.sum() * (np.abs(a * b) ** 2).sum() / ((np.abs(a) ** 2).sum() * (np.abs(b) ** 2).sum())
                assert n.sum() == 0 or d >= 0.999 / 64
            else:
                refused += 1
    assert served and refused
    # like entries are flat, entries over decades are not, and their products are served by their codes as well
    if K == 1500:
        assert fl[0] and not any(fl[4:7])
        n, s = np.ones(K, int), (qs[0] - 1) * np.roll(qs[0] - 1, 1)
        sums = [(ctypes.c_int * runs)(*(int(v[i:j].sum()) for i, j in zip(cut, cut[1:]))) for v in (n, s)]
        assert lib.serves(runs, *sums, K)


def test_errors_where_the_integers_serve(lib):
    """Rounded to the fixed point of the rows against FP64 sums term by term: over the products of 200 pairs
    of each two kinds of rows that are served, the rms error is no larger than the FP64 sums'."""
    import numpy as np
    K = 400
    qmean, *flat = rule(lib)

    def fixed(a):   # whole numbers of a row scaled to a norm in (2^57.33, 2^58.33]
        e = int(np.floor(58.33 - np.log2(np.sqrt((np.abs(a) ** 2).sum()))))
        return [(int(round(float(np.ldexp(z.real, e)))), int(round(float(np.ldexp(z.imag, e))))) for z in a], e

    rng = np.random.default_rng(11)
    kinds = {"even": lambda: 1.0, "third": lambda: 10.0 ** (0.33 * rng.standard_normal(K)),
             "half": lambda: 10.0 ** (0.5 * rng.standard_normal(K)), "few": lambda: np.where(np.arange(K) < 20, 1.0, 1e-3)}
    seen = 0
    for ka in kinds:
        for kb in kinds:
            ei, ef, served = 0.0, 0.0, 0
            for _ in range(12):
                a, b = ((rng.standard_normal(K) + 1j * rng.standard_normal(K)) * kinds[k]() for k in (ka, kb))
                qa, qb = codes(a, qmean), codes(b, qmean)
                n, s = int(((qa > 0) & (qb > 0)).sum()), int(((qa - 1) * (qb - 1)).sum())
                if not lib.serves(1, (ctypes.c_int * 1)(n), (ctypes.c_int * 1)(s), K):
                    continue
                served += 1
                (fa, xa), (fb, xb) = fixed(a), fixed(b)
                got = sum(x[0] * y[0] - x[1] * y[1] for x, y in zip(fa, fb))
                exact = sum(Fraction(x.real) * Fraction(y.real) - Fraction(x.imag) * Fraction(y.imag) for x, y in zip(a, b))
                f64 = 0.0
                for x, y in zip(a, b):
                    f64 += x.real * y.real
                    f64 -= x.imag * y.imag
                scale = np.sqrt((np.abs(a) ** 2).sum() * (np.abs(b) ** 2).sum())
                ei += (float(Fraction(got) / Fraction(2) ** (xa + xb) - exact) / scale) ** 2
                ef += (float(Fraction(f64) - exact) / scale) ** 2
            if served >= 6:
                seen += 1
                assert ei <= ef, (ka, kb, ei, ef, served)
    assert seen >= 8


def test_bounds_of_the_rule(lib):
    """The worst flat rows: their codes in opposite order."""
    qmean, f1, f2, f3 = rule(lib)
    N = 10000
    q = [0] * N                      # codes less one of a flat row at its limits, smallest first
    for f, c in ((f2, 1), (f3, 2)):
        for i in range(round((1 - f) * N), N):
            q[i] = c
    S = sum(x * y for x, y in zip(q, reversed(q))) / N
    assert (2 * f1 - 1) * S >= qmean ** 2 / 64
