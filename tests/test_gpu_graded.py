"""FP64 sigma, entry by entry, of operands whose entries differ by many decades:
each entry within what a FP64 sum of its own terms may be off, on the residue
engine (csrc/rns.h, forced by ADC2_ZGEMM=rns) as on the FP64 MFMA engines.

Tolerance.  A sum of K complex products in FP64, in any order, is off by at most
gamma = (K + 2) u of sum |a_k| |b_k| in each part (u = 2^-53; two real products
a part), sqrt(2) gamma altogether; a chain of two such sums by the sum of
both.  The residue engine's entries may be off by 4 sqrt(K) 2^-58 ||a|| ||b||
<= 40 sqrt(K) 2^-58 sum |a_k| |b_k| where it serves, less than that.
References are sums in long double (64 mantissa bits).
"""
import numpy as np
import pytest
import torch

import paper_2604_27451_amd as A
from synth import make_system

pytestmark = pytest.mark.gpu

U = 2.0 ** -53
NC, NO, NV = 1, 2, 40


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def scaled(s, f):
    """The system with its Cholesky vectors scaled entry by entry by the symmetric f [naux][n][n]."""
    L = s.L * f
    return 0.5 * (L + L.conj().transpose(0, 2, 1))


def blocks(naux, n, kind, rng):
    """Scales f: 'halves' sets virtual-virtual entries to 1e-8 where the valence-virtual ones are 1 and
    the valence-virtual ones to 0 where those are 1; 'decades' spreads all by a log-normal of three decades;
    'disjoint' has no common Cholesky index at all; 'even' leaves them."""
    o = NC + NO
    f = np.ones((naux, n, n))
    h = naux // 2
    if kind in ("halves", "disjoint"):
        f[h:, o:, o:] = 1e-8 if kind == "halves" else 0.0
        f[:h, NC:o, o:] = 0.0
        f[:h, o:, NC:o] = 0.0
    elif kind == "decades":
        g = 10.0 ** (1.5 * rng.standard_normal((naux, n, n)))
        f = np.triu(g) + np.transpose(np.triu(g, 1), (0, 2, 1))
    return f


@pytest.mark.parametrize("engine", ["rns", "wide"])
@pytest.mark.parametrize("kind", ["even", "halves", "decades", "disjoint"])
def test_singles_in(monkeypatch, engine, kind):
    """Doubles of sigma(e_c): Z_ab - Z_ba, Z_ab = sum_P L^P_ac L^P_bj, but for the pairs with c itself."""
    naux = 300
    s = make_system(NC, NO, NV, naux, seed=971)
    n, o = s.n, NC + NO
    L = scaled(s, blocks(naux, n, kind, np.random.default_rng(5)))
    monkeypatch.setenv("ADC2_ZGEMM", engine)
    print(f"[case] graded singles in, {kind}, {engine}", flush=True)
    h = A.adc2_setup(dev(L), dev(s.eps), NC, NO, NV, naux)
    c0 = 7
    x = np.zeros((1, h.dim), complex)
    x[0, c0] = 1.0
    S = A.adc2_sigma(h, dev(x)).cpu().numpy()[0, h.ns:].reshape(NO, -1)
    h.close()
    Lx = L.astype(np.clongdouble)
    iu = np.triu_indices(NV, 1)
    keep = (iu[0] != c0) & (iu[1] != c0)
    worst = 0.0
    for j in range(NO):
        a, b = Lx[:, o:, o + c0], Lx[:, o:, NC + j]          # L^P_ac, L^P_bj  [P][.]
        Z = a.T @ b
        ref = (Z - Z.T)[iu]
        B = np.abs(a).T @ np.abs(b)
        tol = (np.sqrt(2.0) * (naux + 4) * U * (B + B.T))[iu]
        err = np.abs(S[j] - ref)
        assert np.all(err[keep] <= tol[keep]), float((err[keep] / np.maximum(tol[keep], 1e-300)).max())
        if tol[keep].max() > 0:
            worst = max(worst, float((err[keep] / np.maximum(tol[keep], 1e-300)).max()))
    print(f"  worst error {worst:.2e} of the bound", flush=True)


@pytest.mark.parametrize("engine", ["rns", "wide"])
@pytest.mark.parametrize("kind", ["even", "halves", "one"])
def test_doubles_in(monkeypatch, engine, kind):
    """Singles of sigma(0, r2): sum_P,c Lvv[P][a][c] Y[P][c] - sum_jd conj(<Kd||Ij>) R_j[c][d] with
    Y[P][c] = sum_jd conj(L^P_dj) R_j[c][d]; valence spinor 0 large in R and absent from L (halves), one large
    amplitude (one)."""
    naux = 60
    s = make_system(NC, NO, NV, naux, seed=972)
    n, o = s.n, NC + NO
    f = np.ones((naux, n, n))
    if kind == "halves":
        for p in (NC,):
            f[:, p, :] = 0.0
            f[:, :, p] = 0.0
    L = scaled(s, f)
    monkeypatch.setenv("ADC2_ZGEMM", engine)
    print(f"[case] graded doubles in, {kind}, {engine}", flush=True)
    h = A.adc2_setup(dev(L), dev(s.eps), NC, NO, NV, naux)
    rng = np.random.default_rng(8)
    npair = NV * (NV - 1) // 2
    r = rng.standard_normal((NO, npair)) + 1j * rng.standard_normal((NO, npair))
    if kind == "halves":
        r[1] *= 1e-9
    elif kind == "one":
        r *= 1e-9
        r[0, ::97] = 1.0
    x = np.zeros((1, h.dim), complex)
    x[0, h.ns:] = r.reshape(-1)
    S = A.adc2_sigma(h, dev(x)).cpu().numpy()[0, :h.ns]
    h.close()
    Lx = L.astype(np.clongdouble)
    iu = np.triu_indices(NV, 1)
    R = np.zeros((NO, NV, NV), np.clongdouble)               # R[j][c][d]
    R[:, iu[0], iu[1]] = r
    R[:, iu[1], iu[0]] = -r
    Lvv, Ldj = Lx[:, o:, o:], Lx[:, o:, NC:o]                 # [P][a][c], [P][d][j]
    K = NO * NV

    def chain(Lvv, Ldj, R, Lii, Lij, LdI, sign):
        Y = np.einsum("pdj,jcd->pc", Ldj.conj(), R)
        heavy = np.einsum("pac,pc->a", Lvv, Y)
        # <Kd||Ij> = sum_P L_KI L_dj - L_Kj L_dI, K = I the one core spinor
        V = np.einsum("p,pdj->jd", Lii, Ldj) - sign * np.einsum("pj,pd->jd", Lij, LdI)
        return heavy, np.einsum("jd,jad->a", V.conj(), R)

    Lii, Lij, LdI = Lx[:, 0, 0], Lx[:, 0, NC:o], Lx[:, o:, 0]
    heavy, light = chain(Lvv, Ldj, R, Lii, Lij, LdI, 1.0)
    bh, bl = chain(np.abs(Lvv), np.abs(Ldj), np.abs(R), np.abs(Lii), np.abs(Lij), np.abs(LdI), -1.0)
    ref = heavy - light
    tol = np.sqrt(2.0) * ((K + naux * NV + 8) * U * bh + (K + naux + 8) * U * bl + 4 * U * np.abs(ref))
    err = np.abs(S - ref)
    worst = float((err / tol).max())
    print(f"  worst error {worst:.2e} of the bound", flush=True)
    assert worst <= 1.0


@pytest.mark.parametrize("nc,no,nv,naux", [(1, 2, 7, 12), (2, 6, 40, 70)])
def test_setup_transition_and_adjoint(monkeypatch, nc, no, nv, naux):
    """The general products (in place and added to their destination, rows and terms contiguous) on entries
    spread over a decade and a half, a part of which the integers do not serve: the oracle's values to 1e-12 of the
    largest, the tolerance of the like tests on even entries."""
    from oracle import adc2 as O
    from synth import dipole_integrals, random_vectors
    s = make_system(nc, no, nv, naux, seed=980 + naux)
    g = 10.0 ** (0.75 * np.random.default_rng(6).standard_normal((naux, s.n, s.n)))
    L = scaled(s, np.triu(g) + np.transpose(np.triu(g, 1), (0, 2, 1)))
    L *= 0.05 / np.sqrt((np.abs(L) ** 2).mean())
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    print(f"[case] graded setup, transition, adjoint {(nc, no, nv, naux)}", flush=True)
    o = O.Adc2(L, s.eps, nc, no, nv)
    h = A.adc2_setup(dev(L), dev(s.eps), nc, no, nv, naux)
    m11 = A.adc2_get_m11(h).cpu()
    ref = o.m11().reshape(nc * nv, nc * nv)
    assert float((m11 - ref).abs().max() / ref.abs().max()) < 1e-12
    assert abs(A.adc2_mp2_energy(h) / float(o.mp2_energy()) - 1.0) < 1e-12
    k = 2
    x = random_vectors(7, k, h.dim)
    S = A.adc2_sigma(h, dev(x)).cpu()
    ref = o.sigma(torch.from_numpy(x))
    assert float((S - ref).abs().max() / ref.abs().max()) < 1e-12
    dip = dipole_integrals(3, nc + no + nv)
    T, _ = A.adc2_transition(h, dev(dip), dev(x), [9.0, 9.5], order=2)
    Tr, _ = O.oscillator_strengths(torch.from_numpy(L), torch.from_numpy(s.eps), o.sp, torch.from_numpy(dip),
                                   torch.from_numpy(x), [9.0, 9.5], order=2)
    assert np.abs(T - Tr.numpy()).max() < 1e-12 * np.abs(Tr.numpy()).max()
    gw = [1.0, -0.5]
    dL, de = A.adc2_omega_backward(h, dev(x), gw)
    w = np.array(gw) / (np.abs(x) ** 2).sum(1)
    Lr, er = O.omega_gradient(L, s.eps, o.sp, torch.from_numpy(x), w)
    assert float((dL.cpu() - Lr).abs().max() / Lr.abs().max()) < 1e-12
    assert float((de.cpu() - er).abs().max() / er.abs().max()) < 1e-12
    h.close()


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_not_finite_as_the_fp64_sum(monkeypatch, bad):
    """A singles and a doubles entry that are not finite: every doubles entry of sigma is NaN, infinite
    (with its sign) or finite as on the FP64 MFMA engine."""
    from synth import random_vectors
    s = make_system(2, 3, 20, 30, seed=912)
    x = random_vectors(4, 3, s.nc * s.nv + s.nc * s.no * s.nv * (s.nv - 1) // 2)
    ns = s.nc * s.nv
    x[1, ns + 5] = bad
    x[1, 3] = bad
    x[2] = 0.0
    x[2, 7] = bad
    got = {}
    for engine in ("wide", "rns"):
        monkeypatch.setenv("ADC2_ZGEMM", engine)
        print(f"[case] {bad} on {engine}", flush=True)
        h = A.adc2_setup(dev(s.L), dev(s.eps), s.nc, s.no, s.nv, s.naux)
        S = torch.view_as_real(A.adc2_sigma(h, dev(x))[:, ns:])
        got[engine] = (torch.isnan(S).cpu(), (torch.isinf(S) * torch.sign(S)).nan_to_num().cpu())
        h.close()
    assert all(torch.equal(a, b) for a, b in zip(got["wide"], got["rns"]))


def test_more_terms_than_are_looked_at_together(monkeypatch):
    """The pair density of the transition moments, K = 903 pairs x 75 virtuals = 67725 terms: k_rns_fp64 takes
    a sixth of its entries, in runs of 65536 terms, and leaves out the pairs of a spinor without Cholesky
    vectors.  Both engines are held to 1e-12 of the oracle above, so to 2e-12 of each other."""
    from synth import dipole_integrals, random_vectors
    nc, no, nv, naux = 2, 41, 75, 60
    s = make_system(nc, no, nv, naux, seed=990)
    g = 10.0 ** (1.5 * np.random.default_rng(7).standard_normal((naux, s.n, s.n)))
    g[:, nc + 3, :] = 0.0
    g[:, :, nc + 3] = 0.0
    L = scaled(s, np.triu(g) + np.transpose(np.triu(g, 1), (0, 2, 1)))
    L *= 0.05 / np.sqrt((np.abs(L) ** 2).mean())
    T = {}
    for engine in ("wide", "rns"):
        monkeypatch.setenv("ADC2_ZGEMM", engine)
        print(f"[case] graded transition of many pairs, {engine}", flush=True)
        h = A.adc2_setup(dev(L), dev(s.eps), nc, no, nv, naux)
        x = random_vectors(7, 2, h.dim)
        T[engine], _ = A.adc2_transition(h, dev(dipole_integrals(3, nc + no + nv)), dev(x), [9.0, 9.5], order=2)
        h.close()
    assert np.abs(T["rns"] - T["wide"]).max() < 2e-12 * np.abs(T["wide"]).max()
