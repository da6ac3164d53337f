"""Kernels at the edges of their tiles and dispatch rules, against the oracle.

Tolerance: as in test_gpu_rns.py, 1e-12 of the largest entry of a result (sums
of a few thousand FP64 products in another order; 1e-15 relative each).
Eigenvalues converged to residual 1e-10 are quadratic in it; 1e-9 as for the
solvers' other tests.
"""
import numpy as np
import pytest
import torch

import paper_2604_27451_amd as A
from oracle import adc2 as O
from synth import config_system, make_system, random_vectors

pytestmark = pytest.mark.gpu
TOL = 1e-12


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def handle(s):
    return A.adc2_setup(dev(s.L), dev(s.eps), s.nc, s.no, s.nv, s.naux)


def off(a, b):
    return float((a - b).abs().max() / b.abs().max())


# light coupling (groups of 4 valence, 8 core, 64 virtuals; four waves a run up to 128 workgroups a
# vector, one above: the third), sigma2's packing (more than 8 core), singles block and couplings
@pytest.mark.parametrize("nc,no,nv,naux,m", [
    (9, 1, 65, 13, 1), (2, 5, 64, 21, 3), (10, 29, 66, 30, 1), (4, 9, 63, 33, 2), (7, 2, 33, 40, 2)])
def test_setup_and_sigma(nc, no, nv, naux, m):
    print(f"[case] edges {(nc, no, nv, naux)} m={m}", flush=True)
    s = make_system(nc, no, nv, naux, seed=700 + nv)
    o = O.Adc2(s.L, s.eps, nc, no, nv)
    h = handle(s)
    assert off(A.adc2_get_m11(h).cpu(), o.m11().reshape(nc * nv, nc * nv)) < TOL
    x = random_vectors(11, m, h.dim)
    ref = o.sigma(torch.from_numpy(x))
    assert off(A.adc2_sigma(h, dev(x)).cpu(), ref) < TOL
    h.close()


# X and the back contraction: up to 16 rows of an Lvv of 2^23 entries and more on the kernels for
# few rows, others on tiles of 32, 48 or 64 rows, which give the same sums to rounding
def test_few_rows_of_a_large_lvv():
    print("[case] few rows, naux nv^2 above 2^23", flush=True)
    s = make_system(2, 2, 131, 500, seed=731)
    h = handle(s)
    x = random_vectors(12, 8, h.dim)
    S = A.adc2_sigma(h, dev(x))
    assert off(S[:3].cpu(), O.Adc2(s.L, s.eps, 2, 2, 131).sigma(torch.from_numpy(x[:3]))) < TOL
    assert off(A.adc2_sigma(h, dev(x[3:5])), S[3:5]) < TOL
    h.close()


@pytest.mark.parametrize("m", [1, 16, 17, 24, 25, 32, 33, 40, 49])
def test_row_tiles(m):
    """2 m rows of X around the tiles of 32, 48 and 64 rows."""
    s = make_system(2, 2, 21, 40, seed=732)
    h = handle(s)
    print(f"[case] {2 * m} rows", flush=True)
    x = random_vectors(13, m, h.dim)
    ref = O.Adc2(s.L, s.eps, 2, 2, 21).sigma(torch.from_numpy(x))
    assert off(A.adc2_sigma(h, dev(x)).cpu(), ref) < TOL
    h.close()


# subspace sizes of the projected eigenproblem: multiples of k up to the limit, odd ones, one and 64
@pytest.mark.parametrize("k,smax", [(1, 3), (3, 15), (8, 64), (9, 63)])
def test_projected_eigenproblem_sizes(k, smax):
    s = make_system(2, 3, 9, 20, seed=741, sigma=0.3)
    o = O.Adc2(s.L, s.eps, 2, 3, 9)
    h = handle(s)
    print(f"[case] subspace {k} to {smax}", flush=True)
    w, _, info = A.adc2_davidson(h, k, tol=1e-10, max_subspace=smax, max_iter=1000)
    assert info["converged"]
    assert np.abs(np.array(w) - o.roots_exact(k)[0].numpy()).max() < 1e-9
    h.close()


@pytest.mark.parametrize("slices", [1, 17, 1024])
def test_moments_over_slices(monkeypatch, slices):
    """The folded solver's moments in 1, 17 or as many slices of the doubles as there are."""
    s = config_system("c1")
    h = handle(s)
    want = A.adc2_davidson(h, 3, tol=1e-9, solver=A.ADC2_SOLVER_FOLDED, want_vectors=False)[0]
    monkeypatch.setenv("ADC2_CHEB_NCHB", str(slices))
    print(f"[case] moments in {slices} slices", flush=True)
    w, _, info = A.adc2_davidson(h, 3, tol=1e-9, solver=A.ADC2_SOLVER_FOLDED, want_vectors=False)
    assert info["converged"] and np.abs(np.array(w) - np.array(want)).max() < 1e-9
    h.close()


# adjoint: T and the E fill around their 64 and 16 wide tiles, more than 8 core spinors, the sums of
# the doubles diagonal over several vectors; its core term on both engines
@pytest.mark.parametrize("engine", ["auto", "rns"])
@pytest.mark.parametrize("nc,no,nv,naux,m", [(9, 2, 17, 20, 3), (2, 3, 64, 30, 1), (3, 1, 65, 25, 2)])
def test_backward(monkeypatch, engine, nc, no, nv, naux, m):
    print(f"[case] adjoint {(nc, no, nv, naux)} m={m} {engine}", flush=True)
    monkeypatch.setenv("ADC2_ZGEMM", engine)
    s = make_system(nc, no, nv, naux, seed=760 + nv)
    o = O.Adc2(s.L, s.eps, nc, no, nv)
    h = handle(s)
    x = random_vectors(14, m, h.dim)
    g = np.linspace(1.0, -0.7, m)
    dL, de = A.adc2_omega_backward(h, dev(x), list(g))
    Lr, er = O.omega_gradient(s.L, s.eps, o.sp, torch.from_numpy(x), g / (np.abs(x) ** 2).sum(1))
    assert off(dL.cpu(), Lr) < TOL and off(de.cpu(), er) < TOL
    h.close()
