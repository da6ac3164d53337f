"""The projected eigenproblems of the solvers (csrc/jacobi.h) on what is not finite."""
import numpy as np
import pytest
import torch

import paper_2604_27451_amd as A
from synth import make_system, random_vectors

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def handle():
    s = make_system(2, 3, 12, 30, seed=991)
    return A.adc2_setup(dev(s.L), dev(s.eps), s.nc, s.no, s.nv, s.naux)


@pytest.mark.parametrize("solver", [A.ADC2_SOLVER_FULL, A.ADC2_SOLVER_FOLDED])
@pytest.mark.parametrize("rows", [[0], [2], [0, 1, 2]])
def test_guess_that_is_not_finite_is_an_error(solver, rows):
    """A NaN in guess vectors: the Gram matrix of the block has NaN on its diagonal; an error status, and
    the handle solves on afterwards."""
    h = handle()
    g = dev(random_vectors(3, 3, h.dim))
    bad = g.clone()
    for r in rows:
        bad[r, 5] = float("nan")
    print(f"[case] NaN guess rows {rows}, solver {solver}", flush=True)
    with pytest.raises(A.Adc2Error) as e:
        A.adc2_davidson(h, 3, tol=1e-9, guess=bad, solver=solver)
    assert e.value.status in (A.ADC2_ERR_ARG, A.ADC2_ERR_NONFINITE, A.ADC2_ERR_NOCONV)
    w, _, info = A.adc2_davidson(h, 3, tol=1e-9, solver=solver)
    assert info["converged"] and np.all(np.isfinite(w))
    h.close()


@pytest.mark.parametrize("p", [-400, -250, 250, 400])
def test_scaled_guess(p):
    """Guess vectors times 2^p: their Gram matrix is 2^2p times that of the vectors themselves, its squares beyond
    the range of FP64, and its eigenvectors are the same.  Powers of two go through exactly, so the
    solve is the same, bit for bit.  (Two nearly parallel vectors: orthonormal to rounding after the second of
    the two passes only if the first one has rotated them.)"""
    h = handle()
    g = dev(random_vectors(4, 2, h.dim))
    g[1] = g[0] + 5e-7 * g[1]
    print(f"[case] guess times 2^{p}", flush=True)
    w0, _, i0 = A.adc2_davidson(h, 2, tol=1e-11, guess=g)
    w1, _, i1 = A.adc2_davidson(h, 2, tol=1e-11, guess=g * 2.0 ** p)
    print(f"  {i0['iters']} and {i1['iters']} iterations", flush=True)
    assert i1["iters"] == i0["iters"] and list(w1) == list(w0)
    h.close()
