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
