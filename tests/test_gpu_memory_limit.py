"""Device memory of the FP64 MFMA engines is enough for every call: with an allocator that holds no more than a
handle on those engines needs for it (ADC2_ZGEMM=wide), the same call on a handle that may use
the residue engine (ADC2_ZGEMM=rns) succeeds with the same results to rounding."""
import numpy as np
import pytest
import torch

import paper_2604_27451_amd as A
from synth import dipole_integrals, make_system, random_vectors

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


class Counting:
    """PyTorch's allocator that counts the bytes held and holds at most `limit`."""

    def __init__(self, limit=None):
        self.base, self.live, self.held, self.peak, self.limit, self.refused = A.torch_allocator(), {}, 0, 0, limit, 0
        self.alloc = A.Alloc(A._ALLOC_FN(self._alloc), A._RELEASE_FN(self._release), None)

    def _alloc(self, nbytes, ctx):
        if self.limit is not None and self.held + nbytes > self.limit:
            self.refused += 1
            return None
        p = self.base.alloc(nbytes, ctx)
        if p:
            self.live[p] = nbytes
            self.held += nbytes
            self.peak = max(self.peak, self.held)
        return p

    def _release(self, p, ctx):
        self.held -= self.live.pop(p)
        self.base.release(p, ctx)


def results(monkeypatch, engine, s, call, limit=None):
    monkeypatch.setenv("ADC2_ZGEMM", engine)
    al = Counting()
    setup = call == "setup"
    if setup:
        al.limit = limit
    h = A.adc2_setup(dev(s.L), dev(s.eps), s.nc, s.no, s.nv, s.naux, alloc=al.alloc)
    x = dev(random_vectors(9, 3, h.dim))
    if setup:
        out = A.adc2_get_m11(h)
    else:
        A.adc2_sigma(h, x)
        al.peak, al.limit = al.held, limit
        if call == "adjoint":
            out = A.adc2_omega_backward(h, x, [1.0, 0.5, -0.25])[0]
        elif call == "transition":
            dip = dev(dipole_integrals(3, s.n))
            out = torch.from_numpy(np.asarray(A.adc2_transition(h, dip, x, [9.0, 9.5, 10.0], order=2)[0]))
        elif call == "rayleigh":
            out = torch.tensor(A.adc2_rayleigh(h, x)[0])
        else:
            out = A.adc2_sigma(h, dev(random_vectors(9, 24, h.dim)))
    h.close()
    return out.cpu(), al


# more occupied than virtual spinors, and fewer: other steps are the largest
@pytest.mark.parametrize("nc,no,nv,naux", [(3, 30, 12, 40), (2, 5, 40, 70)])
@pytest.mark.parametrize("call", ["setup", "adjoint", "transition", "rayleigh", "sigma"])
def test_what_the_mfma_engines_need_is_enough(monkeypatch, call, nc, no, nv, naux):
    s = make_system(nc, no, nv, naux, seed=957)
    want, al = results(monkeypatch, "wide", s, call)
    print(f"[case] {call} {(nc, no, nv, naux)} within {al.peak} bytes", flush=True)
    got, al2 = results(monkeypatch, "rns", s, call, limit=al.peak)
    print(f"  {al2.refused} requests refused", flush=True)
    assert float((got - want).abs().max() / want.abs().max()) < 1e-12


def test_transition_holds_one_copy_of_the_integrals(monkeypatch):
    """(kj|bc) and its permuted copy are not held together with the Cholesky operands of their product."""
    nc, no, nv, naux = 3, 40, 8, 160
    s = make_system(nc, no, nv, naux, seed=958)
    o = nc + no
    kjbc, ops = 16 * o * o * nv * nv, 16 * naux * (nv * nv + o * o)
    tph, zt = 16 * (o * nv) ** 2, 16 * o * nv * naux
    tau, f = 16 * (o * (o - 1) // 2) * nv * nv, 16 * 3 * s.n * s.n
    _, al = results(monkeypatch, "wide", s, "transition")
    monkeypatch.setenv("ADC2_ZGEMM", "wide")
    al0 = Counting()
    h = A.adc2_setup(dev(s.L), dev(s.eps), nc, no, nv, naux, alloc=al0.alloc)
    A.adc2_sigma(h, dev(random_vectors(9, 3, h.dim)))
    held = al0.held
    h.close()
    print(f"[case] transition peak {al.peak - held}, two copies and operands {2 * kjbc + ops + tph + zt + tau}", flush=True)
    assert al.peak - held < 2 * kjbc + ops + tph + zt + tau + f
