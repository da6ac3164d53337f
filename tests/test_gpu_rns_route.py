"""Which engine serves the FP64 sigmas of a small system (csrc/rns.h): the residue engine, whatever
form the handle was set up in and whatever it had to give back in between; the bits are
those of a handle that always had its memory.  (nc=6 no=10 nv=40 naux=150: within adc2_sigma_noalloc's array,
above the size from which the engine is used.)"""
import numpy as np
import pytest
import torch

import paper_2604_27451_amd as A
from synth import make_system, random_vectors

pytestmark = pytest.mark.gpu

M = 3


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.fixture(scope="module")
def case():
    s = make_system(6, 10, 40, 150, seed=951)
    L, e = dev(s.L), dev(s.eps)
    h = A.adc2_setup(L, e, s.nc, s.no, s.nv, s.naux)
    x = dev(random_vectors(6, M, h.dim))
    want = A.adc2_sigma(h, x)
    h.close()
    return s, L, e, x, want


def noalloc(h, x):
    S = torch.empty_like(x)
    A.adc2_sigma_noalloc(h, x, S)
    return S


class Refusing:
    """PyTorch's allocator that refuses the next `left` requests."""

    def __init__(self):
        self.base, self.left, self.count = A.torch_allocator(), 0, 0
        self.alloc = A.Alloc(A._ALLOC_FN(self._alloc), self.base.release, None)

    def _alloc(self, nbytes, ctx):
        self.count += 1
        if self.left > 0:
            self.left -= 1
            return None
        return self.base.alloc(nbytes, ctx)


@pytest.mark.parametrize("prec", [A.ADC2_C64, A.ADC2_BF16X3])
def test_handle_switched_to_fp64(case, prec):
    s, L, e, x, want = case
    print(f"[case] set up in form {prec}, switched to FP64", flush=True)
    for first in (noalloc, A.adc2_sigma):
        h = A.adc2_setup(L, e, s.nc, s.no, s.nv, s.naux, prec=prec)
        A.adc2_sigma(h, x)
        A.adc2_set_precision(h, A.ADC2_FP64)
        assert torch.equal(first(h, x), want)
        assert torch.equal(A.adc2_sigma(h, x), want) and torch.equal(noalloc(h, x), want)
        h.close()


@pytest.mark.parametrize("refused", [1, 2])
def test_after_a_refused_request(case, refused):
    """A request of the handle refused once (its scratch goes) or twice (its static operands go too), then
    served: the next sigma is what it was before."""
    s, L, e, x, want = case
    al = Refusing()
    h = A.adc2_setup(L, e, s.nc, s.no, s.nv, s.naux, alloc=al.alloc)
    assert torch.equal(A.adc2_sigma(h, x), want)
    print(f"[case] {refused} refused", flush=True)
    al.left = refused
    w, _ = A.adc2_rayleigh(h, x)
    assert al.left == 0 and np.all(np.isfinite(w))
    assert torch.equal(A.adc2_sigma(h, x), want)
    assert torch.equal(noalloc(h, x), want)
    h.close()


class Sized(Refusing):
    """PyTorch's allocator that refuses what `refuse` says, and notes the sizes."""

    def __init__(self):
        super().__init__()
        self.refuse, self.sizes, self.refused = None, [], 0

    def _alloc(self, nbytes, ctx):
        self.sizes.append(nbytes)
        if self.refuse is not None and self.refuse(nbytes):
            self.refused += 1
            return None
        return self.base.alloc(nbytes, ctx)


@pytest.mark.parametrize("case_", ["chunks", "engine"])
def test_short_of_memory_for_a_while(monkeypatch, case_):
    """Memory short during one sigma: smaller chunks, or (not even one row's work space) the FP64 MFMA engine;
    64 sigmas later the handle asks for its whole work space again."""
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    s = make_system(2, 6, 40, 70, seed=952)
    m = 8
    al = Sized()
    h = A.adc2_setup(dev(s.L), dev(s.eps), s.nc, s.no, s.nv, s.naux, alloc=al.alloc)
    x = dev(random_vectors(7, m, h.dim))
    al.sizes = []
    want = A.adc2_sigma(h, x)
    whole = max(al.sizes)
    h.close()
    zb = 16 * m * s.nc * s.no * s.nv * s.nv
    one = 16 * s.nv * s.no * s.nv   # unpacked doubles of one row: less than its work space
    print(f"[case] short for a while, {case_}, whole {whole}", flush=True)
    al = Sized()
    h = A.adc2_setup(dev(s.L), dev(s.eps), s.nc, s.no, s.nv, s.naux, alloc=al.alloc)
    base = 16 * m * s.nc * s.naux * s.nv   # X, and Y in K-splits of it
    al.refuse = (lambda n: n > whole // 8 and n % base) if case_ == "chunks" else (
        lambda n: n > one and n != zb and n % base)
    got = A.adc2_sigma(h, x)
    assert al.refused > 0
    assert torch.equal(got, want) == (case_ == "chunks")
    assert float((got - want).abs().max() / want.abs().max()) < 1e-12
    n = len(al.sizes)
    assert torch.equal(A.adc2_sigma(h, x), got) and len(al.sizes) == n   # nothing is asked for meanwhile
    al.refuse = None
    for _ in range(64):
        got = A.adc2_sigma(h, x)
    assert whole in al.sizes[n:] and torch.equal(got, want)
    n = len(al.sizes)
    assert torch.equal(A.adc2_sigma(h, x), want) and len(al.sizes) == n
    h.close()


@pytest.mark.parametrize("nc,no,nv,naux,mb,most", [(1, 6, 40, 70, 8, 9), (6, 20, 200, 800, 0, 3)])
def test_graph_outlives_smaller_sigmas(monkeypatch, nc, no, nv, naux, mb, most):
    """A graph of a sigma of `most` vectors, then eager sigmas of fewer on the handle: the buffers stay where they
    are.  (Fewer rows may make longer chunks: first case, 9 in three of 3, 8 in two of 4; fewer vectors may run
    their halves side by side, each in a work space of its own: second case, two vectors of 3.8 10^9 terms.)"""
    if mb:
        monkeypatch.setenv("ADC2_ZGEMM", "rns")
        monkeypatch.setenv("ADC2_RNS_MB", str(mb))
    n = nc + no + nv
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    L = 0.05 * torch.randn((naux, n, n), generator=g, dtype=torch.complex128, device="cuda")
    L = 0.5 * (L + L.transpose(1, 2).conj()).contiguous()
    e = dev(make_system(nc, no, nv, 1, seed=953).eps)
    h = A.adc2_setup(L, e, nc, no, nv, naux)
    del L
    x = torch.randn((most, h.dim), generator=g, dtype=torch.complex128, device="cuda")
    print(f"[case] graph and smaller sigmas {(nc, no, nv, naux)}", flush=True)
    gr = A.adc2_graph_sigma_batch([h], [x])
    want = A.adc2_sigma(h, x)
    for m in range(1, most):
        S = A.adc2_sigma(h, x[:m].contiguous())   # (X-build and back-contraction have other tiles for fewer rows)
        assert float((S - want[:m]).abs().max() / want.abs().max()) < 1e-12
        (got,) = gr.launch()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    gr.close()
    h.close()
