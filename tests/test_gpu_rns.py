"""The residue engine of the large FP64 products (csrc/rns.h), forced at small
sizes with ADC2_ZGEMM=rns.

Tolerance against the oracle.  An entry's integers are rounded at 2^-58 of its
row's norm, so a product of K terms is off by at most sqrt(2K) 2^-57 of
||a|| ||b|| (3e-16 at K = 1000), below the K-term FP64 sums around it; with
the FP64 sums of the oracle and of the other terms, 1e-12 of the largest entry
of sigma is a bound with a margin of two decades at these sizes.
"""
import numpy as np
import pytest
import torch

import paper_2604_27451_amd as A
from oracle import adc2 as O
from synth import dipole_integrals, make_system, random_vectors

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def handle(s, **kw):
    return A.adc2_setup(dev(s.L), dev(s.eps), s.nc, s.no, s.nv, s.naux, **kw)


# rows m nc nv and columns no nv around the 128-row blocks and the 256 x 128
# tiles, K = naux and no nv around the 64-k chunks; the last has K above the
# 4096 terms up to which one reduction step is enough
@pytest.mark.parametrize("nc,no,nv,naux,m", [
    (1, 1, 2, 3, 1), (2, 3, 9, 20, 2), (2, 4, 16, 64, 4), (3, 5, 33, 65, 2), (2, 2, 64, 63, 1), (3, 7, 37, 129, 3),
    (1, 52, 80, 40, 1)])
def test_sigma_against_oracle(monkeypatch, nc, no, nv, naux, m):
    s = make_system(nc, no, nv, naux, seed=900 + naux)
    print(f"[case] rns sigma {(nc, no, nv, naux)} m={m}", flush=True)
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    h = handle(s)
    x = random_vectors(9, m, h.dim)
    S = A.adc2_sigma(h, dev(x)).cpu()
    h.close()
    ref = O.Adc2(s.L, s.eps, nc, no, nv).sigma(torch.from_numpy(x))
    err = float((S - ref).abs().max() / ref.abs().max())
    print(f"  rel err {err:.2e}", flush=True)
    assert err < 1e-12


@pytest.mark.parametrize("mb", [1, 4])
def test_chunks_equal_whole(monkeypatch, mb):
    """Exact integer products: work spaces of 1 and 4 MiB (one, several
    (vector, core) rows a chunk) give the same bits as one chunk."""
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    s = make_system(2, 6, 40, 70, seed=905)
    h = handle(s)
    x = dev(random_vectors(8, 3, h.dim))
    want = A.adc2_sigma(h, x)
    h.close()
    monkeypatch.setenv("ADC2_RNS_MB", str(mb))
    h = handle(s)
    print(f"[case] rns chunks of {mb} MiB", flush=True)
    assert torch.equal(A.adc2_sigma(h, x), want)
    h.close()


@pytest.mark.parametrize("nc,no,nv,naux,mb", [(1, 2, 7, 12, 0), (2, 6, 40, 70, 0), (2, 6, 40, 70, 1)])
def test_setup_transition_and_adjoint_against_oracle(monkeypatch, nc, no, nv, naux, mb):
    """The general products: whole and (mb = 1) in chunks of 256 x 128."""
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    if mb:
        monkeypatch.setenv("ADC2_RNS_MB", str(mb))
    s = make_system(nc, no, nv, naux, seed=950 + naux)
    print(f"[case] rns setup, transition, adjoint {(nc, no, nv, naux)} chunk {mb}", flush=True)
    o = O.Adc2(s.L, s.eps, nc, no, nv)
    h = handle(s)
    m11 = A.adc2_get_m11(h).cpu()
    ref = o.m11().reshape(nc * nv, nc * nv)
    assert float((m11 - ref).abs().max() / ref.abs().max()) < 1e-12
    assert abs(A.adc2_mp2_energy(h) / float(o.mp2_energy()) - 1.0) < 1e-12
    k = 2
    x = random_vectors(7, k, h.dim)
    dip = dipole_integrals(3, nc + no + nv)
    T, f = A.adc2_transition(h, dev(dip), dev(x), [9.0, 9.5], order=2)
    Tr, fr = O.oscillator_strengths(torch.from_numpy(s.L), torch.from_numpy(s.eps), o.sp, torch.from_numpy(dip),
                                    torch.from_numpy(x), [9.0, 9.5], order=2)
    assert np.abs(T - Tr.numpy()).max() < 1e-12 * np.abs(Tr.numpy()).max()
    g = [1.0, -0.5]
    dL, de = A.adc2_omega_backward(h, dev(x), g)
    w = np.array(g) / (np.abs(x) ** 2).sum(1)
    Lr, er = O.omega_gradient(s.L, s.eps, o.sp, torch.from_numpy(x), w)
    assert float((dL.cpu() - Lr).abs().max() / Lr.abs().max()) < 1e-12
    assert float((de.cpu() - er).abs().max() / er.abs().max()) < 1e-12
    h.close()


@pytest.mark.parametrize("p", [600, -600])
def test_scales_exactly(monkeypatch, p):
    """Rows whose squares overflow or underflow: sigma(2^p x) = 2^p sigma(x)."""
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    s = make_system(2, 3, 20, 30, seed=911)
    h = handle(s)
    x = dev(random_vectors(3, 2, h.dim))
    f = 2.0 ** p
    print(f"[case] rns scale 2^{p}", flush=True)
    S, T = A.adc2_sigma(h, x), A.adc2_sigma(h, x * f)
    assert torch.equal(S * f, T)
    h.close()


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_vector_stays_alone(monkeypatch, bad):
    """A NaN or Inf in one vector shows in that vector's sigma and no other's;
    zero vectors give exact zeros."""
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    s = make_system(2, 3, 20, 30, seed=912)
    h = handle(s)
    x = dev(random_vectors(4, 3, h.dim))
    x[2] = 0.0
    S = A.adc2_sigma(h, x)
    y = x.clone()
    y[1, h.ns + 5] = bad
    y[1, 3] = bad
    print(f"[case] rns non-finite {bad}", flush=True)
    T = A.adc2_sigma(h, y)
    assert torch.equal(S[0], T[0]) and torch.equal(S[2], T[2])
    assert float(T[2].abs().max()) == 0.0
    # every doubles entry of core 0 that the bad singles entry reaches, and every singles entry
    assert not torch.isfinite(torch.view_as_real(T[1, :h.ns])).any()
    no, npair = 3, 20 * 19 // 2
    d0 = torch.view_as_real(T[1, h.ns:h.ns + no * npair]).reshape(no * npair, 2)
    assert not torch.isfinite(d0).any()
    h.close()


def test_batch_and_graph_replays_equal_separate(monkeypatch):
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    systems = [make_system(2, 3, 21, 40, seed=921), make_system(1, 5, 34, 70, seed=922)]
    hs = [handle(s) for s in systems]
    xs = [dev(random_vectors(5 + q, 2 + q, h.dim)) for q, h in enumerate(hs)]
    ref = [A.adc2_sigma(h, x) for h, x in zip(hs, xs)]
    print("[case] rns batch and graph", flush=True)
    for a, b in zip(ref, A.adc2_sigma_batch(hs, xs)):
        assert torch.equal(a, b)
    g = A.adc2_graph_sigma_batch(hs, xs)
    for k in range(3):
        for q, x in enumerate(xs):
            x.copy_(dev(random_vectors(50 + 10 * k + q, x.shape[0], x.shape[1])))
        want = [A.adc2_sigma(h, x) for h, x in zip(hs, xs)]
        got = g.launch()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(want, got))
    g.close()
    for h in hs:
        h.close()


@pytest.mark.parametrize("nc,no,nv,naux,m,prec", [(2, 3, 21, 40, 1, A.ADC2_FP64), (6, 12, 60, 200, 3, A.ADC2_FP64),
                                                  (6, 30, 160, 500, 6, A.ADC2_FP64), (3, 6, 50, 70, 2, A.ADC2_BF16X3),
                                                  (3, 6, 50, 70, 2, A.ADC2_C64)])
def test_halves_side_by_side(nc, no, nv, naux, m, prec, monkeypatch):
    """Small sigmas run their halves on two streams, large ones X-build and
    back-contraction (the third case is above the 10^10 terms between them);
    timed kernels and adc2_sigma_noalloc use one.  The same bits, call after
    call without a wait between them, on the default stream and another."""
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    s = make_system(nc, no, nv, naux, seed=961)
    h = handle(s, prec=prec)
    xs = [dev(random_vectors(40 + k, m, h.dim)) for k in range(6)]
    A.adc2_profile(h, True)
    want = [A.adc2_sigma(h, x) for x in xs]
    A.adc2_profile(h, False)
    print(f"[case] rns halves {(nc, no, nv, naux)} m={m}", flush=True)
    for st in (None, torch.cuda.Stream()):
        with torch.cuda.stream(st) if st else torch.cuda.stream(torch.cuda.default_stream()):
            if st:
                st.wait_stream(torch.cuda.default_stream())
            got = [A.adc2_sigma(h, x) for _ in range(4) for x in xs]
        torch.cuda.synchronize()
        assert all(torch.equal(g, want[k % 6]) for k, g in enumerate(got))
    if prec == A.ADC2_FP64 and nv < 100:
        S = torch.empty_like(xs[0])
        A.adc2_sigma_noalloc(h, xs[0], S)
        torch.cuda.synchronize()
        assert torch.equal(S, want[0])
    h.close()


def test_without_its_memory_the_mfma_engine_serves(monkeypatch):
    """An allocator that refuses the engine's own buffers: the doubles are bit
    for bit those of the FP64 MFMA engine (the singles hold M11, which the two
    handles' setups built on different engines), and a later call does not ask
    again."""
    s = make_system(2, 3, 21, 40, seed=931)
    monkeypatch.setenv("ADC2_ZGEMM", "wide")
    hw = handle(s)
    x = dev(random_vectors(6, 2, hw.dim))
    want = A.adc2_sigma(hw, x)
    hw.close()
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    base = A.torch_allocator()
    state = {"count": None, "refused": 0}
    zb = 16 * 2 * s.nc * s.no * s.nv * s.nv

    def _alloc(nbytes, ctx):
        if state["count"] is not None:
            state["count"] += 1
            # after X, Y, Tp and the back-contraction partials: every chunk size, not the MFMA engine's doubles
            if state["count"] >= 5 and nbytes != zb:
                state["refused"] += 1
                return None
        return base.alloc(nbytes, ctx)

    al = A.Alloc(A._ALLOC_FN(_alloc), base.release, None)
    h = handle(s, alloc=al)
    state["count"] = 0
    print("[case] rns without its memory", flush=True)
    got = A.adc2_sigma(h, x)
    assert state["refused"] >= 1 and torch.equal(got[:, h.ns:], want[:, h.ns:])
    assert float((got - want).abs().max() / want.abs().max()) < 1e-12
    n = state["count"]
    assert torch.equal(A.adc2_sigma(h, x), got) and state["count"] == n
    h.close()


def test_short_of_memory_other_scratch_goes_first(monkeypatch):
    """No memory beyond what the handle holds after a split-BF16 sigma: the
    FP64 sigma gives back that form's scratch and runs on the engine (the bits
    of a handle with all the memory it wants), and the split-BF16 sigma takes
    its scratch again once there is memory.  (300 vectors: work spaces beyond
    adc2_sigma_noalloc's array, within which a handle set up in a precision
    form stays on the MFMA engine.)"""
    monkeypatch.setenv("ADC2_ZGEMM", "rns")
    s = make_system(2, 6, 40, 70, seed=941)
    h = handle(s)
    x = dev(random_vectors(6, 300, h.dim))
    want = A.adc2_sigma(h, x)
    h.close()
    base = A.torch_allocator()
    live, limit = {}, [None]

    def _alloc(nbytes, ctx):
        if limit[0] is not None and sum(live.values()) + nbytes > limit[0]:
            return None
        p = base.alloc(nbytes, ctx)
        if p:
            live[p] = nbytes
        return p

    def _release(p, ctx):
        live.pop(p, None)
        base.release(p, ctx)

    al = A.Alloc(A._ALLOC_FN(_alloc), A._RELEASE_FN(_release), None)
    h = handle(s, alloc=al, prec=A.ADC2_BF16X3)
    split = A.adc2_sigma(h, x)
    A.adc2_set_precision(h, A.ADC2_FP64)
    limit[0] = sum(live.values()) + (1 << 16)
    print("[case] rns short of memory", flush=True)
    assert torch.equal(A.adc2_sigma(h, x), want)
    assert sum(live.values()) <= limit[0]
    limit[0] = None
    A.adc2_set_precision(h, A.ADC2_BF16X3)
    assert torch.equal(A.adc2_sigma(h, x), split)
    h.close()
