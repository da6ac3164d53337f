"""The work that users of the CVS-ADC(2) library have it do, as cases to measure.

A case is one call (or one short sequence) of the public entry points on a
system of nc core, no valence and nv virtual spinors with naux Cholesky
vectors.  Kinds:

  sigma       S = M X for a block of m vectors: the inner step of every solve
  batch       the same for eight systems of uneven size in one launch sequence
  setup       handle of a new system (Cholesky blocks, MP2, singles block)
  adjoint     d omega / d(L, eps) of k vectors (backward of a solve)
  solve       the k lowest roots by the folded Davidson solver
  transition  transition dipole moments of k states through second order

Sizes run from the smallest system an oracle can follow in seconds
(nc=6 no=10 nv=40 naux=150) to the heavy-element-complex shape of the
benchmark (nc=6 no=120 nv=600 naux=3000); forms are complex FP64 (0),
complex64 (1) and split BF16 (2).  Inputs follow the recipe of the benchmark's
synthetic systems: energies uniform in core / valence / virtual windows,
Hermitian Cholesky slices with normal entries of spread 0.05, trial vectors of
unit norm.
"""
import math

import numpy as np
import torch

import paper_2604_27451_amd as A

C128 = torch.complex128
F64 = torch.float64
SPREAD = 0.05

# (no, nv) of the batch workload's eight systems; naux = 4 nv
BATCH = [(20, 100), (80, 400), (35, 250), (60, 150), (25, 380), (70, 220), (45, 310), (55, 120)]


def listed():
    return [
        # the small molecule: one trial vector, every launch counts
        dict(name="sigma_small_m1", kind="sigma", prec=0, nc=6, no=10, nv=40, naux=150, m=1),
        # a small molecule with a few unconverged roots left
        dict(name="sigma_mid_m4", kind="sigma", prec=0, nc=6, no=12, nv=100, naux=300, m=4),
        # an ordinary system of ragged sizes
        dict(name="sigma_ragged_m7", kind="sigma", prec=0, nc=6, no=45, nv=310, naux=1240, m=7),
        # the 3d-compound size: one block of ten roots
        dict(name="sigma_block_m10", kind="sigma", prec=0, nc=6, no=60, nv=300, naux=1500, m=10),
        # the heavy-element-complex shape, the last two roots of a solve
        dict(name="sigma_large_m2", kind="sigma", prec=0, nc=6, no=120, nv=600, naux=3000, m=2),
        # the precision forms as a solver's first stage runs them
        dict(name="sigma_c64_m5", kind="sigma", prec=1, nc=6, no=25, nv=380, naux=1520, m=5),
        dict(name="sigma_split_m10", kind="sigma", prec=2, nc=6, no=60, nv=300, naux=1500, m=10),
        # eight molecules of half the batch workload's size together
        dict(name="batch_c64_m8", kind="batch", prec=1, nc=6, scale=0.5, m=8),
        # a new geometry: everything before the first sigma
        dict(name="setup_block", kind="setup", prec=0, nc=6, no=60, nv=300, naux=1500),
        # gradients of six roots
        dict(name="adjoint_k6", kind="adjoint", prec=0, nc=6, no=35, nv=250, naux=1000, k=6),
        # a whole solve of a small molecule
        dict(name="solve_k6", kind="solve", prec=0, nc=6, no=20, nv=100, naux=400, k=6),
        # oscillator strengths of the roots found
        dict(name="transition_k6", kind="transition", prec=0, nc=6, no=25, nv=200, naux=800, k=6),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Sizes spread over the ranges of the listed cases; the naux / nv ratio is
    that of the configurations (3 to 5)."""
    kind = rng.choice(["sigma"] * 6 + ["batch", "setup", "adjoint", "solve", "transition"])
    nc = rng.choice([2, 4, 6, 6])
    while True:
        ratio = rng.uniform(3.0, 5.0)
        if kind == "sigma":
            no, nv, m = _log(rng, 8, 120), _log(rng, 40, 600), _log(rng, 1, 16)
            c = dict(kind=kind, prec=rng.choice([0, 0, 0, 1, 2]), nc=nc, no=no, nv=nv, naux=int(ratio * nv), m=m)
            if _handle_bytes(c) > 40e9 or 16.0 * m * _dim(c) > 8e9 or work(c)["flops"] > 2.6e13:
                continue
        elif kind == "batch":
            c = dict(kind=kind, prec=rng.choice([0, 1, 1, 2]), nc=6, scale=round(rng.uniform(0.15, 0.6), 3),
                     m=_log(rng, 2, 16))
        elif kind == "setup":
            c = dict(kind=kind, prec=0, nc=nc, no=_log(rng, 8, 70), nv=_log(rng, 40, 350), naux=0)
            c["naux"] = int(ratio * c["nv"])
            if work(c)["flops"] > 4e12:
                continue
        elif kind == "adjoint":
            c = dict(kind=kind, prec=0, nc=nc, no=_log(rng, 8, 45), nv=_log(rng, 40, 260), naux=0, k=rng.randint(1, 10))
            c["naux"] = int(ratio * c["nv"])
        elif kind == "solve":
            c = dict(kind=kind, prec=0, nc=6, no=rng.randint(16, 26), nv=rng.randint(80, 125), naux=0,
                     k=rng.randint(3, 8))
            c["naux"] = int(rng.uniform(3.6, 4.4) * c["nv"])
        else:
            c = dict(kind=kind, prec=0, nc=nc, no=_log(rng, 8, 30), nv=_log(rng, 40, 210), naux=0, k=rng.randint(1, 10))
            c["naux"] = int(ratio * c["nv"])
        return c


def _batch_sizes(c):
    out = []
    for no, nv in BATCH:
        no_s, nv_s = max(1, int(round(no * c["scale"]))), max(2, int(round(nv * c["scale"])))
        out.append(dict(nc=c["nc"], no=no_s, nv=nv_s, naux=4 * nv_s))
    return out


def _dim(c):
    return c["nc"] * c["nv"] + c["nc"] * c["no"] * c["nv"] * (c["nv"] - 1) // 2


def _handle_bytes(c):
    n = c["nc"] + c["no"] + c["nv"]
    return 16.0 * c["naux"] * n * n


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _gen(seed, part):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + part)
    return g


def _cholesky(c, seed, part=0):
    """L [naux][n][n], Hermitian per slice, and eps [n]."""
    nc, no, nv, naux = c["nc"], c["no"], c["nv"], c["naux"]
    n = nc + no + nv
    g = _gen(seed, 1 + part)
    L = torch.empty((naux, n, n), dtype=C128, device="cuda")
    step = max(1, int(2e9 // (16 * n * n)))
    for p in range(0, naux, step):
        q = min(naux, p + step)
        a = torch.complex(torch.randn((q - p, n, n), generator=g, dtype=F64, device="cuda"),
                          torch.randn((q - p, n, n), generator=g, dtype=F64, device="cuda"))
        a *= 0.5 * SPREAD
        torch.add(a, a.transpose(1, 2).conj(), out=L[p:q])
        del a
    u = torch.rand(n, generator=_gen(seed, 2 + part), dtype=F64, device="cuda")
    windows = ((0, nc, -30.0, -28.0), (nc, nc + no, -1.0, -0.3), (nc + no, n, 0.1, 5.0))
    eps = torch.cat([torch.sort(lo + (hi - lo) * u[a:b])[0] for a, b, lo, hi in windows])
    return L, eps


def _vectors(seed, m, dim, part=0):
    """m trial vectors of unit norm."""
    g = _gen(seed, 3 + part)
    X = torch.empty((m, dim), dtype=C128, device="cuda")
    torch.view_as_real(X).normal_(generator=g)
    X *= 1.0 / math.sqrt(2.0 * dim)
    return X


def _dipole(c, seed):
    n = c["nc"] + c["no"] + c["nv"]
    d = torch.complex(torch.randn((3, n, n), generator=_gen(seed, 4), dtype=F64, device="cuda"),
                      torch.randn((3, n, n), generator=_gen(seed, 5), dtype=F64, device="cuda"))
    return (0.25 * (d + d.transpose(1, 2).conj())).contiguous()


def _energies(k):
    return [9.0 + 0.125 * i for i in range(k)]


def _weights(k):
    return [1.0 / (1 + i) for i in range(k)]


def _handle(c, L, eps):
    return A.adc2_setup(L, eps, c["nc"], c["no"], c["nv"], c["naux"], prec=c.get("prec", 0))


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "batch":
        hs, Xs = [], []
        for q, s in enumerate(_batch_sizes(c)):
            L, eps = _cholesky(s, seed, 16 * (q + 1))
            hs.append(A.adc2_setup(L, eps, s["nc"], s["no"], s["nv"], s["naux"], prec=c["prec"]))
            Xs.append(_vectors(seed, c["m"], hs[-1].dim, 16 * (q + 1)))
            del L
        return dict(c=c, hs=hs, X=Xs, S=[torch.empty_like(x) for x in Xs])
    L, eps = _cholesky(c, seed)
    if kind == "setup":
        return dict(c=c, L=L, eps=eps, h=None)
    h = _handle(c, L, eps)
    st = dict(c=c, h=h)
    # the caller's Cholesky vectors are needed during setup only
    big = _handle_bytes(c) > 4e9
    del L
    if big:
        torch.cuda.empty_cache()
    if kind == "sigma":
        st["X"] = _vectors(seed, c["m"], h.dim)
        st["S"] = torch.empty_like(st["X"])
    elif kind == "adjoint":
        st["X"] = _vectors(seed, c["k"], h.dim)
    elif kind == "transition":
        st["X"] = _vectors(seed, c["k"], h.dim)
        st["dip"] = _dipole(c, seed)
    return st


def run(st):
    c = st["c"]
    kind = c["kind"]
    if kind == "sigma":
        return A.adc2_sigma(st["h"], st["X"], st["S"])
    if kind == "batch":
        return A.adc2_sigma_batch(st["hs"], st["X"], st["S"])
    if kind == "setup":
        st["h"] = None          # the previous geometry's handle
        h = st["h"] = _handle(c, st["L"], st["eps"])
        return dict(m11=A.adc2_get_m11(h), diag=A.adc2_get_diag(h), e_mp2=A.adc2_mp2_energy(h))
    if kind == "adjoint":
        dL, deps = A.adc2_omega_backward(st["h"], st["X"], _weights(c["k"]))
        return dict(dL=dL, deps=deps)
    if kind == "solve":
        # energies only, as a screening program asks for them
        omega, _, _ = A.adc2_davidson(st["h"], c["k"], tol=1e-8, solver=A.ADC2_SOLVER_FOLDED, want_vectors=False)
        return np.array(omega)
    T, f = A.adc2_transition(st["h"], st["dip"], st["X"], _energies(c["k"]), order=2)
    return dict(T=T, f=f)


# --------------------------------------------------------------------------
# work of one pass
# --------------------------------------------------------------------------
def _sigma_work(c, m):
    nc, no, nv, naux = c["nc"], c["no"], c["nv"], c["naux"]
    ns = nc * nv
    flops = 8.0 * m * (2.0 * nc * no * nv * nv * naux + 2.0 * nc * nv * nv * naux + ns * ns
                       + 2.0 * nc * nc * no * nv * nv)
    nbytes = 16.0 * (naux * nv * (nv + no) + ns * ns + 2.0 * m * _dim(c))
    return nbytes, flops


def work(case):
    c = case
    kind = c["kind"]
    if kind == "sigma":
        b, f = _sigma_work(c, c["m"])
        return {"bytes": b, "flops": f}
    if kind == "batch":
        bf = [_sigma_work(s, c["m"]) for s in _batch_sizes(c)]
        return {"bytes": sum(b for b, _ in bf), "flops": sum(f for _, f in bf)}
    nc, no, nv, naux = c["nc"], c["no"], c["nv"], c["naux"]
    o, ns, n = nc + no, nc * nv, nc + no + nv
    mp2 = 4.0 * naux * (o * nv) ** 2                       # (ak|cl), each pair once
    m11 = 4.0 * o * o * nv ** 3 + 8.0 * ns * ns * o * nv   # pair terms of the singles block
    if kind == "setup":
        return {"bytes": 16.0 * (2.0 * naux * n * n + ns * ns) + 8.0 * _dim(c), "flops": mp2 + m11}
    k = c["k"]
    b, f = _sigma_work(c, k)
    if kind == "adjoint":
        return {"bytes": 16.0 * (2.0 * naux * n * n + k * _dim(c)), "flops": f + 3.0 * mp2 + 2.0 * m11}
    if kind == "solve":   # at least ten products per root
        return {"bytes": 10.0 * b, "flops": 10.0 * f}
    return {"bytes": 16.0 * (naux * n * n + k * _dim(c)),
            "flops": mp2 + 4.0 * naux * nv ** 4 + 8.0 * nc * o * nv ** 4 + 16.0 * nc * o * nv * nv * o * nv}


# --------------------------------------------------------------------------
# the same in plain torch, 64 bits
# --------------------------------------------------------------------------
class _Plain:
    """CVS-ADC(2) from the definitions: <pq||rs> = (pr|qs) - (ps|qr),
    (pq|rs) = sum_P L_pq L_rs, D^{ab}_{ij} = e_a + e_b - e_i - e_j."""

    def __init__(self, c, L, eps):
        self.nc, self.no, self.nv, self.naux = c["nc"], c["no"], c["nv"], c["naux"]
        self.o = o = self.nc + self.no
        self.L, self.eps = L, eps
        self.eo, self.ev = eps[:o], eps[o:]
        self.Lvv = L[:, o:, o:]
        # L_ak as [(k, a)][P], k over all occupied
        self.Lka = L[:, o:, :o].permute(2, 1, 0).reshape(o * self.nv, self.naux)

    def slab(self, k):
        """<ac||kl> for one occupied k as [a][c][l], and its denominators."""
        o, nv = self.o, self.nv
        V = (self.Lka[k * nv:(k + 1) * nv] @ self.Lka.T).reshape(nv, o, nv)     # (ak|cl) [a][l][c]
        W = V.permute(0, 2, 1) - V.permute(2, 0, 1)
        D = self.ev[:, None, None] + self.ev[None, :, None] - self.eo[k] - self.eo[None, None, :]
        return W, D

    def m11(self):
        nc, nv, o = self.nc, self.nv, self.o
        ns = nc * nv
        vv = torch.zeros((nv, nv), dtype=C128, device=self.L.device)
        e2 = torch.zeros((), dtype=F64, device=self.L.device)
        core, coreD = [], []
        for k in range(o):
            W, D = self.slab(k)
            T = W / D
            vv = vv + T.reshape(nv, -1) @ W.reshape(nv, -1).conj().T
            e2 = e2 - 0.25 * (W.abs() ** 2 / D).sum()
            if k < nc:
                core.append(W.permute(0, 2, 1).reshape(nv, -1))     # [a][(k', c)]
                coreD.append(T.permute(0, 2, 1).reshape(nv, -1))
        vv = 0.25 * (vv + vv.conj().T)
        G, GD = torch.stack(core), torch.stack(coreD)               # [I][a][(k, c)]
        q = GD.reshape(nc, -1) @ G.reshape(nc, -1).conj().T         # sum tau_I conj(W_J)
        q = 0.25 * (q + q.conj().T)                                 # [I][J]
        t3 = GD.reshape(ns, -1) @ G.reshape(ns, -1).conj().T
        t3 = -0.5 * (t3 + t3.conj().T)
        L, C, U = self.L, slice(0, nc), slice(o, o + nv)
        # <aJ||Ib> = (aI|Jb) - (ab|JI)
        aI = L[:, U, C].permute(2, 1, 0).reshape(ns, -1)            # [(I, a)][P]
        Jb = L[:, C, U].permute(1, 2, 0).reshape(ns, -1)            # [(J, b)][P]
        m = t3 + aI @ Jb.T
        ab = L[:, U, U].reshape(self.naux, -1).T @ L[:, C, C].reshape(self.naux, -1)
        ab = ab.reshape(nv, nv, nc, nc)                             # (ab|JI) [a][b][J][I]
        m = m.reshape(nc, nv, nc, nv) - ab.permute(3, 0, 2, 1)
        eyec = torch.eye(nc, dtype=C128, device=L.device)
        eyev = torch.eye(nv, dtype=C128, device=L.device)
        zero = self.ev[None, :] - self.eo[:nc, None]
        m = m + eyec[:, None, :, None] * vv[None, :, None, :] + q[:, None, :, None] * eyev[None, :, None, :]
        m = m + zero[:, :, None, None] * eyec[:, None, :, None] * eyev[None, :, None, :]
        return m.reshape(ns, ns), e2

    def doubles(self):
        """D of the packed doubles, [I][j][a<b]."""
        ia, ib = torch.triu_indices(self.nv, self.nv, 1, device=self.L.device)
        pair = self.ev[ia] + self.ev[ib]
        hole = self.eo[:self.nc, None] + self.eo[None, self.nc:]
        return (pair[None, None, :] - hole[:, :, None]), ia, ib

    def light(self, I):
        """<Ka||Ij> = (KI|aj) - (Kj|aI) as [j][K][a]."""
        nc, nv, o = self.nc, self.nv, self.o
        L, C, V, U = self.L, slice(0, nc), slice(nc, o), slice(o, o + nv)
        no = self.no
        aj = L[:, U, V].reshape(self.naux, -1)                       # [P][(a, j)]
        x = (L[:, C, I].T @ aj).reshape(nc, nv, no)
        y = (L[:, C, V].reshape(self.naux, -1).T @ L[:, U, I]).reshape(nc, no, nv)
        return x.permute(2, 0, 1) - y.permute(1, 0, 2)

    def sigma(self, X, m11=None):
        nc, nv, no, o = self.nc, self.nv, self.no, self.o
        ns = nc * nv
        if m11 is None:
            m11, _ = self.m11()
        D, ia, ib = self.doubles()
        Lva = self.Lvv.reshape(-1, nv)                               # [(P, a)][c]
        Lvat = self.Lvv.transpose(1, 2).reshape(-1, nv)              # [(P, c)][a]
        Ljb = self.L[:, o:, nc:o].permute(0, 2, 1).reshape(self.naux, -1)    # [P][(j, b)]
        lights = [self.light(I) for I in range(nc)]
        rows = []
        for x in X:
            r1 = x[:ns].reshape(nc, nv)
            x2 = x[ns:].reshape(nc, no, -1)
            s1 = (m11 @ x[:ns]).reshape(nc, nv)
            out2 = []
            add1 = [torch.zeros(nv, dtype=C128, device=x.device) for _ in range(nc)]
            for I in range(nc):
                g = lights[I]
                XP = (Lva @ r1[I]).reshape(self.naux, nv)            # [P][a]
                Z = (XP.T @ Ljb).reshape(nv, no, nv).permute(1, 0, 2)          # [j][a][b]
                Z = Z + g.transpose(1, 2) @ r1                       # sum_K <Ka||Ij> r_Kb
                s2 = Z[:, ia, ib] - Z[:, ib, ia] + D[I] * x2[I]
                out2.append(s2)
                R = torch.zeros((no, nv, nv), dtype=C128, device=x.device)
                R[:, ia, ib] = x2[I]
                R = R - R.transpose(1, 2)                            # [j][c][d]
                # Y^P_c = sum_jd conj(L_dj) R_jcd
                Y = Ljb.conj() @ R.transpose(1, 2).reshape(no * nv, nv)        # [P][c]
                add1[I] = add1[I] + Lvat.T @ Y.reshape(-1)
                # - sum_jb conj(<Kb||Ij>) R_jab
                t = torch.matmul(R, g.conj().transpose(1, 2).contiguous()).sum(0)    # [a][K]
                for K in range(nc):
                    add1[K] = add1[K] - t[:, K]
            rows.append(torch.cat([(s1 + torch.stack(add1)).reshape(-1), torch.stack(out2).reshape(-1)]))
        return torch.stack(rows)

    def roots(self, k):
        """Lowest k eigenvalues below min D by exact elimination of the doubles."""
        nc, nv, no = self.nc, self.nv, self.no
        ns, o = nc * nv, self.o
        m11, _ = self.m11()
        D, ia, ib = self.doubles()
        nd = no * ia.numel()
        Lvo = self.L[:, o:, self.nc:o]
        base = torch.empty((no, ia.numel(), nv), dtype=C128, device=self.L.device)   # <ab||cj>
        for j in range(no):
            V = (self.Lvv.reshape(self.naux, -1).T @ Lvo[:, :, j]).reshape(nv, nv, nv)   # (ac|bj) [a][c][b]
            V = V.transpose(1, 2)                                                       # [a][b][c]
            base[j] = V[ia, ib] - V[ib, ia]
            del V
        pairs = torch.arange(ia.numel(), device=self.L.device)
        blocks = []
        for I in range(nc):
            M = torch.zeros((no, ia.numel(), nc, nv), dtype=C128, device=self.L.device)
            M[:, :, I, :] = base
            g = self.light(I)                                        # [j][K][a]
            for K in range(nc):
                M[:, pairs, K, ia] -= g[:, K][:, ib]
                M[:, pairs, K, ib] += g[:, K][:, ia]
            blocks.append(M.reshape(nd, ns))
        Df = D.reshape(nc, nd)
        dmin = float(D.min())

        def at(w, j):
            Am = m11.clone()
            for I in range(nc):
                Am += blocks[I].conj().T @ (blocks[I] / (w - Df[I])[:, None])
            Am = Am.cpu().numpy()
            ev, vec = np.linalg.eigh(0.5 * (Am + Am.conj().T))
            y = torch.from_numpy(vec[:, j].copy()).to(self.L.device)
            x2 = sum(float((((b @ y) / (w - Df[I])).abs() ** 2).sum()) for I, b in enumerate(blocks))
            return float(ev[j]), x2

        out = []
        w = dmin - 40.0
        for j in range(k):
            for _ in range(30):
                lam, x2 = at(w, j)
                new = w + (lam - w) / (1.0 + x2)
                if new >= dmin:
                    new = 0.5 * (w + dmin)
                done = abs(new - w) <= 1e-12 * max(1.0, abs(w))
                w = new
                if done:
                    break
            out.append(w)
        return np.array(out)

    def transition(self, dip, X, omega):
        nc, nv, no, o, naux = self.nc, self.nv, self.no, self.o, self.naux
        ns = nc * nv
        L = self.L
        tau = torch.empty((nv, nv, o, o), dtype=C128, device=L.device)       # [a][b][i][j]
        for i in range(o):
            W, D = self.slab(i)
            tau[:, :, i, :] = W / D
        Loo = L[:, :o, :o]
        Lov = L[:, :o, o:]                                            # L_kc
        # Y_i[P][a] = sum_kc L_kc tau^{ac}_{ik}
        Y = (Lov.reshape(naux, -1) @ tau.permute(3, 1, 2, 0).reshape(o * nv, o * nv)).reshape(naux, o, nv)
        n1 = torch.stack([self.Lvv.permute(1, 0, 2).reshape(nv, -1) @ Y[:, i].reshape(-1) for i in range(o)])
        n2 = (Loo.permute(2, 0, 1).reshape(o, -1) @ Y.reshape(-1, nv))
        s = (n1 - n2) / (self.ev[None, :] - self.eo[:, None])          # [i][a]
        # doubles u for (I core, j)
        tI = tau[:, :, :nc, :].reshape(nv * nv, nc * o)
        u = torch.empty((nv, nv, nc, o), dtype=C128, device=L.device)
        vv = self.Lvv.reshape(naux, -1)
        for a in range(nv):
            G = (self.Lvv[:, a].T @ vv).reshape(nv, nv, nv)            # (ac|bd) [c][b][d]
            u[a] = (G.permute(1, 0, 2).reshape(nv, -1) @ tI).reshape(nv, nc, o)
        hh = (Loo[:, :, :nc].reshape(naux, -1).T @ Loo.reshape(naux, -1)).reshape(o, nc, o, o)   # (kI|lj)
        u += (tau.reshape(nv * nv, o * o) @ hh.permute(0, 2, 1, 3).reshape(o * o, nc * o)).reshape(nv, nv, nc, o)
        kc = Lov.reshape(naux, -1)                                     # [P][(k, c)]
        bj = L[:, o:, :o].permute(0, 1, 2).reshape(naux, -1)           # [P][(b, j)]
        B = (kc.T @ bj).reshape(o, nv, nv, o)                          # (kc|bj) [k][c][b][j]
        B = B - (Loo.reshape(naux, -1).T @ vv).reshape(o, o, nv, nv).permute(0, 3, 2, 1)    # (kj|bc)
        r = (tau.permute(0, 2, 3, 1).reshape(nv * o, o * nv) @ B.reshape(o * nv, nv * o)).reshape(nv, o, nv, o)
        r = r.permute(0, 2, 1, 3)                                      # [a][b][i][j]
        del B
        rI, rJ = r[:, :, :nc, :], r[:, :, :, :nc].transpose(2, 3)
        u += rI - rI.transpose(0, 1) - rJ + rJ.transpose(0, 1)
        del r, rI, rJ
        u /= (self.ev[:, None, None, None] + self.ev[None, :, None, None] - self.eo[None, None, :nc, None]
              - self.eo[None, None, None, :])
        t = tau.reshape(nv, -1)
        rho = t @ t.conj().T                                           # [a][c]
        t = tau.permute(2, 0, 1, 3).reshape(o, -1)
        sig = t @ t.conj().T                                           # [i][k]
        t = tau.permute(2, 0, 3, 1).reshape(o * nv, -1)                # [(i, a)][(l, b)]
        P = t[:ns] @ t.conj().T                                        # [(I, a)][(k, c)]
        _, ia, ib = self.doubles()
        T = []
        for d in dip:
            doo, dov, dvo, dvv = d[:o, :o], d[:o, o:], d[o:, :o], d[o:, o:]
            f1 = dvo[:, :nc].T - (tau[:, :, :nc, :].permute(2, 0, 3, 1).reshape(ns, -1) @ dov.reshape(-1)).reshape(nc, nv)
            f1 = f1 + s[:nc] @ dvv.T - doo[:, :nc].T @ s
            f1 = f1 + (u.permute(2, 0, 3, 1).reshape(ns, -1) @ dov.reshape(-1)).reshape(nc, nv)
            f1 = f1 - 0.25 * (rho @ dvo[:, :nc]).T - 0.25 * sig[:nc] @ dvo.T
            f1 = f1 + 0.5 * (P @ dvo.T.reshape(-1)).reshape(nc, nv)
            tIj = tau[:, :, :nc, nc:]
            pv = (dvv @ tIj.reshape(nv, -1)).reshape(nv, nv, nc, no)
            pv = pv - pv.transpose(0, 1)
            po = torch.tensordot(tau[:, :, :, nc:], doo[:, :nc], dims=([2], [0])).permute(0, 1, 3, 2)
            po = po + torch.tensordot(tau[:, :, :nc, :], doo[:, nc:], dims=([3], [0]))
            f2 = -(pv - po)[ia, ib].permute(1, 2, 0).reshape(-1)
            T.append(X.conj() @ torch.cat([f1.reshape(-1), f2]))
        T = torch.stack(T, dim=1)                                      # [k][3]
        om = torch.tensor(omega, dtype=F64, device=L.device)
        return T, (2.0 / 3.0) * om * (T.abs() ** 2).sum(1)


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "batch":
        out = []
        for q, s in enumerate(_batch_sizes(c)):
            L, eps = _cholesky(s, seed, 16 * (q + 1))
            out.append(_Plain(s, L, eps).sigma(_vectors(seed, c["m"], _dim(s), 16 * (q + 1))))
            del L
        return out
    L, eps = _cholesky(c, seed)
    if kind == "sigma":
        return _Plain(c, L, eps).sigma(_vectors(seed, c["m"], _dim(c)))
    if kind == "setup":
        p = _Plain(c, L, eps)
        m, e2 = p.m11()
        return dict(m11=m, diag=torch.cat([torch.diagonal(m).real, p.doubles()[0].reshape(-1)]), e_mp2=float(e2))
    if kind == "adjoint":
        if (c["nc"] + c["no"]) * c["nv"] > 11000:   # the recorded graph would not fit
            return None
        X = _vectors(seed, c["k"], _dim(c))
        w = torch.tensor(_weights(c["k"]), dtype=F64, device="cuda") / (X.abs() ** 2).sum(1)
        L = L.requires_grad_(True)
        eps = eps.requires_grad_(True)
        S = _Plain(c, L, eps).sigma(X)
        (w * (X.conj() * S).sum(1).real).sum().backward()
        g = L.grad
        return dict(dL=0.5 * (g + g.transpose(1, 2).conj()), deps=eps.grad)
    if kind == "solve":
        return _Plain(c, L, eps).roots(c["k"])
    T, f = _Plain(c, L, eps).transition(_dipole(c, seed), _vectors(seed, c["k"], _dim(c)), _energies(c["k"]))
    return dict(T=T.cpu().numpy(), f=f.cpu().numpy())
