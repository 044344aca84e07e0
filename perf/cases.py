"""The work that is timed when the library's speed is looked at: products,
eigensolves, density matrices and gradients over spaces of 49 to 16000 strings
per spin, through the entry points that a program calls.

Strings are drawn as ``inputs.sample_strings`` draws them (the Hartree-Fock
string and excitations of geometrically distributed rank), many at a time;
integrals are ``inputs.make_integrals`` with orbital energies of -10 to 2, the
range of a molecule's valence and virtual levels.  Every seed gives other
integrals, other strings and other vectors.  A case holds the orbitals, the
electrons and the strings of each spin; ``kind`` says which call it makes.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2601_16169_amd import autograd, inputs, sqd

DEV = "cuda:0"
TOL = 3e-11      # eigensolves: tight enough for gradients, above the rounding of a product


def _case(name, kind, norb, nea, neb, na, nb, **more):
    return dict(name=name, kind=kind, norb=norb, nalpha=nea, nbeta=neb, na=na, nb=nb, **more)


def listed():
    return [
        # full CI of 8 orbitals (4,900 determinants): the smallest product in
        # use, all launches and latency
        _case("sigma_full8", "sigma", 8, 4, 4, 70, 70, fp32=False),
        # unequal spins and odd string counts: an ordinary sampled space of an
        # open-shell system
        _case("sigma_odd", "sigma", 24, 8, 7, 1237, 731, fp32=False),
        # the 4.0e6-determinant workload's product, in both precisions (FP32 is
        # the first phase of a mixed-precision solve)
        _case("sigma_2000", "sigma", 16, 8, 8, 2000, 2000, fp32=False),
        _case("sigma_2000_fp32", "sigma", 16, 8, 8, 2000, 2000, fp32=True),
        # the 2.56e8-determinant product: rows too long for the LDS
        _case("sigma_16000", "sigma", 36, 12, 12, 16000, 16000, fp32=False),
        # a small solve in FP64: latency of an iteration
        _case("davidson_small", "davidson", 10, 5, 5, 252, 252, mixed=False),
        # the 4.0e6-determinant solve, mixed precision (a solver's default where
        # time matters)
        _case("davidson_2000", "davidson", 16, 8, 8, 2000, 2000, mixed=True),
        # the sampling loop's many uneven spaces, solved together
        _case("batched", "batched", 24, 8, 8, 200, 1200, nspace=16, mixed=True),
        # low-lying states of a middling space with unequal spins
        _case("roots", "roots", 16, 7, 6, 801, 643, nroots=3),
        # the stored Hamiltonian's product, where memory allows it
        _case("stored", "stored", 16, 8, 8, 1001, 903),
        # 1- and 2-RDM of the 1.6e7-determinant workload
        _case("rdm_4000", "rdm", 20, 7, 7, 4000, 4000),
        # one step of an orbital or geometry optimisation: new strings, new
        # tables, the energy and its gradient
        _case("gradient", "gradient", 12, 6, 5, 350, 283),
    ]


def draw(rng):
    kind = rng.choice(["sigma"] * 5 + ["davidson"] * 2 + ["batched", "roots", "stored", "rdm", "gradient"])
    lo, hi = {"sigma": (50, 13000), "davidson": (50, 1900), "batched": (100, 600), "roots": (60, 800),
              "stored": (60, 900), "rdm": (60, 3900), "gradient": (50, 350)}[kind]
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    m = max(49, min(hi, int(round(n * math.exp(rng.uniform(-0.6, 0.6))))))
    if n < 400:
        norb, ne = rng.randint(10, 14), 5
    elif n < 2500:
        norb, ne = rng.randint(15, 24), 7
    else:
        norb, ne = (rng.randint(18, 20), 7) if kind == "rdm" else (rng.randint(30, 36), 11)
    nea, neb = ne, ne - rng.randint(0, 1)
    m = min(m, math.comb(norb, neb))
    n = min(n, math.comb(norb, nea))
    c = dict(kind=kind, norb=norb, nalpha=nea, nbeta=neb, na=n, nb=m)
    if kind == "sigma":
        c["fp32"] = rng.random() < 0.3
    elif kind == "davidson":
        c["mixed"] = rng.random() < 0.5
    elif kind == "batched":
        c.update(nbeta=nea, na=n, nb=min(n + m, math.comb(norb, nea)), nspace=rng.randint(3, 16), mixed=rng.random() < 0.5)
    elif kind == "roots":
        c["nroots"] = rng.randint(2, 4)
    return c


def _strings(norb, n, count, rng):
    """count distinct strings, ascending: the HF string and k-fold excitations
    of it, k geometric, or a random subset where most strings are wanted."""
    if 2 * count > math.comb(norb, n):
        every = inputs.all_strings(norb, n)
        keep = rng.permutation(len(every) - 1)[: count - 1] + 1
        return np.sort(np.concatenate([every[:1], every[keep]]))   # the HF string is the lowest
    kmax = min(n, norb - n)
    got = np.array([inputs.hf_string(n)], dtype=np.uint64)
    while len(got) < count:
        draws = 2 * count + 64
        k = np.minimum(rng.geometric(0.4, draws), kmax)[:, None]
        occ = np.argsort(np.argsort(rng.random((draws, n)), axis=1), axis=1) >= k
        vir = np.argsort(np.argsort(rng.random((draws, norb - n)), axis=1), axis=1) < k
        bits = np.concatenate([occ, vir], axis=1).astype(np.uint64)
        s = (bits << np.arange(norb, dtype=np.uint64)).sum(axis=1, dtype=np.uint64)
        both = np.concatenate([got, s])
        _, first = np.unique(both, return_index=True)
        got = both[np.sort(first)]
    return np.sort(got[:count])


def _inputs(case, seed):
    """(integrals, list of (alpha strings, beta strings)) of a case."""
    rng = np.random.default_rng(seed)
    norb = case["norb"]
    ints = inputs.make_integrals(norb, 3 * norb, seed=int(rng.integers(1 << 31)), diag_range=(-10.0, 2.0))
    if case["kind"] == "batched":
        sets = []
        for n in np.geomspace(case["na"], case["nb"], case["nspace"]):
            s = _strings(norb, case["nalpha"], int(n), rng)
            sets.append((s, s.copy()))
        return ints, sets
    return ints, [(_strings(norb, case["nalpha"], case["na"], rng), _strings(norb, case["nbeta"], case["nb"], rng))]


def _vector(case, seed):
    """A normalised vector, dim doubles."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 1)
    c = torch.randn(case["na"] * case["nb"], dtype=torch.float64, device=DEV, generator=g)
    return c / c.norm()


def prepare(case, seed):
    kind = case["kind"]
    ints, sets = _inputs(case, seed)
    ctx = sqd.Context(0)
    ctx.set_hamiltonian(ints.h, ints.eri, ints.ecore)
    s = {"case": case, "ctx": ctx}
    if kind == "gradient":
        s["strings"] = sets[0]
        s["h"] = torch.tensor(ints.h, requires_grad=True)
        s["eri"] = torch.tensor(ints.eri, requires_grad=True)
        return s
    s["spaces"] = [ctx.build_space(case["nalpha"], case["nbeta"], a, b) for a, b in sets]
    if kind in ("sigma", "stored", "rdm"):
        s["c"] = _vector(case, seed)
        s["out"] = torch.empty_like(s["c"])
    if kind == "stored":
        s["spaces"][0].store_hamiltonian()
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "gradient":
        space = ctx.build_space(case["nalpha"], case["nbeta"], *s["strings"])
        s["h"].grad = s["eri"].grad = None
        e = autograd.energy(s["h"], s["eri"], space, tol=TOL)
        e.backward()
        space.close()
        return {"energy": e.detach(), "dh": s["h"].grad, "deri": s["eri"].grad}
    space = s["spaces"][0]
    if kind == "sigma":
        return space.sigma(s["c"], out=s["out"], precision=sqd.FP32 if case["fp32"] else sqd.FP64)
    if kind == "stored":
        return space.spmv(s["c"], out=s["out"])
    if kind == "rdm":
        return space.rdm(s["c"])
    if kind == "davidson":
        e, x, _ = space.davidson(tol=TOL, max_iter=400, mode=sqd.DAV_MIXED if case["mixed"] else sqd.DAV_FP64)
        return {"energy": e, "vector": x}
    if kind == "roots":
        e, x, _ = space.davidson_block(case["nroots"], tol=TOL, max_iter=400)
        return {"energies": list(e), "vectors": x}
    e, x, _, _ = ctx.davidson_batched(s["spaces"], tol=TOL, max_iter=400, mode=sqd.DAV_MIXED if case["mixed"] else sqd.DAV_FP64)
    return {"energies": list(e), "vectors": list(x)}


# ---- what a pass cannot do without -----------------------------------------

def _links(strings, norb):
    """Mean singles and doubles per string, from 256 of the strings."""
    o = ((strings[:, None] >> np.arange(norb, dtype=np.uint64)) & np.uint64(1)).astype(np.float32)
    some = o[np.linspace(0, len(o) - 1, min(256, len(o))).astype(int)]
    deg = o[0].sum() - some @ o.T
    return float((deg == 1).sum()) / len(some), float((deg == 2).sum()) / len(some)


@functools.lru_cache(maxsize=None)
def _work(items):
    case = dict(items)
    kind, norb = case["kind"], case["norb"]
    _, sets = _inputs(case, 1)
    flops = bytes_ = 0.0
    for a, b in sets:
        (sa, da), (sb, db) = _links(a, norb), _links(b, norb)
        na, nb = len(a), len(b)
        dim = na * nb
        conn = dim * (1 + sa + da + sb + db + sa * sb)    # elements of H among the determinants
        if kind == "stored":
            flops, bytes_ = flops + 2 * conn, bytes_ + 12 * conn + 24 * dim
        elif kind == "rdm":
            # overlaps of the rows and columns of C at the connected pairs,
            # and a product for each pair of singles
            flops += 2 * dim * (1 + sa + da + sb + db + (sa + case["nalpha"]) * (sb + case["nbeta"]))
            bytes_ += 8 * dim + 8 * norb ** 4
        elif kind == "sigma":
            flops, bytes_ = flops + 2 * conn, bytes_ + 16 * dim
        else:
            # some forty iterations to the tolerance, each a product and a
            # pass over about twelve basis vectors and their products
            it = 40 * case.get("nroots", 1)
            flops += it * (2 * conn + 60 * dim)
            bytes_ += it * 8 * dim * 26
    return bytes_, flops


def work(case):
    b, f = _work(tuple(sorted((k, v) for k, v in case.items() if k != "name")))
    return {"bytes": b, "flops": f}


# ---- the same in plain torch, in 64 bits ------------------------------------

class _Spin:
    """Connections within one spin's strings, on the device."""

    def __init__(self, strings, h, g, norb):
        sh = torch.arange(norb, device=DEV)
        self.n, self.norb = len(strings), norb
        self.occ = o = ((torch.tensor(strings.astype(np.int64), device=DEV)[:, None] >> sh) & 1).to(torch.int8)
        below = o.cumsum(1, dtype=torch.int16) - o         # occupied below each orbital
        f = o.double()
        deg = f[0].sum().float() - f.float() @ f.float().T
        J = torch.einsum("ppqq->pq", g) - torch.einsum("pqqp->pq", g)
        self.same = torch.zeros(self.n, self.n, dtype=torch.float64, device=DEV)
        diag = f @ h.diagonal() + 0.5 * ((f @ J) * f).sum(1)

        def count(t, p):
            return below[t, p].long()

        # singles: I = a+_a a_i J
        I, K = (deg == 1).nonzero(as_tuple=True)
        d = o[I] - o[K]
        a, i = d.argmax(1), d.argmin(1)
        sign = 1 - 2 * ((count(K, i) + count(K, a) - (i < a).long()) % 2)
        self.I, self.K, self.a, self.i, self.s = I, K, a, i, sign.double()
        mean = h[a, i].clone()
        for k in range(norb):
            mean += f[K, k] * (g[a, i, k, k] - g[a, k, k, i])
        self.same[I, K] = self.s * mean
        # doubles: I = a+_a a+_b a_j a_i J, i < j, a < b
        I, K = (deg == 2).nonzero(as_tuple=True)
        d = o[I] - o[K]
        a, i = d.argmax(1), d.argmin(1)
        d[torch.arange(len(I), device=DEV), a] = 0
        d[torch.arange(len(I), device=DEV), i] = 0
        b, j = d.argmax(1), d.argmin(1)
        a, b, i, j = torch.minimum(a, b), torch.maximum(a, b), torch.minimum(i, j), torch.maximum(i, j)
        turn = count(K, i) + count(K, j) - 1
        turn += count(K, b) - (i < b).long() - (j < b).long() + count(K, a) - (i < a).long() - (j < a).long()
        self.dI, self.dK, self.da, self.db, self.di, self.dj = I, K, a, b, i, j
        self.ds = (1 - 2 * (turn % 2)).double()
        self.same[I, K] = self.ds * (g[a, i, b, j] - g[a, j, b, i])
        self.same.diagonal().copy_(diag)
        self.diag = diag
        # every <I| a+_p a_q |J>, the diagonal ones included, by pair
        t, p = o.nonzero(as_tuple=True)
        self.eI = torch.cat([self.I, t])
        self.eK = torch.cat([self.K, t])
        self.ep = torch.cat([self.a * norb + self.i, p * norb + p])
        self.es = torch.cat([self.s, torch.ones(len(t), dtype=torch.float64, device=DEV)])

    def by_pair(self):
        order = torch.argsort(self.ep)
        ends = torch.searchsorted(self.ep[order].contiguous(), torch.arange(self.norb ** 2 + 1, device=DEV)).tolist()
        return [order[x:y] for x, y in zip(ends[:-1], ends[1:])]


class _Plain:
    """H = H_alpha + H_beta + sum (pq|rs) E^alpha_pq E^beta_rs as dense matrices."""

    def __init__(self, ints, a, b):
        self.norb = n = ints.norb
        self.h, self.g = torch.tensor(ints.h, device=DEV), torch.tensor(ints.eri, device=DEV)
        self.A, self.B = _Spin(a, self.h, self.g, n), _Spin(b, self.h, self.g, n)
        self.g2 = self.g.reshape(n * n, n * n)
        self.pairs = self.A.by_pair()
        B = self.B
        self.at = B.I * B.n + B.K
        self.kept = None
        if n * n * B.n ** 2 * 8 < (12 << 30):
            # every pair's matrix and rows at once, rows padded with zeros
            self.kept = torch.stack([self.mixed(p).clone() for p in range(n * n)])
            most = max(len(e) for e in self.pairs)
            e = torch.stack([torch.nn.functional.pad(e, (0, most - len(e))) for e in self.pairs])
            here = torch.arange(most, device=DEV)[None] < torch.tensor([[len(x)] for x in self.pairs], device=DEV)
            self.to, self.of, self.by = self.A.eI[e].view(-1), self.A.eK[e], self.A.es[e] * here

    def mixed(self, p):
        """sum_rs (p|rs) E^beta_rs as a dense (symmetric) matrix."""
        B, n = self.B, self.norb
        off = len(B.I)
        if not hasattr(self, "M"):
            self.M = torch.zeros(B.n * B.n, dtype=torch.float64, device=DEV)
        self.M[self.at] = B.s * self.g2[p][B.ep[:off]]
        M = self.M.view(B.n, B.n)
        M.diagonal().copy_(B.occ.double() @ self.g2[p].view(n, n).diagonal())
        return M

    def sigma(self, c):
        C = c.view(self.A.n, self.B.n)
        out = self.A.same @ C + C @ self.B.same
        if self.kept is not None:
            x = torch.bmm(C[self.of] * self.by[:, :, None], self.kept)
            return out.index_add_(0, self.to, x.view(-1, self.B.n)).view(-1)
        for p, e in enumerate(self.pairs):
            if len(e):
                out.index_add_(0, self.A.eI[e], (C[self.A.eK[e]] * self.A.es[e][:, None]) @ self.mixed(p))
        return out.view(-1)

    def diagonal(self):
        n = self.norb
        J = torch.einsum("ppqq->pq", self.g)
        x = self.A.occ.double() @ J @ self.B.occ.double().T
        return (x + self.A.diag[:, None] + self.B.diag[None, :]).view(-1)

    def rdms(self, c):
        n = self.norb
        C = c.view(self.A.n, self.B.n)
        g1 = torch.zeros(n * n, dtype=torch.float64, device=DEV)
        g2 = torch.zeros(n, n, n, n, dtype=torch.float64, device=DEV)
        flat = g2.view(-1)
        for S, P in ((self.A, C @ C.T), (self.B, C.T @ C)):
            g1.index_add_(0, S.ep, S.es * P[S.eI, S.eK])

            def add(p, q, r, s, v):
                flat.index_add_(0, ((p * n + q) * n + r) * n + s, v)

            v = S.ds * P[S.dI, S.dK]
            for p, r, s1 in ((S.da, S.db, 1), (S.db, S.da, -1)):
                for q, s, s2 in ((S.di, S.dj, 1), (S.dj, S.di, -1)):
                    add(p, q, r, s, v * (s1 * s2))
            v = S.s * P[S.I, S.K]
            for k in range(n):
                w = v * (S.occ[S.K, k] * S.occ[S.I, k]).double()
                kk = torch.full_like(S.a, k)
                add(S.a, S.i, kk, kk, w)
                add(kk, kk, S.a, S.i, w)
                add(S.a, kk, kk, S.i, -w)
                add(kk, S.i, S.a, kk, -w)
            d = (S.occ.double() * P.diagonal()[:, None]).T @ S.occ.double()
            p, q = (~torch.eye(n, dtype=torch.bool, device=DEV)).nonzero(as_tuple=True)
            add(p, p, q, q, d[p, q])
            add(p, q, q, p, -d[p, q])
        ab = torch.zeros(n * n, n * n, dtype=torch.float64, device=DEV)
        for p, e in enumerate(self.pairs):
            if len(e):
                X = (C[self.A.eI[e]] * self.A.es[e][:, None]).T @ C[self.A.eK[e]]
                ab[p].index_add_(0, self.B.ep, self.B.es * X[self.B.eI, self.B.eK])
        g2 += (ab + ab.T).view(n, n, n, n)
        return g1.view(n, n), g2

    def lowest(self, nroots):
        """The nroots lowest eigenpairs by block Davidson, vectors as rows, to
        residuals at the rounding of a product."""
        diag = self.diagonal()
        gen = torch.Generator(device=DEV)
        gen.manual_seed(3)
        t = 1e-3 * torch.randn(nroots, len(diag), dtype=torch.float64, device=DEV, generator=gen) / math.sqrt(len(diag))
        t[torch.arange(nroots, device=DEV), torch.argsort(diag)[:nroots]] += 1.0
        V = W = diag.new_empty(0, len(diag))
        G = torch.zeros(0, 0, dtype=torch.float64)
        best = math.inf
        for it in range(300):
            for v in t:
                for _ in range(3):      # Gram-Schmidt, repeated
                    if len(V):
                        v = v - (V * v).sum(1) @ V
                    v = v / v.norm()
                V = torch.cat([V, v[None]])
                W = torch.cat([W, self.sigma(v)[None]])
                g = (V * W[-1]).sum(1).cpu()
                G = torch.cat([torch.cat([G, g[:-1, None]], 1), g[None]])
            e, y = torch.linalg.eigh(G)
            y = y.T.contiguous().to(DEV)
            x = y[:nroots] @ V
            r = y[:nroots] @ W - e[:nroots, None].to(DEV) * x
            worst = float(r.norm(dim=1).max())
            if worst < 2e-14 * abs(float(e[0])) or (worst < 1e-12 * abs(float(e[0])) and worst > 0.5 * best):
                break
            best = min(best, worst)
            if len(V) + nroots > 40:
                k = 3 * nroots
                V, W, G = y[:k] @ V, y[:k] @ W, torch.diag(e[:k])
            den = e[:nroots, None].to(DEV) - diag
            t = r / torch.where(den.abs() < 1e-8, torch.full_like(den, 1e-8), den)
        x = x / x.norm(dim=1, keepdim=True)
        top = x.gather(1, x.abs().argmax(1, keepdim=True))
        return e[:nroots].tolist(), x * torch.sign(top)


def exact(case, seed):
    kind = case["kind"]
    ints, sets = _inputs(case, seed)
    if kind == "batched":
        # the larger spaces would take too long one after another
        e, x = zip(*(_Plain(ints, a, b).lowest(1) if len(a) <= 600 else ([None], [None]) for a, b in sets))
        return {"energies": [v[0] for v in e], "vectors": [v[0] for v in x]}
    P = _Plain(ints, *sets[0])
    if kind in ("sigma", "stored"):
        return P.sigma(_vector(case, seed))
    if kind == "rdm":
        return P.rdms(_vector(case, seed))
    e, x = P.lowest(case.get("nroots", 1))
    if kind == "davidson":
        return {"energy": e[0], "vector": x[0]}
    if kind == "roots":
        return {"energies": e, "vectors": x}
    g1, g2 = P.rdms(x[0])
    return {"energy": torch.tensor(e[0], dtype=torch.float64), "dh": g1, "deri": 0.5 * g2}
