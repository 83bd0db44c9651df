"""Timed cases: what a program does with this library, through its public entry points.

``listed()`` names the fixed cases, ``draw(rng)`` gives more from the same ranges, ``prepare``
makes what a program holds before the call (points, operator, right-hand sides), ``run`` is one
pass, ``work`` counts the bytes and operations a pass cannot do without, and ``exact`` gives the
same results in 64 bits from plain torch (its own cluster tree, block lists and interpolation).
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2509_17257_amd as h2x
from paper_2509_17257_amd import workloads as W
from paper_2509_17257_amd.autograd import h2_apply

ETA = 1.0
_BYTES = {"f64": 8, "f32": 4, "bf16": 2}


def _product(geometry, n, p, leaf, m, storage="f64", ell=0.5, shift=1.0, **name):
    return dict(name, kind="product", geometry=geometry, n=n, p=p, leaf=leaf, m=m, storage=storage, ell=ell,
                shift=shift)


def listed():
    return [
        # one product of a small system: a handful of columns, every stage a few work-groups
        _product("sphere", 4096, 3, 32, 4, name="small"),
        # the product of a single right-hand side (matrix-vector product, single-vector solvers)
        _product("sphere", 65536, 4, 64, 1, name="matvec"),
        # the block product inside block CG at the benchmark's size
        _product("sphere", 65536, 4, 64, 32, name="block"),
        # many right-hand sides in one product (more columns than one tile of any kernel)
        _product("sphere", 65536, 4, 64, 100, name="wide"),
        # a higher interpolation order, for operators that need a smaller kernel error
        _product("sphere", 32768, 5, 128, 16, name="order5"),
        # the volume operator of the mixed-precision solves: its FP64 product (the largest case) ...
        _product("cube", 262144, 4, 64, 64, ell=0.25, shift=0.5, name="volume"),
        # ... its FP32 product, which the residual-replacement iterations run on ...
        _product("cube", 262144, 4, 64, 64, "f32", ell=0.25, shift=0.5, name="volume_f32"),
        # ... and a BF16 product, at an odd size and a ragged column count
        _product("cube", 99991, 4, 64, 45, "bf16", ell=0.25, shift=0.5, name="volume_bf16"),
        # many independent systems of uneven size and both ranks in one call
        dict(name="batch", kind="batch", systems=16, n_lo=2048, n_hi=32768, m=32, storage="f64"),
        # one training step on the kernel's length scale: refill, forward, backward
        dict(name="gradient", kind="gradient", geometry="sphere", n=131072, p=4, leaf=64, m=16, ell=0.5, shift=1.0,
             wrt="ell"),
        # a budget of iterations of the shared-space block CG (its m x m algebra beside the product)
        dict(name="solve_shared", kind="solve", method="shared", geometry="sphere", n=65536, p=4, leaf=64, m=32,
             ell=0.5, shift=1.0, iters=4),
        # one cycle of block GMRES on the complex Helmholtz operator (m complex columns)
        dict(name="solve_helmholtz", kind="solve", method="gmres", geometry="sphere", n=32768, p=4, leaf=64, m=8,
             ell=1.0, shift=1.0, iters=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["product"] * 6 + ["low"] * 2 + ["batch", "gradient", "solve", "solve"])
    geometry = rng.choice(["sphere", "sphere", "cube"])
    ell, shift = round(rng.uniform(0.2, 1.0), 3), rng.choice([0.5, 1.0])
    if kind == "low":
        p = rng.choice([3, 4, 4, 5])
        n = _log_int(rng, 2000, 16384 if p == 5 else 131072)
        return _product(geometry, n, p, {3: 32, 4: 64, 5: 128}[p], _log_int(rng, 1, 48 if p == 5 else 100),
                        rng.choice(["f32", "bf16"]), ell, shift)
    if kind == "product":
        p = rng.choice([2, 3, 4, 4, 4, 5])
        n = _log_int(rng, 1000, 32768 if p == 5 else 131072)
        return _product(geometry, n, p, {2: 16, 3: 32, 4: 64, 5: 128}[p], _log_int(rng, 1, 48 if p == 5 else 100), "f64",
                        ell, shift)
    if kind == "batch":
        return dict(kind="batch", systems=rng.randint(3, 24), n_lo=2048, n_hi=rng.randint(8000, 32768),
                    m=_log_int(rng, 1, 32), storage=rng.choice(["f64", "f64", "f32"]))
    if kind == "gradient":
        wrt = rng.choice(["ell", "coupling"])
        p = rng.choice([3, 4, 4])
        return dict(kind="gradient", geometry="sphere", n=_log_int(rng, 4000, 100000), p=p, leaf={3: 32, 4: 64}[p],
                    m=_log_int(rng, 1, 32), ell=ell, shift=1.0, wrt=wrt)
    method = rng.choice(["independent", "shared", "gmres"])
    p = rng.choice([3, 4])
    return dict(kind="solve", method=method, geometry="sphere", n=_log_int(rng, 2000, 65536), p=p,
                leaf={3: 32, 4: 64}[p], m=_log_int(rng, 2, 16 if method == "gmres" else 48), ell=ell, shift=1.0,
                iters=rng.randint(3, 4) if method == "shared" else rng.randint(4, 9))


# ---------------------------------------------------------------------------------------------
# inputs


def _points(case, seed):
    if case.get("wrt") == "coupling":
        seed = 1004  # the coupling matrices are fitted on a fixed geometry: their number is the cloud's
    return (W.sphere_points if case["geometry"] == "sphere" else W.cube_points)(case["n"], seed)


def _params(case):
    return dict(ell=case["ell"], shift=case["shift"], eta=ETA, leaf=case["leaf"], p=case["p"])


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _block(n, m, seed, dtype=torch.float64):
    """N(0, 1) right-hand sides on the GPU."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed)
    if dtype.is_complex:
        return torch.view_as_complex(torch.randn(n, m, 2, generator=g, device=dev, dtype=torch.float64))
    return torch.randn(n, m, generator=g, device=dev, dtype=dtype)


def _systems(case, seed):
    """The systems of a batch: (points, parameters) with n log-uniform, both ranks alternating."""
    g = np.random.default_rng(case["systems"])  # the sizes are the case's, the points the seed's
    out = []
    for i in range(case["systems"]):
        n = int(round(math.exp(g.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
        ell = float(g.uniform(0.2, 1.0))
        p = 3 + i % 2
        out.append((W.sphere_points(n, seed * 1000 + i), dict(ell=ell, shift=1.0, eta=ETA, leaf=32 if p == 3 else 64,
                                                              p=p)))
    return out


def _is_complex(case):
    return case["kind"] == "solve" and case["method"] == "gmres"


def prepare(case, seed):
    s = SimpleNamespace(case=case)
    if case["kind"] == "batch":
        s.A = h2x.Batch(_systems(case, seed), storage=case["storage"])
        s.X = _block(s.A.n, case["m"], seed + 1)
        return s
    prm = dict(_params(case), kernel="helmholtz" if _is_complex(case) else "exp")
    s.A = h2x.H2Matrix(_points(case, seed), storage=case.get("storage", "f64"), **prm)
    s.X = _block(case["n"], case["m"], seed + 1, torch.complex128 if _is_complex(case) else torch.float64)
    if case["kind"] == "gradient":
        s.dY = _block(case["n"], case["m"], seed + 2)
        if case["wrt"] == "ell":
            s.X.requires_grad_(True)
            s.ell = torch.tensor(case["ell"], dtype=torch.float64, requires_grad=True)
    return s


def run(s):
    case = s.case
    if case["kind"] == "product":
        return h2x.h2_matmul(s.A, s.X)
    if case["kind"] == "batch":
        return h2x.batch_matmul(s.A, s.X)
    if case["kind"] == "gradient":
        if case["wrt"] == "coupling":  # the adjoint product and the gradient of the coupling matrices
            dS, _, _ = h2x.h2_grad(s.A, s.X, s.dY, want_dS=True, want_dell=False)
            return {"dX": h2x.h2_matmul_adjoint(s.A, s.dY), "dS": dS}
        s.A.set_ell(case["ell"])  # every step of a fit moves the length scale
        Y = h2_apply(s.A, s.X, ell=s.ell)
        dX, dell = torch.autograd.grad(Y, (s.X, s.ell), s.dY)
        return {"Y": Y, "dX": dX, "dell": dell}
    if case["method"] == "gmres":
        X, info = h2x.block_gmres_solve(s.A, s.X, rtol=1e-14, restart=case["iters"], max_iter=case["iters"])
    else:
        X, info = h2x.block_cg_solve(s.A, s.X, rtol=1e-14, max_iter=case["iters"], variant=case["method"])
    return {"X": X, "iters": info.iters}


# ---------------------------------------------------------------------------------------------
# work


def _plan_work(pl, case, m, sb, sn):
    """(bytes of the stored operator, bytes of V, transfers and vectors, flops) of one product."""
    k, p = pl.k, round(pl.k ** (1 / 3))
    op = sb * pl.n_adm * k * k + sn * pl.near_entries
    rest = sb * pl.n * k + 8 * 3 * p * p * pl.C + 16 * pl.n * m
    fl = 2 * m * (2 * pl.n * k + 2 * pl.C * 3 * p * k + pl.n_adm * k * k + pl.near_entries)
    return op, rest, fl


def work(case):
    if case["kind"] == "batch":
        sb = _BYTES[case["storage"]]
        by = fl = 0
        for pts, prm in _systems(case, 0):
            op, rest, f = _plan_work(h2x.Plan(pts, **prm), case, case["m"], sb, max(sb, 4))
            by, fl = by + op + rest, fl + f
        return {"bytes": by, "flops": fl}
    sb = _BYTES[case.get("storage", "f64")]
    pl = h2x.Plan(_points(case, 0), **_params(case))
    op, rest, fl = _plan_work(pl, case, case["m"], sb, max(sb, 4))
    if case["kind"] == "gradient":
        entries = pl.n_adm * pl.k ** 2 + pl.near_entries
        if case["wrt"] == "coupling":  # adjoint reads the operator; dS is written
            return {"bytes": op + 2 * rest + 8 * pl.n_adm * pl.k ** 2, "flops": 2 * fl}
        # refill writes the operator, forward and backward each read it
        return {"bytes": 3 * op + 3 * rest, "flops": 3 * fl + 20 * entries}
    if case["kind"] == "solve":
        if _is_complex(case):  # complex S and N on real bases, m complex columns
            op, fl, rest = 2 * op, 4 * fl, rest + 16 * pl.n * case["m"]
            # step j of a cycle: projections on j + 1 basis blocks, the subtraction, the new block
            extra = sum(16 * pl.n * case["m"] * (2 * j + 4) for j in range(case["iters"]))
        else:
            extra = case["iters"] * 8 * pl.n * case["m"] * 7
        return {"bytes": case["iters"] * (op + rest) + extra, "flops": case["iters"] * fl}
    return {"bytes": op + rest, "flops": fl}


# ---------------------------------------------------------------------------------------------
# the same results in 64 bits, in plain torch


class _Exact:
    """The H^2 approximation of one point cloud (Chebyshev interpolation on a bisection tree), applied
    from its definition: coupling matrices and near blocks are evaluated chunk by chunk."""

    CHUNK = 1 << 25  # entries of a batch of blocks

    def __init__(self, pts, ell, shift, eta, leaf, p, helmholtz=False):
        self.dev = _device()
        self.ell, self.shift, self.p, self.k, self.n = ell, shift, p, p ** 3, len(pts)
        self.helmholtz = helmholtz
        self._tree(pts, leaf)
        self._blocks(eta)
        d = self.dev
        j = torch.arange(p, dtype=torch.float64, device=d)
        cheb = torch.cos((2 * j + 1) * math.pi / (2 * p))
        lo, hi = torch.from_numpy(self.lo).to(d), torch.from_numpy(self.hi).to(d)
        flat = hi - lo < 1e-10
        mid = 0.5 * (lo + hi)
        lo, hi = torch.where(flat, mid - 0.5e-10, lo), torch.where(flat, mid + 0.5e-10, hi)
        self.x1 = (0.5 * (lo + hi))[:, :, None] + (0.5 * (hi - lo))[:, :, None] * cheb  # C x 3 x p
        nu = torch.arange(self.k, device=d)
        self.digit = [nu % p, (nu // p) % p, nu // (p * p)]
        self.nodes = torch.stack([self.x1[:, a, self.digit[a]] for a in range(3)], 2)  # C x k x 3
        self.pts = torch.from_numpy(np.ascontiguousarray(pts[self.perm])).to(d)
        self.perm_t = torch.from_numpy(self.perm).to(d)
        lv = np.nonzero(self.son[:, 0] < 0)[0]
        self.leaf_of = np.full(len(self.first), -1, np.int64)
        self.leaf_of[lv] = np.arange(len(lv))
        self.lv = torch.from_numpy(lv).to(d)
        sz = torch.from_numpy(self.size[lv]).to(d)
        w = int(sz.max())
        at = torch.from_numpy(self.first[lv]).to(d)[:, None] + torch.arange(w, device=d)[None, :]
        self.mask = torch.arange(w, device=d)[None, :] < sz[:, None]  # leaves x w
        self.at = torch.where(self.mask, at, torch.zeros_like(at))
        self.pad = self.pts[self.at]  # leaves x w x 3

    def _tree(self, pts, leaf):
        perm, first, size, son, depth, lo, hi = np.arange(len(pts)), [], [], [], [], [], []
        todo = [(0, len(pts), 0, -1, 0)]
        while todo:
            a, cnt, dep, par, which = todo.pop()
            c = len(first)
            if par >= 0:
                son[par][which] = c
            q = pts[perm[a:a + cnt]]
            l, h = q.min(0), q.max(0)
            first.append(a), size.append(cnt), son.append([-1, -1]), depth.append(dep), lo.append(l), hi.append(h)
            dim = int(np.argmax(h - l))
            if cnt <= leaf or h[dim] == l[dim]:
                continue
            left = q[:, dim] < 0.5 * (l[dim] + h[dim])
            c0 = int(left.sum())
            if c0 in (0, cnt):
                continue
            seg = perm[a:a + cnt].copy()
            perm[a:a + c0], perm[a + c0:a + cnt] = seg[left], seg[~left]
            todo.append((a + c0, cnt - c0, dep + 1, c, 1))
            todo.append((a, c0, dep + 1, c, 0))
        self.perm, self.first, self.size = perm, np.array(first), np.array(size)
        self.son, self.depth = np.array(son), np.array(depth)
        self.lo, self.hi = np.array(lo), np.array(hi)

    def _blocks(self, eta):
        ext = self.hi - self.lo
        diam = np.sqrt((ext * ext).sum(1))
        t = s = np.zeros(1, np.int64)
        adm, near = [], []
        while len(t):
            g = np.maximum(0.0, np.maximum(self.lo[s] - self.hi[t], self.lo[t] - self.hi[s]))
            dist = np.sqrt((g * g).sum(1))
            ok = (dist > 0) & (np.maximum(diam[t], diam[s]) <= eta * dist)
            adm.append(np.stack([t[ok], s[ok]]))
            t, s = t[~ok], s[~ok]
            lt, ls = self.son[t, 0] < 0, self.son[s, 0] < 0
            near.append(np.stack([t[lt & ls], s[lt & ls]]))
            nt, ns = [], []
            for i in range(2):
                for j in range(2):
                    q = ~(lt & ls) & ((i == 0) | ~lt) & ((j == 0) | ~ls)
                    nt.append(np.where(lt[q], t[q], self.son[t[q], i]))
                    ns.append(np.where(ls[q], s[q], self.son[s[q], j]))
            t, s = np.concatenate(nt), np.concatenate(ns)
        adm, near = np.concatenate(adm, 1), np.concatenate(near, 1)
        o = np.lexsort((adm[1], adm[0]))  # by row cluster, then by column cluster
        self.adm = torch.from_numpy(adm[:, o]).to(self.dev)
        self.near = near

    def _lagrange(self, cl, x):
        """One-dimensional Lagrange values of the clusters cl at x (len(cl) x q x 3): ... x 3 x p."""
        nd = self.x1[cl][:, None]  # B x 1 x 3 x p
        out = []
        for j in range(self.p):
            v = torch.ones_like(x)
            for i in range(self.p):
                if i != j:
                    v = v * (x - nd[..., i]) / (nd[..., j] - nd[..., i])
            out.append(v)
        return torch.stack(out, 3)

    def _basis(self, cl, x):
        L = self._lagrange(cl, x)
        return L[:, :, 0][..., self.digit[0]] * L[:, :, 1][..., self.digit[1]] * L[:, :, 2][..., self.digit[2]]

    def _levels(self):
        for d in range(int(self.depth.max()), -1, -1):
            c = np.nonzero((self.depth == d) & (self.son[:, 0] >= 0))[0]
            if len(c):
                yield torch.from_numpy(c).to(self.dev), torch.from_numpy(self.son[c]).to(self.dev)

    def _chunks(self, count, each):
        step = max(1, self.CHUNK // each)
        for a in range(0, count, step):
            yield slice(a, min(count, a + step))

    def forward(self, X):
        """x-hat of every cluster (C x k x m) of X in tree order."""
        xh = torch.zeros(len(self.first), self.k, X.shape[1], dtype=X.dtype, device=self.dev)
        w = self.pad.shape[1]
        for q in self._chunks(len(self.lv), w * max(self.k, X.shape[1]) * 4):
            V = self._basis(self.lv[q], self.pad[q]) * self.mask[q][:, :, None]
            xh[self.lv[q]] = torch.bmm(V.transpose(1, 2).contiguous().to(X.dtype), X[self.at[q]])
        for c, sons in self._levels():
            for q in self._chunks(len(c), self.k * self.k * 4):
                for i in range(2):
                    s = sons[q, i]
                    E = self._basis(c[q], self.nodes[s])
                    xh[c[q]] += torch.bmm(E.transpose(1, 2).contiguous().to(X.dtype), xh[s])
        return xh

    def _kernel(self, a, b, derivative=False):
        """g between the points a (B x q x 3) and b (B x r x 3); derivative: dg / d ell."""
        r = torch.zeros(a.shape[0], a.shape[1], b.shape[1], dtype=torch.float64, device=self.dev)
        for d in range(3):
            r += (a[:, :, None, d] - b[:, None, :, d]) ** 2
        r = r.sqrt_()
        if self.helmholtz:
            f = torch.where(r == 0, torch.zeros_like(r), 1.0 / (self.n * r))
            return torch.complex(torch.cos(self.ell * r) * f, torch.sin(self.ell * r) * f)
        g = torch.exp(-r / self.ell)
        return g * r / self.ell ** 2 if derivative else g

    def _near(self, derivative=False):
        lt, ls = self.leaf_of[self.near[0]], self.leaf_of[self.near[1]]
        w = self.pad.shape[1]
        for q in self._chunks(len(lt), w * w):
            t, s = torch.from_numpy(lt[q]).to(self.dev), torch.from_numpy(ls[q]).to(self.dev)
            N = self._kernel(self.pad[t], self.pad[s], derivative)
            if not derivative:
                same = torch.nonzero(t == s)[:, 0]
                N[same] += self.shift * torch.eye(w, dtype=N.dtype, device=self.dev)
            yield t, s, N * (self.mask[t][:, :, None] & self.mask[s][:, None, :])

    def tree(self, X):
        return X[self.perm_t]

    def matmul(self, X):
        X = self.tree(X)
        xh = self.forward(X)
        yh = torch.zeros_like(xh)
        for q in self._chunks(self.adm.shape[1], self.k * self.k):
            t, s = self.adm[0, q], self.adm[1, q]
            yh.index_add_(0, t, torch.bmm(self._kernel(self.nodes[t], self.nodes[s]).to(X.dtype), xh[s]))
        for c, sons in reversed(list(self._levels())):
            for q in self._chunks(len(c), self.k * self.k * 4):
                for i in range(2):
                    s = sons[q, i]
                    yh[s] += torch.bmm(self._basis(c[q], self.nodes[s]).to(X.dtype), yh[c[q]])
        Yp = torch.zeros(len(self.lv), self.pad.shape[1], X.shape[1], dtype=X.dtype, device=self.dev)
        for q in self._chunks(len(self.lv), self.pad.shape[1] * max(self.k, X.shape[1]) * 4):
            Yp[q] = torch.bmm(self._basis(self.lv[q], self.pad[q]).to(X.dtype), yh[self.lv[q]])
        for t, s, N in self._near():
            Yp.index_add_(0, t, torch.bmm(N, X[self.at[s]]))
        Y = torch.zeros_like(X)
        Y[self.perm_t[self.at[self.mask]]] = Yp[self.mask]
        return Y

    def d_ell(self, X, dY):
        X, dY = self.tree(X), self.tree(dY)
        xh, dh = self.forward(X), self.forward(dY)
        total = torch.zeros((), dtype=torch.float64, device=self.dev)
        for q in self._chunks(self.adm.shape[1], self.k * self.k):
            t, s = self.adm[0, q], self.adm[1, q]
            total += (dh[t] * torch.bmm(self._kernel(self.nodes[t], self.nodes[s], True), xh[s])).sum()
        for t, s, N in self._near(True):
            total += (dY[self.at[t]] * torch.bmm(N, X[self.at[s]])).sum()
        return total

    def d_coupling(self, X, dY):
        xh, dh = self.forward(self.tree(X)), self.forward(self.tree(dY))
        return torch.cat([torch.bmm(dh[self.adm[0, q]], xh[self.adm[1, q]].transpose(1, 2).contiguous())
                          for q in self._chunks(self.adm.shape[1], self.k * (self.k + 2 * X.shape[1]))])


def _cg(A, B, iters, shared):
    """Block CG from zero: m independent iterations, or one shared block Krylov space."""
    X, R = torch.zeros_like(B), B.clone()
    if shared:
        P = torch.linalg.qr(R)[0]
        for _ in range(iters):
            Q = A.matmul(P)
            G = P.T @ Q
            lam = torch.linalg.solve(G, P.T @ R)
            X, R = X + P @ lam, R - Q @ lam
            P = torch.linalg.qr(R - P @ torch.linalg.solve(G, Q.T @ R))[0]
        return X
    P, rr = R.clone(), (R * R).sum(0)
    for _ in range(iters):
        Q = A.matmul(P)
        a = rr / (P * Q).sum(0)
        X, R = X + P * a, R - Q * a
        new = (R * R).sum(0)
        P, rr = R + P * (new / rr), new
    return X


def _gmres(A, B, steps):
    """One cycle of GMRES from zero, column by column on a shared product."""
    m = B.shape[1]
    beta = B.abs().square().sum(0).sqrt()
    Q = [B / beta]
    H = torch.zeros(m, steps + 1, steps, dtype=B.dtype, device=B.device)
    for j in range(steps):
        a = A.matmul(Q[j])
        for _ in range(2):
            h = [(q.conj() * a).sum(0) for q in Q]
            for i, q in enumerate(Q):
                H[:, i, j] += h[i]
                a = a - q * h[i]
        nrm = a.abs().square().sum(0).sqrt()
        H[:, j + 1, j] = nrm
        Q.append(a / nrm)
    e = torch.zeros(m, steps + 1, 1, dtype=B.dtype, device=B.device)
    e[:, 0, 0] = beta
    q, r = torch.linalg.qr(H)
    y = torch.linalg.solve_triangular(r, q.mH.contiguous() @ e, upper=True)
    return sum(Q[j] * y[:, j, 0] for j in range(steps))


def exact(case, seed):
    if case["kind"] == "batch":
        parts = _systems(case, seed)
        order = [i for p in (3, 4) for i in range(len(parts)) if parts[i][1]["p"] == p]
        X = _block(sum(len(pts) for pts, _ in parts), case["m"], seed + 1)
        out, a = [], 0
        for i in order:
            pts, prm = parts[i]
            out.append(_Exact(pts, **prm).matmul(X[a:a + len(pts)]))
            a += len(pts)
        return torch.cat(out)
    A = _Exact(_points(case, seed), **_params(case), helmholtz=_is_complex(case))
    X = _block(case["n"], case["m"], seed + 1, torch.complex128 if _is_complex(case) else torch.float64)
    if case["kind"] == "product":
        return A.matmul(X)
    if case["kind"] == "gradient":
        dY = _block(case["n"], case["m"], seed + 2)
        dX = A.matmul(dY)  # the operator is symmetric
        if case["wrt"] == "coupling":
            return {"dX": dX, "dS": A.d_coupling(X, dY)}
        return {"Y": A.matmul(X), "dX": dX, "dell": A.d_ell(X, dY)}
    if case["method"] == "gmres":
        return {"X": _gmres(A, X, case["iters"]), "iters": None}
    return {"X": _cg(A, X, case["iters"], case["method"] == "shared"), "iters": None}
