"""Workloads of the aTTN ground-state path, called as a user's program calls it.

A case names a lattice model (L x L sites, `model`), a bond dimension `m`, and
what is done with the state: one H_eff matvec at a node, a centre move across
one link and back, one local eigensolve, a sweep from a fresh state, one
lock-step sweep of several instances, or a two-body correlation matrix.
Inputs are the seeded synthetic problems of `problems/` (Haar disentanglers,
Gaussian tensors, L^2 / 4 gates).  `exact` contracts the same network in 64
bits with plain torch (operator-Schmidt factors of every rotated term, one
link at a time), independent of the library.
"""
from __future__ import annotations

import copy
import functools
import math

import numpy as np
import torch

from paper_2507_21236_amd import (ATTN_BF16X2, ATTN_F32, ATTN_F64, ATTN_HOST_ONLY, AttnBatch,
                                  AttnHandle)
from problems import make_problem

DTYPES = {"f64": ATTN_F64, "f32": ATTN_F32, "bf16x2": ATTN_BF16X2}
KRYLOV = 20   # the library's default number of Lanczos matvecs per node


def listed():
    """The cases, smallest first within each kind."""
    return [
        # the smallest useful call: a matvec of the 4 x 4 tutorial lattice, all launch latency
        dict(name="matvec_4x4_m8_f64", kind="matvec", L=4, m=8, model="ising", dtype="f64", rank=0.0),
        # a bond dimension chosen by accuracy, not by the hardware: 50 is no multiple of 16
        dict(name="matvec_8x8_m50_f64", kind="matvec", L=8, m=50, model="ising", dtype="f64", rank=0.0),
        # single precision at the bond dimension of the Heisenberg workload
        dict(name="matvec_8x8_m96_f32", kind="matvec", L=8, m=96, model="ising", dtype="f32", rank=0.0),
        # the (128, 128, 128) node shape of the largest workload
        dict(name="matvec_8x8_m128_f64", kind="matvec", L=8, m=128, model="ising", dtype="f64", rank=0.0),
        # the headline workload's heaviest node, in double and in split precision
        dict(name="matvec_16x16_m64_f64", kind="matvec", L=16, m=64, model="ising", dtype="f64", rank=0.0),
        dict(name="matvec_16x16_m64_bf16x2", kind="matvec", L=16, m=64, model="ising", dtype="bf16x2",
             rank=0.0),
        # what a sweep does between two solves: QR, absorption and the effective-operator update of
        # a link, there and back, at the headline size
        dict(name="move_16x16_m64", kind="move", L=16, m=64, model="ising", rank=0.0),
        # local eigensolves: a small node (vector steps and latency), and a ragged bond dimension
        dict(name="eigsolve_8x8_m16", kind="eigsolve", L=8, m=16, model="ising", rank=0.0),
        dict(name="eigsolve_8x8_m40", kind="eigsolve", L=8, m=40, model="ising", rank=0.0),
        # a whole run's first sweep, from raw tensors to the energy
        dict(name="sweep_8x8_m32", kind="sweep", L=8, m=32, model="ising"),
        # a scan over field strengths and bond dimensions in lock step
        dict(name="batch_8x8_m32", kind="batch", L=8, m=32, model="ising", n=4),
        # observables of the finished state: the 64 x 64 correlation matrix
        dict(name="correlation_8x8_m32", kind="correlation", L=8, m=32, model="ising"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same kinds: lattices of 4 x 4 to 16 x 16 sites, bond dimensions of 4 to
    128, odd ones among them, light and heavy nodes, every precision of a matvec."""
    kind = rng.choice(["matvec"] * 5 + ["move", "move", "eigsolve", "eigsolve", "sweep", "batch", "correlation"])
    model = rng.choice(["ising", "ising", "heisenberg_tri"])
    L = rng.choice([4, 5, 6, 8, 8, 10, 12, 16] if kind in ("matvec", "move") else [4, 5, 6, 7, 8])
    top = {"matvec": 128, "move": 96, "eigsolve": 64, "sweep": 32, "batch": 32, "correlation": 32}[kind]
    if model != "ising" or L > 8:
        top = min(top, 64)
    m = _log_int(rng, 4, top)
    if rng.random() < 0.5 and m >= 8:
        m = max(16, 16 * round(m / 16))
    elif m > (20 if kind in ("sweep", "batch") else 36 if kind == "eigsolve" else 48 if L <= 8 else 32):
        m = 16 * round(m / 16)
    case = dict(kind=kind, L=L, m=m, model=model)
    if kind == "matvec":
        case["dtype"] = rng.choice(["f64", "f64", "f32", "bf16x2"])
    if kind in ("matvec", "move", "eigsolve"):
        case["rank"] = round(0.5 * rng.random() ** 2, 3)
    if kind == "batch":
        case["n"] = rng.randint(2, 6)
    return case


# ---------------------------------------------------------------------------- inputs
def _problem(case, seed, m=None, k=0):
    field = 3.0 if k == 0 else 2.5 + ((7 * k) % 11) / 10.0
    L = case["L"]
    return make_problem("perf", L, case["model"], case["m"] if m is None else m, 1000 * seed + k, L * L // 4, h=field)


def _batch_ms(case):
    """Bond dimensions of a batch's instances: m, 3 m / 4, m / 2, m / 4, m, ..."""
    return [max(4, case["m"] * (4 - k % 4) // 4) for k in range(case["n"])]


@functools.lru_cache(maxsize=64)
def _structure(L, m, model):
    """(dims, flops) per node and the bytes of the effective operators of a problem."""
    p = make_problem("perf", L, model, m, 0, L * L // 4)
    h = AttnHandle(p, flags=ATTN_HOST_ONLY)
    info = [h.node_info(n) for n in range(h.n_nodes)]
    env_bytes, tree = h.env_bytes, _Tree(p.n_sites, m)
    h.close()
    return [i[0] for i in info], [i[2] for i in info], env_bytes, tree


def _node(case):
    """The node a case works at: rank 0 is the one with the most work, rank 1 the one with the least."""
    dims, flops, _, tree = _structure(case["L"], case["m"], case["model"])
    order = sorted(range(len(flops)), key=lambda n: (-flops[n], n))
    if case["kind"] == "move":
        order = [n for n in order if n != tree.root]
    return order[min(len(order) - 1, int(case["rank"] * len(order)))]


def _gauss(shape, seed, dtype):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, dtype=torch.float64, device="cuda").to(dtype)


def _schmidt_gauge(tn, tq, leg):
    """The pair (centre, its parent) of numpy tensors with the link between them in its Schmidt basis."""
    u, s, vt = np.linalg.svd(tn.reshape(-1, tn.shape[2]), full_matrices=False)
    sign = np.sign(vt[np.arange(len(s)), np.abs(vt).argmax(axis=1)])
    vt = vt * sign[:, None]
    tq = np.moveaxis(np.tensordot(vt, tq, axes=(1, leg)), 0, leg)
    return np.ascontiguousarray((u * (s * sign)).reshape(tn.shape)), np.ascontiguousarray(tq)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        probs = [_problem(case, seed, m, k) for k, m in enumerate(_batch_ms(case))]
        handles = [AttnHandle(p) for p in probs]
        raws = [p.raw_concat() for p in probs]
        for h, r in zip(handles, raws):
            h.init_state(r)
        return dict(kind=kind, handles=handles, raws=raws, batch=AttnBatch(handles, krylov_k=KRYLOV, precision=ATTN_F64))
    p = _problem(case, seed)
    h = AttnHandle(p)
    st = dict(kind=kind, h=h, raw=p.raw_concat())
    if kind != "sweep":
        h.init_state(st["raw"])
    if kind in ("matvec", "move", "eigsolve"):
        dims, _, _, tree = _structure(case["L"], case["m"], case["model"])
        n = st["node"] = _node(case)
        h.move_center(n)
        if kind == "move":
            # the link in its Schmidt gauge: the QR there and back then return the same state
            q = st["to"] = tree.parent[n]
            leg = tree.child[q].index(n)
            tn, tq = _schmidt_gauge(h.get_tensor(n), h.get_tensor(q), leg)
            h.set_tensor(n, tn)
            h.set_tensor(q, tq)
            h.update_env(q, leg)
        if kind == "matvec":
            st["dtype"] = DTYPES[case["dtype"]]
            st["x"] = _gauss(dims[n], seed + 1, torch.float64 if case["dtype"] == "f64" else torch.float32)
            st["y"] = torch.empty_like(st["x"])
        elif kind == "move":
            st["x"], st["xq"] = _gauss(dims[n], seed + 1, torch.float64), _gauss(dims[q], seed + 2, torch.float64)
            st["y"], st["yq"] = torch.empty_like(st["x"]), torch.empty_like(st["xq"])
        else:
            st["guess"] = h.get_tensor(n)
    torch.cuda.synchronize()
    return st


SIGMA_X = np.array([[0.0, 1.0], [1.0, 0.0]])
SIGMA_Z = np.array([[1.0, 0.0], [0.0, -1.0]])


def _magnetisation(h):
    """<sigma_x> of every site: what a run reports of its state beside the energy."""
    return h.measure([[(s, SIGMA_X)] for s in range(h.problem.n_sites)])


def run(st):
    kind = st["kind"]
    if kind == "batch":
        for h, r in zip(st["handles"], st["raws"]):
            h.init_state(r)
        energies, _ = st["batch"].sweep(1)
        return [energies] + [_magnetisation(h) for h in st["handles"]]
    h = st["h"]
    if kind == "matvec":
        h.heff_apply(st["node"], st["x"], st["y"], dtype=st["dtype"])
        return st["y"]
    if kind == "move":
        h.move_center(st["to"])
        h.heff_apply(st["to"], st["xq"], st["yq"])
        h.move_center(st["node"])
        h.heff_apply(st["node"], st["x"], st["y"])
        return [st["yq"], st["y"]]
    if kind == "eigsolve":
        h.set_tensor(st["node"], st["guess"])
        theta, _ = h.eigsolve(st["node"])
        return [theta, h.get_tensor(st["node"])]
    if kind == "sweep":
        h.init_state(st["raw"])
        energies, _ = h.sweep(1)
        return [energies, _magnetisation(h)]
    return h.correlation(SIGMA_Z, SIGMA_Z)


def work(case):
    """Bytes: the effective operators and tensors that the call reads, and what it writes, once.
    Flops: those of the matvecs (the minimal count that the library reports per node); for a centre
    move those of its two matvecs, the QR and, per stored operator block of a link (counted as the
    mean over links), one contraction and one Gram product."""
    kind = case["kind"]
    if kind == "batch":
        parts = [work(dict(case, kind="sweep", m=m)) for m in _batch_ms(case)]
        return {k: sum(w[k] for w in parts) for k in ("bytes", "flops")}
    dims, flops, env_bytes, tree = _structure(case["L"], case["m"], case["model"])
    size = [int(np.prod(d)) for d in dims]
    if kind in ("matvec", "move", "eigsolve"):
        n = _node(case)
        fmt = 8 if case.get("dtype", "f64") == "f64" else 4
        squares = sum(2 * d[2] ** 2 for d in dims[:-1])
        blocks = env_bytes / 8 / squares   # mean stored blocks per link and direction
        env = lambda q: blocks * sum(d * d for d in dims[q] if d > 2)  # noqa: E731
        if kind == "matvec":
            return {"bytes": fmt * (2 * size[n] + env(n)), "flops": flops[n]}
        if kind == "eigsolve":
            k = min(KRYLOV, size[n])
            return {"bytes": 8 * ((k + 2) * size[n] + env(n)), "flops": k * flops[n]}
        q = tree.parent[n]
        link = dims[n][2]
        move = (size[n] + size[q]) * link * (4 + 4 * blocks)
        return {"bytes": 8 * (4 * (size[n] + size[q]) + env(n) + env(q)), "flops": flops[n] + flops[q] + move}
    if kind == "sweep":
        return {"bytes": env_bytes + 16 * sum(size), "flops": sum(min(KRYLOV, s) * f for s, f in zip(size, flops))}
    # correlation: every site's images on the links above it, and the pairs closed at their common node
    n_sites = case["L"] ** 2
    up = sum((tree.hi[n] - tree.lo[n]) * 4.0 * size[n] * (dims[n][0] + dims[n][1]) for n in range(len(dims)))
    return {"bytes": 8 * (sum(size) + n_sites ** 2), "flops": up}


# ---------------------------------------------------------------------------- 64-bit values
class _Tree:
    """The binary tree over leaf positions 0 .. N - 1, nodes in post-order."""

    def __init__(self, n_sites, m):
        self.child, self.lo, self.hi, self.parent = [], [], [], []

        def build(lo, hi):   # a leaf is -1 - position
            if hi - lo == 1:
                return -1 - lo
            mid = lo + (hi - lo + 1) // 2
            a, b = build(lo, mid), build(mid, hi)
            self.child.append((a, b))
            self.lo.append(lo)
            self.hi.append(hi)
            return len(self.child) - 1

        self.root = build(0, n_sites)
        self.parent = [-1] * len(self.child)
        for n, c in enumerate(self.child):
            for x in c:
                if x >= 0:
                    self.parent[x] = n


def _canonical_q(a):
    q, r = np.linalg.qr(a)
    s = np.where(np.diag(r) < 0, -1.0, 1.0)
    return q * s[None, :], r * s[:, None]


class _Network:
    """The state of a problem and its rotated terms, contracted link by link.

    A term on leaf positions S is a tensor with one index of size 4 (row and column of the site)
    per position.  On a link that has the positions A of S on its far side the term is held as the
    left singular vectors of (A | S without A), each renormalised to a matrix on the link; terms
    with all of S on the far side are summed into one matrix."""

    def __init__(self, p):
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        self.tree = _Tree(p.n_sites, p.m)
        self.pos = {s: i for i, s in enumerate(p.leaf_order)}
        self.gate = {}
        for (a, b), u in zip(p.de_sites, p.de_u):
            self.gate[a] = self.gate[b] = (a, b, np.asarray(u).reshape(2, 2, 2, 2))
        self.terms = [self._rotate(s, o, c, self.pos) for s, o, c in p.terms]
        self.T = []
        for n, raw in enumerate(p.raw_tensors):
            raw = np.asarray(raw, dtype=np.float64)
            if n == self.tree.root:
                t = raw / np.linalg.norm(raw)
            else:
                t = _canonical_q(raw.reshape(-1, raw.shape[2]))[0].reshape(raw.shape)
            self.T.append(torch.from_numpy(t).to(self.dev))
        self.center = self.tree.root
        self.bases, self.links = {}, {}

    def _rotate(self, sites, ops, coef, pos):
        gates = {self.gate[s][:2]: self.gate[s] for s in sites if s in self.gate}
        S = sorted(set(sites) | {x for g in gates for x in g}, key=pos.get)
        k = len(S)
        H = np.array(float(coef))
        for s in S:
            H = np.multiply.outer(H, np.asarray(ops[list(sites).index(s)]) if s in sites else np.eye(2))
        H = H.transpose([2 * i for i in range(k)] + [2 * i + 1 for i in range(k)])
        for a, b, u in gates.values():   # U^T H U on the gate's two sites
            i, j = S.index(a), S.index(b)
            for off in (0, k):
                H = np.moveaxis(np.tensordot(u, H, axes=([0, 1], [i + off, j + off])), (0, 1), (i + off, j + off))
        H = H.transpose([x for i in range(k) for x in (i, k + i)]).reshape((4,) * k)
        return tuple(pos[s] for s in S), H

    def _sides(self, n):
        """Predicate per leg of node n: is a position beyond that leg?"""
        (a, b), lo, hi = self.tree.child[n], self.tree.lo[n], self.tree.hi[n]
        mid = lo + (hi - lo + 1) // 2
        return [lambda s: lo <= s < mid, lambda s: mid <= s < hi, lambda s: not lo <= s < hi]

    def _basis(self, t, A):
        """Orthonormal operators on the positions A of term t that span it, as columns."""
        key = (t, A)
        if key not in self.bases:
            S, H = self.terms[t]
            rows = [i for i, s in enumerate(S) if s in A]
            mat = H.transpose(rows + [i for i in range(len(S)) if i not in rows]).reshape(4 ** len(rows), -1)
            u, s, _ = np.linalg.svd(mat, full_matrices=False)
            self.bases[key] = u[:, s > 1e-13 * s[0]]
        return self.bases[key]

    def _coupling(self, t, parts):
        """The term as a tensor over the bases of disjoint position sets that cover it."""
        S, H = self.terms[t]
        H = H.transpose([S.index(s) for A in parts for s in sorted(A)]).reshape([4 ** len(A) for A in parts])
        for A in parts:   # each contraction moves the new index to the back
            H = np.tensordot(H, self._basis(t, A), axes=([0], [0]))
        return H

    def _into(self, n, leg):
        """What comes into node n over a leg: (summed matrix or None, {term: stack of matrices})."""
        c = self.tree.child[n][leg] if leg < 2 else None
        if leg == 2:
            return self._link(self.tree.parent[n], n) if n != self.tree.root else (None, {})
        return self._leaf(-1 - c) if c < 0 else self._link(c, n)

    def _leaf(self, s):
        key = ("leaf", s)
        if key not in self.links:
            total, stack = np.zeros((2, 2)), {}
            for t, (S, H) in enumerate(self.terms):
                if S == (s,):
                    total = total + H.reshape(2, 2)
                elif s in S:
                    stack[t] = torch.from_numpy(np.ascontiguousarray(self._basis(t, (s,)).T).reshape(-1, 2, 2)).to(self.dev)
            self.links[key] = (torch.from_numpy(total).to(self.dev), stack)
        return self.links[key]

    def _mul(self, op, x, leg):
        """The matrix op on one leg of x."""
        y = torch.tensordot(op, x, dims=([1], [leg]))
        return y if leg == 0 else torch.movedim(y, 0, leg).contiguous()

    def _link(self, n, to):
        """The effective operators that node n sends to its neighbour `to`."""
        if (n, to) in self.links:
            return self.links[(n, to)]
        out = 2 if self.tree.parent[n] == to else self.tree.child[n].index(to)
        la, lb = [x for x in range(3) if x != out]
        (Ea, Sa), (Eb, Sb) = self._into(n, la), self._into(n, lb)
        T, sides = self.T[n], self._sides(n)
        flat = T.movedim(out, 2).reshape(-1, T.shape[out])
        close = lambda z: flat.T @ z.movedim(out, 2).reshape(-1, T.shape[out])  # noqa: E731
        Z = torch.zeros_like(T)
        for E, leg in ((Ea, la), (Eb, lb)):
            if E is not None:
                Z = Z + self._mul(E, T, leg)
        stack = {}
        for t in sorted(set(Sa) | set(Sb)):
            S, H = self.terms[t]
            A, B = (tuple(s for s in S if sides[leg](s)) for leg in (la, lb))
            rest = tuple(s for s in S if s not in A and s not in B)
            G = self._coupling(t, [X for X in (A, B, rest) if X])   # axes in that order
            G = G.reshape([len(St[t]) if t in St else 1 for St in (Sa, Sb)] + [-1])
            if rest:
                # couple the far basis away: operators orthonormal on A u B
                u = self._basis(t, tuple(sorted(A + B)))
                order = [sorted(A + B).index(s) for s in A + B]
                u = u.reshape([4] * len(order) + [-1]).transpose(order + [len(order)])
                u = u.reshape(4 ** len(A), 4 ** len(B), -1)
                fa = self._basis(t, A) if A else np.ones((1, 1))
                fb = self._basis(t, B) if B else np.ones((1, 1))
                G = np.einsum("ix,jy,ijk->xyk", fa, fb, u)
            G = torch.from_numpy(np.ascontiguousarray(G)).to(self.dev)
            wa = [self._mul(o, T, la) for o in Sa[t]] if t in Sa else [T]
            blocks = []
            for k in range(G.shape[2]):
                z = torch.zeros_like(T)
                for x, w in enumerate(wa):
                    if t in Sb:
                        z += self._mul(torch.tensordot(G[x, :, k], Sb[t], dims=1), w, lb)
                    else:
                        z += G[x, 0, k] * w
                blocks.append(z)
            if rest:
                stack[t] = torch.stack([close(z) for z in blocks])
            else:
                Z = Z + blocks[0]
        self.links[(n, to)] = (close(Z), stack)
        return self.links[(n, to)]

    def heff(self, n):
        """x -> H_eff(n) x, the operators of every term stacked per set of legs."""
        ins, sides = [self._into(n, leg) for leg in range(3)], self._sides(n)
        items = {}   # legs -> lists of matrices
        for leg, (E, _) in enumerate(ins):
            if E is not None:
                items.setdefault((leg,), [[]])[0].append(E[None])
        for t, (S, H) in enumerate(self.terms):
            parts = [(leg, tuple(s for s in S if sides[leg](s))) for leg in range(3)]
            parts = [(leg, A) for leg, A in parts if A]
            if len(parts) < 2:
                continue
            G = torch.from_numpy(np.ascontiguousarray(self._coupling(t, [A for _, A in parts]))).to(self.dev)
            ops = [ins[leg][1][t] for leg, _ in parts]
            last = torch.tensordot(G, ops[-1], dims=1)   # the last leg's operators, coupled
            last = last.reshape((-1,) + last.shape[-2:])
            if len(parts) == 2:
                put = [ops[0], last]
            else:
                ra, rb = len(ops[0]), len(ops[1])
                put = [ops[0].repeat_interleave(rb, 0), ops[1].repeat(ra, 1, 1), last]
            keep = last.abs().amax(dim=(1, 2)) > 0
            for lst, o in zip(items.setdefault(tuple(leg for leg, _ in parts), [[] for _ in put]), put):
                lst.append(o[keep])
        items = {legs: [torch.cat(o) for o in lst] for legs, lst in items.items()}

        def apply(x):
            y = torch.zeros_like(x)
            step = max(1, (1 << 28) // x.numel())
            for legs, ops in items.items():
                for r in range(0, len(ops[0]), step):
                    z = None
                    for leg, o in zip(legs, ops):
                        o = o[r:r + step]
                        v = (x.unsqueeze(0) if z is None else z).movedim(leg + 1, 1)
                        w = torch.matmul(o, v.reshape(v.shape[0], v.shape[1], -1))
                        z = w.reshape((len(o), o.shape[1]) + v.shape[2:]).movedim(1, leg + 1)
                    y += z.sum(0)
            return y
        return apply

    def move(self, target):
        """The centre to `target`, link by link (QR with a non-negative diagonal of R)."""
        def path_up(n):
            out = [n]
            while self.tree.parent[out[-1]] >= 0:
                out.append(self.tree.parent[out[-1]])
            return out
        a, b = path_up(self.center), path_up(target)
        while len(a) > 1 and len(b) > 1 and a[-2] == b[-2]:
            a.pop()
            b.pop()
        path = a + b[::-1][1:]
        for n, q in zip(path, path[1:]):
            out = 2 if self.tree.parent[n] == q else self.tree.child[n].index(q)
            leg = 2 if self.tree.parent[q] == n else self.tree.child[q].index(n)
            t = self.T[n].movedim(out, 2)
            Q, R = _canonical_q(t.reshape(-1, t.shape[2]).cpu().numpy())
            self.T[n] = torch.from_numpy(Q).to(self.dev).reshape(t.shape).movedim(2, out).contiguous()
            self.set(q, self._mul(torch.from_numpy(R).to(self.dev), self.T[q], leg))
            self.stale(n)
        self.center = target

    def stale(self, n):
        """Drop what depends on the tensor of node n."""
        lo, hi = self.tree.lo[n], self.tree.hi[n]
        for key in [k for k in self.links if k[0] != "leaf"]:
            src, to = key
            up = self.tree.parent[src] == to
            e = src if up else to   # the node below the link
            below = self.tree.lo[e] <= lo and hi <= self.tree.hi[e]
            if below == up:
                del self.links[key]

    def set(self, n, t):
        self.T[n] = t
        self.stale(n)

    def solve(self, n):
        """KRYLOV Lanczos steps from T_n (two Gram-Schmidt passes); T_n <- Ritz vector."""
        H = self.heff(n)
        shape, T = self.T[n].shape, self.T[n].reshape(-1)
        V, al, be = [T / T.norm()], [], []
        for j in range(min(KRYLOV, T.numel())):
            w = H(V[j].reshape(shape)).reshape(-1)
            al.append(float(V[j] @ w))
            if j + 1 == min(KRYLOV, T.numel()):
                break
            B = torch.stack(V)
            for _ in range(2):
                w = w - B.T @ (B @ w)
            b = float(w.norm())
            if b <= 1e-14 * max(abs(a) for a in al):
                break
            be.append(b)
            V.append(w / b)
        k = len(al)
        ev, y = np.linalg.eigh(np.diag(al) + np.diag(be[:k - 1], 1) + np.diag(be[:k - 1], -1))
        y = y[:, 0]
        y = y * np.sign(y[np.argmax(np.abs(y) >= 1e-8 * np.abs(y).max())])
        r = torch.stack(V).T @ torch.from_numpy(y).to(self.dev)
        self.set(n, (r / r.norm()).reshape(shape))
        return float(ev[0])

    def expect(self, term):
        """The expectation value of one product of one-site operators, the centre at the root."""
        other = copy.copy(self)
        other.terms, other.bases, other.links = [self._rotate(*term, self.pos)], {}, {}
        T = self.T[self.tree.root]
        return float((T * other.heff(self.tree.root)(T)).sum())

    def sweep(self):
        e = 0.0
        for n in range(len(self.T)):
            self.move(n)
            e = self.solve(n)
        return e


def exact(case, seed):
    kind = case["kind"]
    if kind == "correlation":
        return _exact_correlation(case, seed) if case["L"] <= 4 else None
    if kind in ("sweep", "batch"):
        ms = _batch_ms(case) if kind == "batch" else [case["m"]]
        if case["L"] ** 2 * sum(ms) * (1 if case["model"] == "ising" else 3) > 8 * 8 * 128:
            return None   # over 20 seconds
        nets = [_Network(_problem(case, seed, m, k)) for k, m in enumerate(ms)]
        energies = [[net.sweep()] for net in nets]
        mags = [np.array([net.expect(((i,), (SIGMA_X,), 1.0)) for i in range(case["L"] ** 2)]) for net in nets]
        return [np.array(energies if kind == "batch" else energies[0])] + mags
    net = _Network(_problem(case, seed))
    n = _node(case)
    net.move(n)
    if kind == "eigsolve":
        theta = net.solve(n)
        return [theta, net.T[n].cpu().numpy()]
    if kind == "matvec":
        x = _gauss(tuple(net.T[n].shape), seed + 1, torch.float64 if case["dtype"] == "f64" else torch.float32)
        return net.heff(n)(x.double())
    q = net.tree.parent[n]
    leg = net.tree.child[q].index(n)
    tn, tq = _schmidt_gauge(net.T[n].cpu().numpy(), net.T[q].cpu().numpy(), leg)
    net.set(n, torch.from_numpy(tn).to(net.dev))
    net.set(q, torch.from_numpy(tq).to(net.dev))
    x, xq = _gauss(tuple(net.T[n].shape), seed + 1, torch.float64), _gauss(tuple(net.T[q].shape), seed + 2, torch.float64)
    y = net.heff(n)(x)
    net.move(q)
    return [net.heff(q)(xq), y]


def _exact_correlation(case, seed):
    net, n = _Network(_problem(case, seed)), case["L"] ** 2
    C = np.eye(n)   # sigma_z squared on the diagonal
    for i in range(n):
        for j in range(i):
            C[i, j] = C[j, i] = net.expect(((i, j), (SIGMA_Z, SIGMA_Z), 1.0))
    return C
