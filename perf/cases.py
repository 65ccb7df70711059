"""The workloads that stand for this framework's use, each through its public entry points.

A case says what is evaluated (`op`), on how many charges and elements, and with which options of the
context; `prepare` draws the charges and makes the context that a program keeps from step to step, `run`
is one evaluation, and `exact` gives the same outputs from a plain torch evaluation of the method in 64 bits
(dense one-dimensional eigenbases for the mesh problem, table sums for the near field, explicit pair lists)
that shares no code with the package.
"""
import math
import random

import numpy as np
import torch

import paper_1503_08509_amd as fp

#: Defaults of a case: one periodic configuration, the one-element q = 3 screen, the default options.
BASE = {"q": 3, "support": "one", "kind": "uniform", "charges": "pm1", "L": 1.0, "nconf": 1, "nmin": 0,
        "mixed": False, "graph": False, "fdm": False, "box": False}


def _case(name, op, N, n, **more):
    c = dict(BASE, op=op, N=N, n=n, **more)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest step of a program that moves charges: a thousand of them, where launches and latency count
        _case("forces-1k-n8", "forces", 1000, 8),
        # the same use in a long run: a captured evaluation replayed at every step
        _case("replay-4k-n16", "forces", 4096, 16, graph=True, L=10.0),
        # energies alone (Monte Carlo moves, tests of a configuration) on a mesh whose edge is no power of two
        _case("energy-30k-n20", "energy", 30011, 20, charges="uniform"),
        # autograd: forward, then the hand-written backward with a solve of its own, on an odd mesh
        _case("autograd-60k-n27", "autograd", 60000, 27, charges="uniform"),
        # an ordinary step
        _case("forces-100k-n32", "forces", 100000, 32, charges="uniform"),
        # the benchmark's step
        _case("forces-1M-n64", "forces", 1000000, 64),
        # the same number of charges in clusters: skewed occupancy, up to hundreds of charges in an element
        _case("clustered-1M-n64", "forces", 1000000, 64, kind="clustered"),
        # mixed precision at the benchmark's size
        _case("mixed-1M-n64", "forces", 1000000, 64, mixed=True),
        # many small independent configurations of uneven size in one call
        _case("batch-32-n16", "forces", 32000, 16, nconf=32, nmin=2000, charges="uniform"),
        # the exact mesh solver at the benchmark's size
        _case("exact-1M-n64", "forces", 1000000, 64, fdm=True),
        # charges in a grounded box
        _case("grounded-100k-n32", "forces", 100000, 32, box=True, fdm=True),
        # the 27-element screens of degree 2, for more accuracy
        _case("screen27-q2-60k-n24", "forces", 60000, 24, q=2, support="27"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _coarsens(n):
    """Whether the multigrid hierarchy takes a mesh of n elements per axis (factors 2 and 3 down to 16)."""
    while n > 4 and n % 2 == 0:
        n //= 2
    while n > 6 and n % 3 == 0:
        n //= 3
    return n <= 16


def draw(rng):
    """Another evaluation of the same kinds: mesh edges from the smallest the near block allows to the largest
    power of two with a near field by FFTs, odd ones among them, a third of a charge to six per element."""
    what = rng.choice(["forces", "forces", "energy", "autograd", "clustered", "mixed", "replay", "batch", "exact",
                       "box", "screen"])
    n = rng.choice([8, 16, 32, 64]) if rng.random() < 0.4 else _log(rng, 7, 56)
    more, op = {}, "forces"
    if what in ("energy", "autograd"):
        op = what
        n = min(n, 48)
    elif what == "clustered":
        more["kind"] = "clustered"
        n = max(n, 12)
    elif what == "mixed":
        more["mixed"] = True
    elif what == "replay":
        more["graph"] = True
        n = min(n, 32)
    elif what == "batch":
        n = min(n, 20)
        more["nconf"] = rng.randint(2, 40)
    elif what == "exact":
        more["fdm"] = True
        n = n if n & (n - 1) == 0 else min(n, 40)
    elif what == "box":
        more.update(box=True, fdm=True)
        n = min(n, 32)
    elif what == "screen":
        more["q"], more["support"] = rng.choice([(2, "one"), (4, "one"), (1, "27"), (2, "27"), (3, "27")])
        n = min(n, 24)
    while not _coarsens(n):
        n -= 1
    N = max(16, min(400000 if what == "clustered" else 1000000, int(n ** 3 * math.exp(rng.uniform(math.log(0.33), math.log(6.0))))))
    if what == "batch":
        more["nmin"] = max(8, N // 16)
    more["charges"] = rng.choice(["pm1", "uniform"])
    if more["charges"] == "pm1":
        N -= N % 2
    return _case(None, op, N, n, L=rng.choice([1.0, 1.0, 10.0, 37.5]), **more)


def _counts(case):
    """Charges of each configuration: log-uniform between nmin and N, the same for every seed."""
    if case["nconf"] == 1:
        return [case["N"]]
    r = random.Random(case["nconf"] * 1000003 + case["N"])
    return [2 * (_log(r, case["nmin"], case["N"]) // 2) for _ in range(case["nconf"])]


def _inputs(case, seed):
    """Positions [N, 3] and charges [N] of all configurations, neutral in each."""
    g = torch.Generator("cuda").manual_seed(seed)
    kw = {"device": "cuda", "dtype": torch.float64, "generator": g}
    L, xs, Qs = case["L"], [], []
    for N in _counts(case):
        x = torch.rand(N, 3, **kw)
        if case["kind"] == "clustered":   # 64 Gaussian clusters over a tenth of uniform background
            at = torch.rand(64, 3, **kw)[torch.randint(64, (N,), device="cuda", generator=g)]
            y = at + 0.02 * torch.randn(N, 3, **kw)
            x = torch.where(torch.rand(N, 1, **kw) < 0.1, x, y - torch.floor(y))
        if case["box"]:                   # charges keep half an element from the faces
            m = 0.5 / case["n"]
            x = m + (1.0 - 2.0 * m) * x
        if case["charges"] == "pm1":
            Q = 1.0 - 2.0 * (torch.randperm(N, device="cuda", generator=g) % 2).to(torch.float64)
        else:
            Q = 2.0 * torch.rand(N, **kw) - 1.0
            Q = Q - Q.mean()
        xs.append(x * L)
        Qs.append(Q)
    return torch.cat(xs), torch.cat(Qs)


def prepare(case, seed):
    x, Q = _inputs(case, seed)
    opts = {}
    if case["support"] == "27":
        opts["support"] = fp.SUPPORT_27
    if case["mixed"]:
        opts["precision"] = fp.PRECISION_MIXED
    if case["graph"]:
        opts["use_graph"] = 1
    if case["fdm"]:
        opts["solver"] = fp.SOLVER_FDM
    if case["box"]:
        opts["boundary"] = fp.BOUNDARY_GROUNDED
    counts = _counts(case)
    ctx = fp.Context(case["L"], counts if case["nconf"] > 1 else counts[0], case["n"], q=case["q"], **opts)
    if case["op"] == "autograd":
        x.requires_grad_()
        Q.requires_grad_()
    return {"op": case["op"], "ctx": ctx, "x": x, "Q": Q}


def run(state):
    ctx, x, Q = state["ctx"], state["x"], state["Q"]
    if state["op"] == "energy":
        Phi, U = ctx.energy(x, Q)
        return {"Phi": Phi, "U": U}
    if state["op"] == "forces":
        return ctx.energy_forces(x, Q, dUdQ=True, Phi=True)
    U = fp.FEP3MEnergy.apply(x, Q, ctx)
    gx, gQ = torch.autograd.grad(U, (x, Q))
    return {"U": U.detach(), "gx": gx, "gQ": gQ}


def _order(case):
    return case["q"] + 2, case["q"] + 1 if case["support"] == "27" else case["q"] - 1


def work(case):
    """Inputs read and results written once, the mesh load(s) and potential(s) once each; 20 operations per near
    pair (11 without forces), two per screen moment and node for the transforms between elements and mesh, and
    the mesh operator applied once per system (seven banded products of p + 1 to 2 p + 2 terms per node)."""
    counts, n = _counts(case), case["n"]
    N, (p, nl) = sum(counts), _order(case)
    forces = case["op"] != "energy"
    dof = len(counts) * (p * n) ** 3 * (2 if forces else 1)
    pairs = sum(c * c for c in counts) * 343.0 / n ** 3
    if case["kind"] == "clustered":
        # clusters of standard deviation s: an element block of side 7/n holds about (erf(3.5 / (2 n s)))^3 of its own
        # cluster's charges, 0.9 N / 64 of them
        pairs = N * (0.1 * N * 343.0 / n ** 3 + 0.81 * N / 64 * math.erf(3.5 / (2.0 * n * 0.02)) ** 3)
    return {"bytes": 32.0 * N + 8.0 * N * (6 if forces else 1) + 16.0 * dof,
            "flops": pairs * (20 if forces else 11) + dof * (14.0 * (p + 2) + 2.0 * nl ** 3)}


# ----------------------------------------------------------------- 64-bit values

def _gauss(m):
    t, w = np.polynomial.legendre.leggauss(m)
    return 0.5 * t, 0.5 * w


def _gll(p):
    c = np.zeros(p + 1)
    c[p] = 1.0
    inner = np.polynomial.legendre.legroots(np.polynomial.legendre.legder(c))
    return 0.5 * np.concatenate([[-1.0], np.sort(inner.real), [1.0]])


def _lagrange(nodes, x):
    """Values [..., len(nodes)] of the Lagrange basis at the points x (numpy or torch)."""
    cols = []
    for k, a in enumerate(nodes):
        v = 1.0 + 0.0 * x
        for j, b in enumerate(nodes):
            if j != k:
                v = v * ((x - float(b)) / float(a - b))
        cols.append(v)
    return np.stack(cols, -1) if isinstance(x, np.ndarray) else torch.stack(cols, -1)


def _element_matrices(p):
    nodes, (x, w) = _gll(p), _gauss(p + 1)
    V = np.polynomial.polynomial.polyvander
    coef = np.linalg.inv(V(nodes, p))                                # column k: monomials of basis k
    D = V(x, p - 1) @ (coef[1:] * np.arange(1, p + 1)[:, None])
    B = _lagrange(nodes, x)
    return (D * w[:, None]).T @ D, (B * w[:, None]).T @ B


def _assembled(p, n, periodic):
    P = p * n if periodic else p * n + 1
    ke, me = _element_matrices(p)
    K, M = np.zeros((P, P)), np.zeros((P, P))
    for e in range(n):
        i = (p * e + np.arange(p + 1)) % P if periodic else p * e + np.arange(p + 1)
        K[np.ix_(i, i)] += ke
        M[np.ix_(i, i)] += me
    return K, M


def _pencil(K, M):
    """lam, V with K V = M V diag(lam), V^T M V = 1."""
    R = np.linalg.inv(np.linalg.cholesky(M))
    lam, W = np.linalg.eigh(R @ K @ R.T)
    return lam, R.T @ W


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _axes(A, X):
    """The matrix A applied along each of the three axes of X."""
    for _ in range(3):
        s = X.shape
        X = torch.movedim((A @ X.reshape(s[0], -1)).reshape(A.shape[0], s[1], s[2]), 0, 2)
    return X


def _axis3(A, B, C, X):
    """A along z, B along y, C along x of X[z, y, x]."""
    for T in (A, B, C):
        s = X.shape
        X = torch.movedim((T @ X.reshape(s[0], -1)).reshape(T.shape[0], s[1], s[2]), 0, 2)
    return X


def _stiffness(K, M, X):
    return _axis3(K, M, M, X) + _axis3(M, K, M, X) + _axis3(M, M, K, X)


def _solve(lam, V, drop, b):
    y = _axes(V.T.contiguous(), b)
    D = lam[:, None, None] + lam[None, :, None] + lam[None, None, :]
    if drop:
        D = D.clone()
        D[0, 0, 0] = math.inf
    return _axes(V, y / D)


def _duals(q, support, x):
    """The functions r_l with int x^m r_l = [m == l], l = 0 .. d, at the points x: [len(x), d + 1]."""
    nodes, span = np.linspace(-0.5, 0.5, q + 1), 3 if support == "27" else 1

    def basis(t):
        inside = np.abs(t) <= 0.5
        B = _lagrange(nodes, t) * inside[:, None]
        if support == "one":
            return B[:, 1:q]
        B[:, 0] += np.where((t < -0.5) & (t >= -1.5), _lagrange(nodes, t + 1.0)[:, q], 0.0)
        B[:, q] += np.where((t > 0.5) & (t <= 1.5), _lagrange(nodes, t - 1.0)[:, 0], 0.0)
        return B

    t, w = _gauss(q + 3)
    t = np.concatenate([t + e - (span - 1) // 2 for e in range(span)])
    B, w = basis(t), np.tile(w, span)
    mom = np.stack([(w * t ** m) @ B for m in range(B.shape[1])])
    return basis(x) @ np.linalg.inv(mom)


def _load_weights(p, q, support):
    span, (t, w) = 3 if support == "27" else 1, _gauss(p + 1)
    B = _lagrange(_gll(p), t)
    d1 = _duals(q, support, t).shape[1]
    g = np.zeros((d1, span * p + 1))
    for e in range(span):
        g[:, e * p:e * p + p + 1] += (_duals(q, support, t + e - (span - 1) // 2) * w[:, None]).T @ B
    return g


def _tables(q, support, nsr=3, box=15):
    """T[dz, dy, dx, a, node]: order-p Dirichlet solutions for each screen moment on box^3 elements, with the
    free-space potential of the moment's density on the outer faces."""
    p, span = q + 2, 3 if support == "27" else 1
    c, (t, w) = (box - 1) // 2, _gauss(16)
    t = np.concatenate([t + e - (span - 1) // 2 for e in range(span)])
    R = _duals(q, support, t) * np.tile(w, span)[:, None]
    d1, P = R.shape[1], box * p + 1
    gll = _gll(p)
    xs = np.concatenate([(np.arange(box)[:, None] - c + gll[None, :p]).ravel(), [box - c - 0.5]])
    t, R, xs = _dev(t), _dev(R), _dev(xs)
    g = _dev(_load_weights(p, q, support))
    K, M = _assembled(p, box, False)
    lam, V = _pencil(K[1:-1, 1:-1], M[1:-1, 1:-1])
    K, M, lam, V = _dev(K), _dev(M), _dev(lam), _dev(V)
    dens = torch.einsum("ka,jb,ic->kjiabc", R, R, R).reshape(-1, d1 ** 3)          # quadrature point, moment
    src = torch.stack(torch.meshgrid(t, t, t, indexing="ij"), -1).reshape(-1, 3)
    grid = torch.stack(torch.meshgrid(xs, xs, xs, indexing="ij"), -1)
    on = torch.ones(P, P, P, dtype=torch.bool, device="cuda")
    on[1:-1, 1:-1, 1:-1] = False
    at = grid[on]
    step = max(1, (1 << 27) // src.shape[0])
    pot = []
    for i in range(0, at.shape[0], step):
        r2 = sum((at[i:i + step, k, None] - src[None, :, k]) ** 2 for k in range(3))
        pot.append(torch.rsqrt(r2) @ dens)
    pot = torch.cat(pot)
    S, out = 2 * nsr + 1, []
    k0 = p * (c - (span - 1) // 2)
    for a in range(d1 ** 3):
        az, ay, ax = a // (d1 * d1), a // d1 % d1, a % d1
        b = torch.zeros(P, P, P, dtype=torch.float64, device="cuda")
        s = slice(k0, k0 + span * p + 1)
        b[s, s, s] = 4.0 * math.pi * g[az][:, None, None] * g[ay][None, :, None] * g[ax][None, None, :]
        full = torch.zeros_like(b)
        full[on] = pot[:, a]
        r = (b - _stiffness(K, M, full))[1:-1, 1:-1, 1:-1]
        full[1:-1, 1:-1, 1:-1] = _solve(lam, V, False, r)
        idx = (p * (c - nsr + torch.arange(S, device="cuda"))[:, None] + torch.arange(p + 1, device="cuda")).reshape(-1)
        blk = full[idx][:, idx][:, :, idx].reshape(S, p + 1, S, p + 1, S, p + 1)
        out.append(blk.permute(0, 2, 4, 1, 3, 5).reshape(S, S, S, -1))
    return torch.stack(out, 3)


class _Bins:
    """Charges sorted by element: coordinates, offsets (with their gradient in x), element starts."""

    def __init__(self, x, Q, L, n, periodic):
        s = x / L
        s = s - torch.floor(s).detach() if periodic else s
        t = s * n
        e = torch.clamp(torch.floor(t.detach()), max=n - 1)
        self.n, self.periodic = n, periodic
        self.u, self.e, self.Q = t - e - 0.5, e.long(), Q
        self.lin = self.linear(self.e)
        self.order = torch.argsort(self.lin, stable=True)
        self.count = torch.bincount(self.lin, minlength=n ** 3)
        self.start = torch.cumsum(self.count, 0) - self.count

    def linear(self, e):
        return e[:, 0] + self.n * (e[:, 1] + self.n * e[:, 2])

    def near(self, te, most, nsr=3):
        """(targets, lengths, sources, offset D) in pieces of about `most` pairs: the charges of the element at D
        from each target's element te, as indices into the sorted charges, grouped by target."""
        for dz in range(-nsr, nsr + 1):
            for dy in range(-nsr, nsr + 1):
                for dx in range(-nsr, nsr + 1):
                    D = torch.tensor([dx, dy, dz], device=te.device)
                    s = te + D
                    if self.periodic:
                        c = self.count[self.linear(s % self.n)]
                        s = s % self.n
                    else:
                        ok = ((s >= 0) & (s < self.n)).all(1)
                        s = torch.where(ok[:, None], s, torch.zeros_like(s))
                        c = torch.where(ok, self.count[self.linear(s)], 0)
                    first, total = self.start[self.linear(s)], torch.cumsum(c, 0)
                    marks = torch.arange(0, int(total[-1]), most, device=te.device)
                    cuts = torch.unique(torch.searchsorted(total, marks)).tolist() + [len(c)]
                    for a, b in zip(cuts[:-1], cuts[1:]):
                        k = c[a:b]
                        m = int(k.sum())
                        if m == 0:
                            continue
                        i = torch.repeat_interleave(torch.arange(b - a, device=te.device), k, output_size=m)
                        j = torch.arange(m, device=te.device) - (torch.cumsum(k, 0) - k)[i] + first[a:b][i]
                        yield slice(a, b), i, k, j, D


def _pairs(b):
    """Near sums of the sorted charges: potential [N] and its gradient's sum_j Q_j d / r^3 [N, 3]."""
    u, Q, e = b.u.detach()[b.order], b.Q.detach()[b.order], b.e[b.order]
    pot, grad = torch.zeros_like(Q), torch.zeros_like(u)
    for t, i, k, j, D in b.near(e, 24_000_000):
        d = D + (u[j] - u[t][i])
        r = (d * d).sum(1).sqrt()
        if not D.any():
            r = torch.where(j == i + t.start, math.inf, r)
        w = Q[j] / r
        v = torch.cat([w[:, None], d * (w / (r * r))[:, None]], 1)
        v = torch.segment_reduce(v, "sum", lengths=k, axis=0, unsafe=True)
        pot[t] += v[:, 0]
        grad[t] += v[:, 1:]
    return pot, grad


def _near_screens(C, T, n, periodic):
    """Psi[z, y, x, node] = sum_D T[D] C[E - D] for C[z, y, x, moment]."""
    S, M = T.shape[0], T.shape[4]
    r = S // 2
    if periodic:
        i = torch.arange(-r, n + r, device=C.device) % n
        Cp = C[i][:, i][:, :, i]
    else:
        Cp = torch.nn.functional.pad(C, (0, 0, r, r, r, r, r, r))
    out = torch.zeros(n ** 3, M, dtype=torch.float64, device=C.device)
    for dz in range(S):
        for dy in range(S):
            for dx in range(S):
                s = Cp[S - 1 - dz:S - 1 - dz + n, S - 1 - dy:S - 1 - dy + n, S - 1 - dx:S - 1 - dx + n]
                out = out + s.reshape(n ** 3, -1) @ T[dz, dy, dx]
    return out


def _configuration(case, x, Q):
    """U, Phi, dU/dx and dU/dQ of one configuration."""
    L, n, q, support, periodic = case["L"], case["n"], case["q"], case["support"], not case["box"]
    (p, d1), span, h = _order(case), 3 if support == "27" else 1, L / n
    x, Q = x.detach().clone().requires_grad_(), Q.detach().clone().requires_grad_()
    b = _Bins(x, Q, L, n, periodic)
    pw = [torch.stack([b.u[:, k] ** l for l in range(d1)], -1) for k in range(3)]
    mono = (pw[2][:, :, None, None] * pw[1][:, None, :, None] * pw[0][:, None, None, :]).reshape(len(Q), -1)
    C = torch.zeros(n ** 3, d1 ** 3, dtype=torch.float64, device="cuda").index_add(0, b.lin, mono * Q[:, None])
    C = C.reshape(n, n, n, -1)
    # load: the moments spread along each axis by the weights of their support's nodes
    P = p * n if periodic else p * n + 1
    g, E = _load_weights(p, q, support), np.zeros((d1, P, n))
    for e in range(n):
        k = p * (e - (span - 1) // 2) + np.arange(span * p + 1)
        for l in range(d1):
            np.add.at(E[l, :, e], k % P if periodic else k, g[l])
    E = _dev(E)
    load = 0.0
    for a in range(d1 ** 3):
        load = load + _axis3(E[a // (d1 * d1)], E[a // d1 % d1], E[a % d1], C[..., a])
    load = 4.0 * math.pi * load
    T = _tables(q, support)
    Psi = _near_screens(C, T, n, periodic)
    K, M = _assembled(p, n, periodic)
    node = torch.arange(n, device="cuda")[:, None] * p + torch.arange(p + 1, device="cuda")
    if periodic:
        lam, V = _pencil(K, M)
        lam, V = _dev(lam), _dev(V)
        w1 = _dev(M.sum(1))
        load = load - load.sum() / n ** 3 * w1[:, None, None] * w1[None, :, None] * w1[None, None, :]
        phi = _solve(lam, V, True, load)
        node = node % P
    else:
        # boundary nodes take minus the near sums of their element: pairs, less the screens' potential there
        lam, V = _pencil(K[1:-1, 1:-1], M[1:-1, 1:-1])
        lam, V, K, M = _dev(lam), _dev(V), _dev(K), _dev(M)
        on = torch.ones(P, P, P, dtype=torch.bool, device="cuda")
        on[1:-1, 1:-1, 1:-1] = False
        z = torch.nonzero(on)[:, [2, 1, 0]]
        e = torch.clamp(z // p, max=n - 1)
        k = z - p * e
        xi = _dev(_gll(p))[k]
        us, Qs = b.u.index_select(0, b.order), Q.index_select(0, b.order)
        near = torch.zeros(len(z), dtype=torch.float64, device="cuda")
        for t, i, _, j, D in b.near(e, 24_000_000):
            d = D + us.index_select(0, j) - xi[t][i]
            near = near.index_add(0, i + t.start, Qs.index_select(0, j) / (d * d).sum(1).sqrt())
        near = near - Psi[b.linear(e), k[:, 0] + (p + 1) * (k[:, 1] + (p + 1) * k[:, 2])]
        edge = torch.zeros(P, P, P, dtype=torch.float64, device="cuda").masked_scatter(on, -near)
        inner = (load - _stiffness(K, M, edge))[1:-1, 1:-1, 1:-1]
        phi = edge + torch.nn.functional.pad(_solve(lam, V, False, inner), (1, 1, 1, 1, 1, 1))
    i = node.reshape(-1)
    phiE = phi[i][:, i][:, :, i].reshape(n, p + 1, n, p + 1, n, p + 1).permute(0, 2, 4, 1, 3, 5).reshape(n ** 3, -1)
    W = (phiE - Psi).index_select(0, b.lin).reshape(-1, p + 1, p + 1, p + 1)
    for k in range(3):
        B = _lagrange(_gll(p), b.u[:, k])
        W = (W * B.reshape(B.shape[0], *([1] * (2 - k)), p + 1)).sum(-1)
    Um = 0.5 * (Q * W).sum() / h
    gx, gQ = torch.autograd.grad(Um, (x, Q))
    pot, grad = _pairs(b)
    near, slope = torch.empty_like(pot), torch.empty_like(grad)
    near[b.order], slope[b.order] = pot, grad
    Q, Phi = Q.detach(), (near + W.detach()) / h
    return 0.5 * (Q * Phi).sum(), Phi, gx + Q[:, None] * slope / (h * h), gQ + near / h


def exact(case, seed):
    x, Q = _inputs(case, seed)
    at, got = 0, []
    for N in _counts(case):
        got.append(_configuration(case, x[at:at + N], Q[at:at + N]))
        at += N
    U = torch.stack([v[0] for v in got]) if case["nconf"] > 1 else got[0][0]
    Phi, gx, gQ = (torch.cat([v[k] for v in got]) for k in (1, 2, 3))
    if case["op"] == "energy":
        return {"Phi": Phi, "U": U}
    if case["op"] == "forces":
        return {"U": U, "F": -gx, "dUdQ": gQ, "Phi": Phi}
    return {"U": U, "gx": gx, "gQ": gQ}
