"""Workloads of the library's public calls, with their inputs, one pass of each,
its indispensable work and the same result computed in plain torch FP64.

A case is a dict of plain values; "do" names the call, the rest its sizes and
options.  The geometry is (0,L)^p x (0,1)^q with h = 1/ne and `delta` overlap
layers; the potential is drawn from the seed (four Fourier terms with an
envelope for p = 1, fifteen plane waves for p = 2, as in the workloads).
"""
import itertools
import math

import numpy as np
import torch

import paper_2311_08757_amd as dd
from paper_2311_08757_amd import autograd as ag


def listed():
    return [
        # one operator apply on a small problem (the 2-D L = 8, h = 1/32 workload): launch latency
        dict(name="op-2d-small", do="op", which="A", p=1, q=1, L=8, ne=32, delta=2),
        # operator apply at the longest domain and finest mesh of the paper's parameter study (§4.1)
        dict(name="op-2d-ne30", do="op", which="A", p=1, q=1, L=1024, ne=30, delta=3),
        # operator apply at HBM scale: 62,979,135 unknowns in 3-D
        dict(name="op-3d-63M", do="op", which="A", p=1, q=2, L=2048, ne=32, delta=2),
        # the default (FP64) two-level additive Schwarz preconditioner on the 2-D L = 256, h = 1/64
        # workload: one application per CG step
        dict(name="as2-2d-fp64", do="schwarz", kind="as2", pu="equal", prec="fp64", p=1, q=1, L=256,
             ne=64, delta=4),
        # restricted Schwarz with the distance partition of unity on the paper's 1/30 mesh, an odd
        # number of cells, hi/lo bf16 local solves: what a GMRES step applies
        dict(name="ras2-2d-bf16x3", do="schwarz", kind="ras2", pu="distance", prec="bf16x3", p=1, q=1,
             L=101, ne=30, delta=3),
        # two expanding axes, many clipped subdomains (the 3-D L = 16, h = 1/16 workload)
        dict(name="as2-3d-p2-bf16", do="schwarz", kind="as2", pu="equal", prec="bf16", p=2, q=1, L=16,
             ne=16, delta=1),
        # one shifted solve by GMRES with the restricted preconditioner, default precision
        dict(name="gmres-2d-fp64", do="solve", solver="gmres", prec="fp64", rtol=1e-8, p=1, q=1, L=64,
             ne=64, delta=4),
        # a differentiable shifted solve: set-up, forward CG, adjoint CG and the parameter gradient
        dict(name="solve-grad-2d-fp64", do="grad", prec="fp64", p=1, q=1, L=32, ne=32, delta=2),
        # set-up for a new potential (tables, cell problem, dense local inverse, coarse matrix) with
        # one application of the preconditioner it gives
        dict(name="setup-2d-bf16", do="setup", prec="bf16", p=1, q=1, L=256, ne=64, delta=4),
        # the smallest eigenpair, 2-D L = 256, h = 1/64, 1,032,129 unknowns (the benchmark's step)
        dict(name="eig-2d-bf16", do="eig", prec="bf16", p=1, q=1, L=256, ne=64, delta=4),
        # the smallest eigenpair in 3-D with FP32 chain local solves (the h = 1/32 workload, L = 16)
        dict(name="eig-3d-fp32", do="eig", prec="fp32", p=1, q=2, L=16, ne=32, delta=2),
        # a batch of independent 2-D eigenproblems of mixed lengths (16..256), h = 1/32
        dict(name="batch-32", do="batch", prec="bf16", p=1, q=1, n=32, lmin=16, lmax=256, ne=32, delta=2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    do = rng.choice(["op", "op", "schwarz", "schwarz", "solve", "grad", "setup", "eig", "eig", "batch"])
    ne = rng.choice([10, 12, 15, 16, 20, 24, 30, 32, 40, 48, 64])
    if do == "op":
        p, q = rng.choice([(1, 1), (1, 1), (1, 2), (2, 1)])
        ne = ne if p + q == 2 else rng.choice([6, 8, 10, 12, 16, 20, 24, 32])
        lmax = 60e6 / (ne - 1) ** q
        L = _log_int(rng, 2, int(lmax / ne if p == 1 else math.sqrt(lmax) / ne))
        return dict(do=do, which=rng.choice(["A", "A", "M", "K"]), p=p, q=q, L=min(L, 4096), ne=ne,
                    delta=rng.randint(1, max(1, ne // 8)))
    if do == "schwarz":
        p, prec = rng.choice([1, 1, 1, 2]), rng.choice(["fp64", "fp64", "fp32", "bf16x3", "bf16"])
        if p == 2:
            ne, L, delta, prec = rng.choice([8, 10, 12, 16]), rng.randint(5, 16), 1, rng.choice(["bf16", "bf16x3"])
        else:
            L, delta = _log_int(rng, 6, 256), rng.randint(1, max(1, ne // 10))
        return dict(do=do, kind=rng.choice(["as1", "as2", "as2", "ras1", "ras2"]),
                    pu=rng.choice(["equal", "distance"]), prec=prec, p=p, q=1, L=L, ne=ne, delta=delta)
    if do == "solve":
        return dict(do=do, solver=rng.choice(["gmres", "cg", "ras2"]), prec="fp64", rtol=1e-8, p=1, q=1,
                    L=_log_int(rng, 6, 64), ne=ne, delta=max(1, ne // 16))
    if do == "grad":
        return dict(do=do, prec="fp64", p=1, q=1, L=_log_int(rng, 6, 64), ne=min(ne, 40), delta=max(1, ne // 16))
    if do == "setup":
        return dict(do=do, prec=rng.choice(["bf16", "fp64", "bf16x3", "fp32"]), p=1, q=1,
                    L=_log_int(rng, 6, 256), ne=ne, delta=max(1, ne // 16))
    if do == "eig":
        if rng.random() < 0.4:
            ne = rng.choice([8, 10, 12, 16, 20, 24])
            return dict(do=do, prec="fp32", p=1, q=2, L=_log_int(rng, 4, 24), ne=ne, delta=rng.choice([1, 2]))
        return dict(do=do, prec=rng.choice(["bf16", "bf16", "bf16x3", "fp64"]), p=1, q=1,
                    L=_log_int(rng, 8, 256), ne=ne, delta=max(1, ne // 16))
    lmin = rng.randint(5, 40)
    return dict(do=do, prec=rng.choice(["bf16", "bf16x3"]), p=1, q=1, n=rng.randint(2, 32), lmin=lmin,
                lmax=rng.randint(lmin + 1, 256), ne=rng.choice([8, 16, 32]), delta=rng.choice([1, 2]))


# ---- inputs and one pass ----------------------------------------------------

def _potential(p, seed):
    rng = np.random.default_rng(seed)
    if p == 1:
        a, phi = rng.uniform(0.0, 10.0, 4), rng.uniform(0.0, 2.0 * math.pi, 4)
        return dict(kind="sep_fourier", a=a.tolist(), phi=phi.tolist(), k=[1, 2, 3, 4], cy=0.5)
    km = [(k, m) for m in range(4) for k in range(4) if (k, m) != (0, 0)]
    a, phi = rng.uniform(0.0, 5.0, 15), rng.uniform(0.0, 2.0 * math.pi, 15)
    return dict(kind="fourier2", a=a.tolist(), phi=phi.tolist(), k=[k for k, _ in km], m=[m for _, m in km])


def _n_dof(c):
    return (c["L"] * c["ne"] - 1) ** c["p"] * (c["ne"] - 1) ** c["q"]


def _vector(c, seed, j):
    """A seeded standard-normal vector of the case's unknowns, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + j)
    return torch.randn(_n_dof(c), dtype=torch.float64, device="cuda", generator=g)


def _assemble(c, V, **kw):
    return dd.assemble(c["p"], c["q"], c["L"], c["ne"], V, c["delta"], **kw)


def _lengths(c, seed):
    return [int(v) for v in np.random.default_rng(77).integers(c["lmin"], c["lmax"] + 1, c["n"])]


def prepare(case, seed):
    c = case
    s = dict(case=c, V=_potential(c["p"], seed))
    if c["do"] == "op":
        # a plain operator apply needs no shift: K, M and A = K + M_V come from assembly
        s["prob"] = _assemble(c, s["V"], coarse=False)
        s["x"] = _vector(c, seed, 1)
        s["y"] = torch.empty_like(s["x"])
    elif c["do"] in ("schwarz", "solve"):
        kw = dict(pu=c["pu"]) if c["do"] == "schwarz" else dict(graphs=True)
        s["prob"] = _assemble(c, s["V"], local_prec=c["prec"], **kw)
        dd.cell_shift(s["prob"])
        s["x"] = _vector(c, seed, 1)
        s["y"] = torch.empty_like(s["x"])
    elif c["do"] == "grad":
        s["theta"] = torch.tensor(ag.param_vector(s["V"]), device="cuda").requires_grad_()
        s["b"], s["g"] = _vector(c, seed, 1).requires_grad_(), _vector(c, seed, 2)
        s["geom"] = dict(p=c["p"], q=c["q"], L=c["L"], ne=c["ne"], delta=c["delta"], V=s["V"])
    elif c["do"] == "setup":
        s["x"] = _vector(c, seed, 1)
        s["y"] = torch.empty_like(s["x"])
    elif c["do"] == "eig":
        s["prob"] = _assemble(c, s["V"], local_prec=c["prec"], graphs=True)
        dd.cell_shift(s["prob"])
        s["x"] = torch.empty(s["prob"].n_dof, dtype=torch.float64, device="cuda")
    elif c["do"] == "batch":
        s["probs"] = []
        for j, L in enumerate(_lengths(c, seed)):
            prob = _assemble(dict(c, L=L), _potential(1, 1000 * seed + j), local_prec=c["prec"])
            dd.cell_shift(prob)
            s["probs"].append(prob)
        s["batch"] = dd.batch_create(s["probs"], reproducible=True)
        s["xs"] = [torch.empty(p.n_dof, dtype=torch.float64, device="cuda") for p in s["probs"]]
    return s


def run(state):
    s = state
    c = s["case"]
    if c["do"] == "op":
        dd.apply_op(s["prob"], c["which"], s["x"], s["y"])
        return s["y"]
    if c["do"] == "schwarz":
        dd.apply_schwarz(s["prob"], c["kind"], s["x"], s["y"])
        return s["y"]
    if c["do"] == "solve":
        s["y"].zero_()
        if c["solver"] == "gmres":
            dd.gmres_solve(s["prob"], s["x"], s["y"], rtol=c["rtol"])
        elif c["solver"] == "cg":
            dd.pcg_solve(s["prob"], s["x"], s["y"], rtol=c["rtol"])
        else:
            dd.stationary_ras(s["prob"], s["x"], s["y"], levels=2, rtol=c["rtol"])
        return s["y"]
    if c["do"] == "grad":
        u = ag.ShiftedSolveFn.apply(s["theta"], s["b"], s["geom"], dict(local_prec=c["prec"]))
        gt, gb = torch.autograd.grad(u, (s["theta"], s["b"]), s["g"])
        return dict(u=u.detach(), gtheta=gt, gb=gb)
    if c["do"] == "setup":
        prob = _assemble(c, s["V"], local_prec=c["prec"], graphs=True)
        sigma, psi = dd.cell_shift(prob)
        dd.apply_precond(prob, s["x"], s["y"])
        return dict(sigma=sigma, psi=psi, z=s["y"])
    if c["do"] == "eig":
        s["x"].zero_()
        r = dd.inverse_iteration(s["prob"], s["x"])
        return dict(lam=r["lam"], x=s["x"])
    for x in s["xs"]:
        x.zero_()
    _, info = dd.batch_inverse_iteration(s["batch"], s["xs"])
    return dict(lam=np.array([r["lam"] for r in info]), x=torch.cat(s["xs"]))


# ---- indispensable work -----------------------------------------------------

# Steps of the iterative calls, as rounded typical counts of the method: CG or
# GMRES steps of one shifted solve, the two-level stationary iteration's, and
# outer steps of an eigen-solve.
_STEPS = dict(cg=100, gmres=100, ras2=400, outer=10)


def _local_flops(c):
    """Exact banded solves of every subdomain: 4 m hb flops for m unknowns of half-bandwidth hb."""
    d = sorted([c["ne"] + 2 * c["delta"] - 1] * c["p"] + [c["ne"] - 1] * c["q"])
    m = math.prod(d)
    hb = d[0] + 1 if len(d) == 2 else d[0] * (d[1] + 1) + 1
    return 4.0 * m * hb * c["L"] ** c["p"], 8.0 * m * hb, m, hb


def work(case):
    c = case
    if c["do"] == "batch":
        ws = [work(dict(c, do="eig", L=L)) for L in _lengths(c, 0)]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    n = float(_n_dof(c))
    taps = 3 ** (c["p"] + c["q"])
    table = 8.0 * taps * c["ne"] ** c["p"] * (c["ne"] - 1) ** c["q"]
    flops, factor, m, hb = _local_flops(c)
    if c["do"] == "op":
        return dict(bytes=16.0 * n + table, flops=2.0 * taps * n)
    if c["do"] == "schwarz":
        return dict(bytes=16.0 * n + factor, flops=flops + 4.0 * n)
    if c["do"] == "setup":
        # tables and the banded factorisations of the cell and of one local matrix, one application
        return dict(bytes=16.0 * n + table + factor, flops=flops + 4.0 * m * hb * hb)
    # a step: operator, local solves and five vectors' updates; every vector of it
    # read and written once (96 bytes per unknown)
    step = dict(bytes=96.0 * n + table + factor, flops=flops + (2.0 * taps + 14.0) * n)
    k = {"solve": _STEPS[c.get("solver", "cg")], "grad": 2 * _STEPS["cg"],
         "eig": _STEPS["outer"] * _STEPS["cg"]}[c["do"]]
    return dict(bytes=k * step["bytes"], flops=k * step["flops"])


# ---- the same results in plain torch FP64 -----------------------------------

_GP = (0.5 * (1.0 - 1.0 / math.sqrt(3.0)), 0.5 * (1.0 + 1.0 / math.sqrt(3.0)))


def _V_at(V, p, z):
    """V at coordinates z (one tensor per axis, broadcast against each other)."""
    if V["kind"] == "sep_fourier":
        v = sum(a * torch.cos(2.0 * math.pi * k * z[0] + f) for a, f, k in zip(V["a"], V["phi"], V["k"]))
        env = 1.0
        for y in z[p:]:
            env = env * torch.sin(math.pi * y)
        return v * (1.0 + V["cy"] * env)
    v = sum(a * torch.cos(2.0 * math.pi * (k * z[0] + m * z[1]) + f)
            for a, f, k, m in zip(V["a"], V["phi"], V["k"], V["m"]))
    return v + 0.0 * z[-1]


class _Fem:
    """Q1 forms with the tensor 2-point rule on a box of elements of the periodic
    mesh: first element e0 and count nel per axis (axis 0 fastest in memory)."""

    def __init__(self, c, V, e0=None, nel=None, device="cuda"):
        p, d = c["p"], c["p"] + c["q"]
        self.c, self.V, self.p, self.d, self.h, self.dev = c, V, p, d, 1.0 / c["ne"], device
        self.e0 = e0 or [0] * d
        self.nel = nel or [c["L"] * c["ne"]] * p + [c["ne"]] * c["q"]
        self.pts = list(itertools.product((0, 1), repeat=d))  # per axis, both points and corners
        self.w = self.h ** d / 2 ** d

    def pot(self, b, V=None):
        z = []
        for a in range(self.d):
            e = torch.arange(self.nel[a], dtype=torch.float64, device=self.dev) + self.e0[a]
            t = (torch.remainder(e, self.c["ne"]) if a < self.p else e) + _GP[b[a]]
            z.append((t * self.h).reshape([-1 if k == self.d - 1 - a else 1 for k in range(self.d)]))
        return _V_at(V or self.V, self.p, z)

    def shape(self, b, k, da=-1):
        """Corner k's shape function (or its derivative along axis da) at point b."""
        v = 1.0
        for a in range(self.d):
            t = _GP[b[a]]
            v *= ((1.0 if k[a] else -1.0) / self.h) if a == da else (t if k[a] else 1.0 - t)
        return v

    def at(self, k):
        return tuple(slice(k[self.d - 1 - i], k[self.d - 1 - i] + self.nel[self.d - 1 - i]) for i in range(self.d))

    def apply(self, x, kin, V=None, mass=0.0, pot=True):
        """(kin K + M_V + mass M) x on the interior nodes; pot=False leaves M_V out."""
        sh = [self.nel[self.d - 1 - i] + 1 for i in range(self.d)]
        xp = torch.zeros(sh, dtype=torch.float64, device=self.dev)
        inner = tuple(slice(1, -1) for _ in sh)
        xp[inner] = x.reshape([v - 2 for v in sh])
        y = torch.zeros_like(xp)
        for b in self.pts:
            coef = (self.pot(b, V) if pot else 0.0) + mass
            val = sum(self.shape(b, k) * xp[self.at(k)] for k in self.pts)
            val = val * (coef * self.w)
            gr = [sum(self.shape(b, k, a) * xp[self.at(k)] for k in self.pts) * (kin * self.w)
                  for a in range(self.d)] if kin else []
            for k in self.pts:
                y[self.at(k)] += self.shape(b, k) * val
                for a, g in enumerate(gr):
                    y[self.at(k)] += self.shape(b, k, a) * g
        return y[inner].reshape(-1)

    def dense(self, kin, mass, pot=True, periodic=False):
        """The dense matrix of kin K + M_V + mass M: interior nodes, or (periodic)
        wrapped along the expanding axes."""
        sh = [self.nel[self.d - 1 - i] for i in range(self.d)]
        num = []  # node number along each axis, -1 on a Dirichlet boundary
        for a in range(self.d):
            i = torch.arange(self.nel[a] + 1, device=self.dev)
            if periodic and a < self.p:
                num.append(i % self.nel[a])
            else:
                num.append(torch.where((i == 0) | (i == self.nel[a]), -1, i - 1))
        ext = [self.nel[a] if periodic and a < self.p else self.nel[a] - 1 for a in range(self.d)]
        N = math.prod(ext)
        node = {}
        for k in self.pts:
            idx, stride, ok = 0, 1, True
            for a in range(self.d):
                t = num[a][k[a]:k[a] + self.nel[a]].reshape([-1 if j == self.d - 1 - a else 1 for j in range(self.d)])
                idx, ok, stride = idx + t * stride, ok & (t >= 0), stride * ext[a]
            node[k] = (idx.expand(sh).reshape(-1), torch.as_tensor(ok).expand(sh).reshape(-1))
        A = torch.zeros(N * N, dtype=torch.float64, device=self.dev)
        pots = {b: ((self.pot(b) if pot else 0.0) + mass) * torch.ones(sh, dtype=torch.float64, device=self.dev)
                for b in self.pts}
        for k in self.pts:
            for l in self.pts:
                E = torch.zeros(sh, dtype=torch.float64, device=self.dev)
                for b in self.pts:
                    E += self.w * self.shape(b, k) * self.shape(b, l) * pots[b]
                    E += kin * self.w * sum(self.shape(b, k, a) * self.shape(b, l, a) for a in range(self.d))
                ok = node[k][1] & node[l][1]
                A.index_put_(((node[k][0] * N + node[l][0])[ok],), E.reshape(-1)[ok], accumulate=True)
        return A.reshape(N, N)


def _cell(c, V):
    """(sigma, psi) of the periodic cell problem, psi > 0 and M-normalised: subspace
    iterations from a lower bound, then Rayleigh quotient steps."""
    f = _Fem(c, V, nel=[c["ne"]] * (c["p"] + c["q"]))
    A, M = f.dense(1.0, 0.0, periodic=True), f.dense(0.0, 1.0, pot=False, periodic=True)
    low = min(float(f.pot(b).min()) for b in f.pts)
    Lc = torch.linalg.cholesky(A - low * M)
    x = torch.ones(A.shape[0], 1, dtype=torch.float64, device=f.dev)
    for _ in range(30):
        x = torch.cholesky_solve(M @ x, Lc)
        x = x / torch.sqrt(x.T @ M @ x)
    for _ in range(3):
        s = float(x.T @ A @ x)
        x = torch.linalg.solve(A - (s - 1e-9) * M, M @ x)
        x = x / torch.sqrt(x.T @ M @ x)
    x = x * torch.sign(x.sum())
    return float(x.T @ A @ x), x[:, 0]


def _boxes(c):
    """Per subdomain: first interior node (0-based) and extent along each axis, and its class."""
    L, ne, dl = c["L"], c["ne"], c["delta"]
    ax = []
    for i in range(1, L + 1):
        lo, hi = max((i - 1) * ne - dl + 1, 1), min(i * ne + dl - 1, L * ne - 1)
        ax.append((lo - 1, hi - lo + 1, (i == 1) + 2 * (i == L)))
    out = []
    for cells in itertools.product(range(L), repeat=c["p"]):  # last cell index slowest
        cells = cells[::-1]
        o = [ax[i][0] for i in cells] + [0] * c["q"]
        m = [ax[i][1] for i in cells] + [ne - 1] * c["q"]
        out.append((o, m, tuple(ax[i][2] for i in cells), cells))
    return out


def _pu(c, boxes):
    """Partition-of-unity weights on every box: equal, or distance to the interior faces."""
    N = [c["L"] * c["ne"] - 1] * c["p"] + [c["ne"] - 1] * c["q"]
    total = torch.zeros(N[::-1], dtype=torch.float64, device="cuda")
    ws = []
    for o, m, _, cells in boxes:
        w = torch.full(m[::-1], float("inf") if c.get("pu") == "distance" else 1.0,
                       dtype=torch.float64, device="cuda")
        if c.get("pu") == "distance":
            d = len(m)
            for a in range(c["p"]):
                i = torch.arange(m[a], dtype=torch.float64, device="cuda") + o[a] + 1
                t = torch.full_like(i, float("inf"))
                if cells[a] > 0:
                    t = torch.minimum(t, i - (cells[a] * c["ne"] - c["delta"]))
                if cells[a] < c["L"] - 1:
                    t = torch.minimum(t, (cells[a] + 1) * c["ne"] + c["delta"] - i)
                w = torch.minimum(w, t.reshape([-1 if j == d - 1 - a else 1 for j in range(d)]))
            w = torch.where(torch.isinf(w), 1.0, w)
        total[_at(o, m)] += w
        ws.append(w)
    return [w / total[_at(b[0], b[1])] for w, b in zip(ws, boxes)]


def _at(o, m):
    return tuple(slice(o[a], o[a] + m[a]) for a in reversed(range(len(o))))


def _schwarz(c, V, kind, r):
    """The preconditioner `kind` on r with exact local and coarse solves; also sigma and psi."""
    sigma, psi = _cell(c, V)
    boxes = _boxes(c)
    pu = _pu(c, boxes)
    N = [c["L"] * c["ne"] - 1] * c["p"] + [c["ne"] - 1] * c["q"]
    R = r.reshape(N[::-1])
    z = torch.zeros_like(R)
    classes = {}
    for i, b in enumerate(boxes):
        classes.setdefault(b[2], []).append(i)
    for mem in classes.values():
        o, m = boxes[mem[0]][:2]
        A = _Fem(c, V, e0=list(o), nel=[v + 1 for v in m]).dense(1.0, -sigma)
        rhs = torch.stack([R[_at(boxes[i][0], boxes[i][1])].reshape(-1) for i in mem], 1)
        sol = torch.cholesky_solve(rhs, torch.linalg.cholesky(A))
        for j, i in enumerate(mem):
            y = sol[:, j].reshape(m[::-1])
            z[_at(boxes[i][0], boxes[i][1])] += y * pu[i] if kind.startswith("ras") else y
    if kind.endswith("2"):
        ps = psi.reshape([c["ne"] - 1] * c["q"] + [c["ne"]] * c["p"])
        for a in range(c["p"]):  # node i of an expanding axis is cell node i mod ne
            ps = ps.index_select(len(N) - 1 - a, (torch.arange(N[a], device="cuda") + 1) % c["ne"])
        phi = [w * ps[_at(b[0], b[1])] for w, b in zip(pu, boxes)]
        n, f = len(boxes), _Fem(c, V)
        A0 = torch.zeros(n, n, dtype=torch.float64, device="cuda")
        for col in itertools.product(range(3), repeat=c["p"]):
            mine = {b[3]: i for i, b in enumerate(boxes) if all(v % 3 == k for v, k in zip(b[3], col))}
            v = torch.zeros_like(R)
            for i in mine.values():
                v[_at(boxes[i][0], boxes[i][1])] += phi[i]
            av = f.apply(v.reshape(-1), 1.0, mass=-sigma).reshape(R.shape)
            dots = torch.stack([(phi[t] * av[_at(boxes[t][0], boxes[t][1])]).sum() for t in range(n)])
            for t in range(n):
                for step in itertools.product((-1, 0, 1), repeat=c["p"]):
                    i = mine.get(tuple(u + s for u, s in zip(boxes[t][3], step)))
                    if i is not None:  # the other columns of this colour do not reach row t
                        A0[t, i] = dots[t]
        c0 = torch.stack([(phi[t] * R[_at(boxes[t][0], boxes[t][1])]).sum() for t in range(n)])
        y0 = torch.linalg.solve(0.5 * (A0 + A0.T), c0)
        for i, b in enumerate(boxes):
            z[_at(b[0], b[1])] += y0[i] * phi[i]
    return z.reshape(-1), sigma, psi


class _Direct:
    """Solves with K + M_V - sigma M for p = 1 by block elimination along x1."""

    def __init__(self, c, V, sigma):
        self.ns, self.ny, ne = c["L"] * c["ne"] - 1, (c["ne"] - 1) ** c["q"], c["ne"]
        d00, d01 = [], []
        ny = self.ny
        for e in range(ne):  # columns of elements e .. e+2 give the blocks of the nodes between them
            B = _Fem(c, V, e0=[e] + [0] * c["q"], nel=[3] + [ne] * c["q"], device="cpu").dense(1.0, -sigma)
            B = B.reshape(ny, 2, ny, 2)
            d00.append(B[:, 0, :, 0].contiguous())
            d01.append(B[:, 0, :, 1].contiguous())
        self.C, S = d01, None
        self.inv = []
        for i in range(self.ns):  # node i + 1 lies between element columns i and i + 1
            D = d00[i % ne]
            S = D if i == 0 else D - d01[(i - 1) % ne].T @ self.inv[-1] @ d01[(i - 1) % ne]
            self.inv.append(torch.cholesky_inverse(torch.linalg.cholesky(0.5 * (S + S.T))))

    def solve(self, b):
        ne = len(self.C)
        r = b.reshape(self.ny, self.ns, -1).permute(1, 0, 2).contiguous().cpu()
        y = [r[0]]
        for i in range(1, self.ns):
            y.append(r[i] - self.C[(i - 1) % ne].T @ (self.inv[i - 1] @ y[i - 1]))
        x = [None] * self.ns
        x[-1] = self.inv[-1] @ y[-1]
        for i in range(self.ns - 2, -1, -1):
            x[i] = self.inv[i] @ (y[i] - self.C[i % ne] @ x[i + 1])
        return torch.stack(x).permute(1, 0, 2).reshape(b.shape).to(b.device)


def exact(case, seed):
    c, V = case, _potential(case["p"], seed)
    if c["do"] == "op":
        return _Fem(c, V).apply(_vector(c, seed, 1), 0.0 if c["which"] == "M" else 1.0,
                                mass=1.0 if c["which"] == "M" else 0.0, pot=c["which"] == "A")
    if c["do"] == "schwarz":
        return _schwarz(c, V, c["kind"], _vector(c, seed, 1))[0]
    if c["do"] == "setup":
        z, sigma, psi = _schwarz(c, V, "as2", _vector(c, seed, 1))
        return dict(sigma=sigma, psi=psi.cpu().numpy(), z=z)
    if c["do"] == "batch" or c["q"] == 2:
        return None  # a direct solve takes too long here
    sigma, psi = _cell(c, V)
    D = _Direct(c, V, sigma)
    f = _Fem(c, V)
    if c["do"] == "solve":
        return D.solve(_vector(c, seed, 1))
    if c["do"] == "grad":
        u, w = D.solve(_vector(c, seed, 1)), D.solve(_vector(c, seed, 2))
        cell = _Fem(c, V, nel=[c["ne"]] * 2)
        Mu, grad = f.apply(u, 0.0, mass=1.0, pot=False), []
        for t in range(8):
            one = dict(V, k=[V["k"][t % 4]], a=[1.0 if t < 4 else V["a"][t - 4]],
                       phi=[V["phi"][t % 4] + (0.0 if t < 4 else 0.5 * math.pi)])
            ds = psi @ (_Fem(c, one, nel=cell.nel).dense(0.0, 0.0, periodic=True) @ psi)
            grad.append(-(w @ f.apply(u, 0.0, V=one) - ds * (w @ Mu)))
        return dict(u=u, gtheta=torch.stack(grad), gb=w)
    # eigenpair: a block of three vectors with Rayleigh-Ritz
    X = torch.stack([torch.sin(math.pi * (j + 1) * torch.arange(1, D.ns + 1, device="cuda") / (D.ns + 1))
                     for j in range(3)], 1).to(torch.float64)
    X = (X[None] * psi.reshape(D.ny, c["ne"]).sum(1)[:, None, None]).reshape(-1, 3)
    on = lambda X, **kw: torch.stack([f.apply(X[:, j].contiguous(), **kw) for j in range(3)], 1)  # noqa: E731
    MX = on(X, kin=0.0, mass=1.0, pot=False)
    for _ in range(15):
        X = D.solve(MX)
        AX, MX = MX, on(X, kin=0.0, mass=1.0, pot=False)  # A_sigma X is the previous M X
        GA, GM = X.T @ AX, X.T @ MX
        Lm = torch.linalg.cholesky(GM.cpu())
        G = torch.linalg.solve_triangular(Lm, (0.5 * (GA + GA.T)).cpu(), upper=False)
        ev, Q = torch.linalg.eigh(torch.linalg.solve_triangular(Lm, G.T, upper=False))
        Q = torch.linalg.solve_triangular(Lm.T, Q, upper=True).to(X.device)
        X, MX = X @ Q, MX @ Q
    x = X[:, 0] * torch.sign(MX[:, 0].sum())
    return dict(lam=float(sigma + ev[0]), x=x)
