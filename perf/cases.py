"""Performance cases: what a program that uses the library has it do.

Each case is one call, or the few calls of one short run, through the
package's public functions, on inputs made on the GPU from a seed.  The
listed cases cover the calls by use: from a 200-cell advection line, where
launches and latency count, to the 256^3 Euler step; both stencil widths, the
fixed and the adaptive cutoff, several limiters, periodic and transmissive
axes, odd extents; the forward calls, the batched problems and the adjoint.
`draw` gives further cases of the same ranges.

`exact` is the same result in plain float64 torch operations, written from
the scheme's definition (polynomials on the candidate stencils, their
smoothness measures, the cutoff, the limiters, Roe projection, SSP-RK3) and,
for the adjoint, torch's own differentiation of it; it calls nothing of the
package.
"""
import functools
import math
from fractions import Fraction

import numpy as np
import torch

import paper_2010_13289_amd as T
from paper_2010_13289_amd import opcount

DEV = "cuda"
GAMMA = 1.4
CFL = 0.4
SCALAR, EULER = T.SYS_SCALAR, T.SYS_EULER


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def _case(kind, scheme=6, limiter=T.LIM_MP, **more):
    return {"kind": kind, "scheme": scheme, "limiter": limiter, **more}


def _grid_case(kind, n, bc="p", system=EULER, **more):
    """n: extents in x, y, z order; bc: p (periodic) or t (transmissive) per axis."""
    d = dict(zip(("nx", "ny", "nz"), n))
    return _case(kind, ndim=len(n), bc=(bc * len(n))[:len(n)], system=system, **d, **more)


def listed():
    tvd, va = T.LIM_TVD_MINMOD, T.LIM_VA
    return [
        # the scalar test problem of every scheme study: tiny, bound by launches
        {"name": "advection_1d_200", **_grid_case("step", (200,), system=SCALAR, call="fixed", steps=10)},
        # one shock tube on a fine line: few workgroups, latency
        {"name": "riemann_1d_4096", **_grid_case("step", (4096,), "t", scheme=8, limiter=tvd, call="cfl", steps=5)},
        # face fluxes and smoothness flags of one axis, for analysis
        {"name": "faces_flags_3d_64", **_grid_case("faces", (64, 64, 64), scheme=8, axis=2)},
        # the semi-discrete operator alone, for a program's own time integrator; odd extents, mixed boundaries
        {"name": "divergence_2d_517x389", **_grid_case("divergence", (517, 389), "pt", scheme=T.SCHEME_8A, limiter=va)},
        # an ordinary 2D run, steps without allocation
        {"name": "step_2d_1024", **_grid_case("step", (1024, 1024), call="noalloc", steps=2)},
        # the 3D benchmark step
        {"name": "step_3d_256", **_grid_case("step", (256, 256, 256), call="cfl", steps=1)},
        # a 3D run on an odd box, adaptive eight-point scheme
        {"name": "step_3d_187x150x93", **_grid_case("step", (187, 150, 93), "tpp", scheme=T.SCHEME_8A, call="cfl", steps=1)},
        # thousands of ragged 1D problems in one captured graph
        {"name": "batch_graph_4096", **_case("batch", scheme=8, count=4096, lo=256, hi=16384, bc="t", call="graph", steps=10)},
        # a few hundred of them in one persistent launch
        {"name": "batch_persistent_300", **_case("batch", scheme=8, count=300, lo=256, hi=16384, bc="t", call="persistent",
                                                 steps=10)},
        # one vector-Jacobian product of the operator, for a program's own adjoint
        {"name": "vjp_2d_1024", **_grid_case("vjp", (1024, 1024))},
        # gradient of a loss through a short differentiable run
        {"name": "rollout_2d_256", **_grid_case("rollout", (256, 256), steps=20, checkpoint=10)},
        # adjoint of one 3D step, stage states recomputed
        {"name": "step_vjp_3d_72x64x56", **_grid_case("step_vjp", (72, 64, 56))},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    limiters = (T.LIM_MP, T.LIM_MP, T.LIM_MP, T.LIM_TVD_MINMOD, T.LIM_TVD5, T.LIM_VA, T.LIM_TENO, T.LIM_MP_M4_B2,
                T.LIM_MP_MM_B1)
    method = {"scheme": rng.choice((6, 6, 8, T.SCHEME_8A)), "limiter": rng.choice(limiters)}

    def box(nd):
        if nd == 1:
            return (size(64, 65536),)
        if nd == 2:
            return (size(48, 1400), size(48, 1400))
        return (size(24, 160), size(24, 160), size(24, 160))

    def bc(nd):
        return "".join(rng.choice("ppt") for _ in range(nd))

    kind = rng.choice(("step", "step", "step", "step", "faces", "divergence", "batch", "batch", "vjp", "rollout",
                       "step_vjp"))
    if kind == "step":
        nd = rng.choice((1, 2, 3, 3))
        system = SCALAR if rng.random() < 0.15 else EULER
        n = box(nd)
        call = rng.choice(("fixed", "cfl", "cfl", "noalloc" if math.prod(n) <= 1 << 20 else "cfl"))
        return _grid_case(kind, n, bc(nd), system, **method, call=call, steps=rng.randint(1, 8 if nd == 1 else 2))
    if kind in ("faces", "divergence"):
        nd = rng.choice((1, 2, 3))
        n = box(nd)
        more = {"axis": rng.randrange(nd)} if kind == "faces" else {}
        return _grid_case(kind, n, bc(nd), **method, **more)
    if kind == "batch":
        return _case(kind, **method, count=size(8, 1024), lo=size(64, 512), hi=size(1024, 16384), bc=rng.choice("pt"),
                     call=rng.choice(("eager", "graph", "persistent")), steps=rng.randint(1, 10))
    if kind == "rollout":
        n = (size(48, 256), size(48, 256))
        return _grid_case(kind, n, bc(2), **method, steps=rng.randint(2, 12), checkpoint=rng.randint(2, 8))
    n = (size(48, 1024), size(48, 1024)) if rng.random() < 0.5 else (size(24, 80), size(24, 80), size(24, 80))
    return _grid_case(kind, n, bc(len(n)), **method)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _cutoff(case):
    """The cutoff the tests and the benchmark use for each stencil width."""
    return 1e-5 if case["scheme"] & 0xFF == 6 else 1e-7


def _extents(case):
    return [case[k] for k in ("nx", "ny", "nz")[:case["ndim"]]]


def _lengths(case):
    """Unit box, [-1, 1] for advection, 2 pi for the 3D vortex."""
    length = 2.0 if case["system"] == SCALAR else (2.0 * math.pi if case["ndim"] == 3 else 1.0)
    return [length] * case["ndim"]


def _grid(case):
    n = _extents(case)
    dx = [length / m for length, m in zip(_lengths(case), n)]
    bc = [T.BC_PERIODIC if b == "p" else T.BC_TRANSMISSIVE for b in case["bc"]]
    return T.Grid(ndim=len(n), n=n, dx=dx, bc=bc, system=case["system"], adv=(1.0, -0.7, 0.4)[:len(n)])


def _axes(n):
    """Cell centres of the unit interval along each axis, shaped to broadcast over [z][y][x]."""
    out = []
    for d, m in enumerate(n):
        x = (torch.arange(m, dtype=torch.float64, device=DEV) + 0.5) / m
        out.append(x.reshape([m if len(n) - 1 - k == d else 1 for k in range(len(n))]))
    return out


def _waves(n, rng, kmax, count, amp):
    """A sum of `count` cosine modes with integer wavevectors 0 < |k| <= kmax and random phases, of largest value amp."""
    x = _axes(n)
    f = torch.zeros([m for m in reversed(n)], dtype=torch.float64, device=DEV)
    for _ in range(count):
        while True:
            k = rng.integers(-kmax, kmax + 1, size=len(n))
            if 0 < int(k @ k) <= kmax * kmax:
                break
        f += torch.cos(2.0 * math.pi * sum(int(k[d]) * x[d] for d in range(len(n))) + rng.uniform(0.0, 2.0 * math.pi))
    return f * (amp / float(f.abs().max()))


def _conservative(rho, vel, p):
    ke = 0.5 * rho * sum(v * v for v in vel)
    return torch.stack([rho] + [rho * v for v in vel] + [p / (GAMMA - 1.0) + ke]).contiguous()


def _riemann_states(rng, count):
    """rho in [0.1, 1], u in [-1, 1], p in [0.1, 1] on either side: [count, 2, 3]."""
    return rng.uniform([0.1, -1.0, 0.1], [1.0, 1.0, 1.0], size=(count, 2, 3))


def _initial(case, seed):
    """The state a run of this kind starts from (float64 on the GPU)."""
    rng = np.random.default_rng(seed)
    n = _extents(case)
    x = _axes(n)
    nd = len(n)
    if case["system"] == SCALAR:  # a sine and a square pulse, moved by the seed
        s = [(v + rng.uniform()) % 1.0 for v in x]
        u = sum(torch.sin(2.0 * math.pi * v) for v in s)
        pulse = functools.reduce(torch.logical_and, [(v >= 0.3) & (v <= 0.4) for v in s])
        return (u + pulse.double())[None].contiguous()
    if nd == 1:  # a shock tube
        st = torch.from_numpy(_riemann_states(rng, 1)[0]).to(DEV)
        side = (x[0] >= rng.uniform(0.45, 0.55)).long()
        rho, u, p = (st[side, c] for c in range(3))
        return _conservative(rho, [u], p)
    if nd == 2:  # density modes, halved inside a circle, in slow motion
        rho = 1.0 + _waves(n, rng, 32, 48, 0.05)
        cx, cy = rng.uniform(0.4, 0.6, size=2)
        rho = torch.where((x[0] - cx) ** 2 + (x[1] - cy) ** 2 < 0.04, 0.5 * rho, rho)
        return _conservative(rho, [_waves(n, rng, 16, 16, 1e-2) for _ in range(2)], 1.0 + _waves(n, rng, 16, 16, 1e-2))
    # Taylor-Green velocity and pressure (moved by the seed, off the grid's symmetry), a planar density jump,
    # perturbed velocity
    a = [2.0 * math.pi * (v + rng.uniform()) for v in x]
    u = torch.sin(a[0]) * torch.cos(a[1]) * torch.cos(a[2])
    v = -torch.cos(a[0]) * torch.sin(a[1]) * torch.cos(a[2])
    p = 100.0 + ((torch.cos(2 * a[0]) + torch.cos(2 * a[1])) * (2.0 + torch.cos(2 * a[2])) - 2.0) / 16.0
    rho = 1.0 - 0.875 * (x[0] >= 0.5).double() + torch.zeros_like(u)
    vel = [c + _waves(n, rng, 16, 16, 1e-2) for c in (u, v, torch.zeros_like(u))]
    return _conservative(rho, vel, p)


def _batch_sizes(case):
    """Log-uniform problem sizes, the same for every seed."""
    rng = np.random.default_rng(case["count"])
    n = np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), size=case["count"])))
    return n.astype(np.int64)


def _batch_initial(n, seed):
    """One shock tube per problem on [0, 1], split at 0.5, packed end to end: [3][total]."""
    st = torch.from_numpy(_riemann_states(np.random.default_rng(seed + 1), len(n))).to(DEV)
    nt = torch.from_numpy(n).to(DEV)
    prob = torch.repeat_interleave(torch.arange(len(n), device=DEV), nt)
    first = torch.cumsum(nt, 0) - nt
    x = (torch.arange(int(n.sum()), device=DEV) - first[prob] + 0.5) / nt[prob]
    side = (x >= 0.5).long()
    rho, u, p = (st[prob, side, c] for c in range(3))
    return _conservative(rho, [u], p)


def _fixed_dt(case, U):
    """CFL / largest signal rate of the initial state."""
    return CFL / float(_rate(U, _extents(case), [length / m for length, m in zip(_lengths(case), _extents(case))],
                             case["system"]))


def prepare(case, seed):
    s = {"case": case, "method": (case["scheme"], case["limiter"], _cutoff(case), GAMMA)}
    if case["kind"] == "batch":
        n = _batch_sizes(case)
        s["plan"] = T.BatchPlan(n, 1.0 / n, T.BC_PERIODIC if case["bc"] == "p" else T.BC_TRANSMISSIVE)
        s["U0"] = _batch_initial(n, seed)
        s["U"] = s["U0"].clone()
        return s
    g = s["grid"] = _grid(case)
    U0 = s["U0"] = _initial(case, seed)
    kind = case["kind"]
    if kind == "step":
        s["U"] = U0.clone()
        if case["call"] == "fixed":
            s["dt"] = _fixed_dt(case, U0)
        if case["call"] != "noalloc":
            s["ws"] = T.Workspace(g, case["scheme"], DEV)
    elif kind == "vjp":
        s["Lbar"] = _cotangent(U0, seed)
        s["ws"] = T.vjp_workspace(g, case["scheme"], DEV)
    elif kind == "step_vjp":
        s["Ubar0"] = _cotangent(U0, seed)
        s["Ubar"] = s["Ubar0"].clone()
        s["dt"] = _fixed_dt(case, U0)
        s["ws"] = T.rk3_vjp_workspace(g, case["scheme"], DEV)
    elif kind == "rollout":
        s["target"] = _target(case, seed)
        s["dt"] = _fixed_dt(case, U0)
        U0.requires_grad_(True)
    return s


def _cotangent(U, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed + 2)
    return torch.randn(U.shape, dtype=torch.float64, device=DEV, generator=gen)


def _target(case, seed):
    """The density a run's result is held against."""
    return _initial(case, seed + 1)[0].contiguous()


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    c, m = s["case"], s["method"]
    kind = c["kind"]
    if kind == "batch":
        advance = {"eager": s["plan"].rk3, "graph": s["plan"].rk3_graph, "persistent": s["plan"].rk3_persistent}[c["call"]]
        s["U"].copy_(s["U0"])
        return advance(s["U"], *m, CFL, steps=c["steps"])
    g = s["grid"]
    if kind == "step":
        U = s["U"]
        U.copy_(s["U0"])
        for _ in range(c["steps"]):
            if c["call"] == "fixed":
                T.rk3_step(U, g, *m, s["dt"], workspace=s["ws"])
            elif c["call"] == "cfl":
                T.rk3_step_cfl(U, g, *m, CFL, workspace=s["ws"])
            else:
                T.rk3_step_cfl_noalloc(U, g, *m, CFL)
        return U
    if kind == "faces":
        flux, flags = T.reconstruct_faces(s["U0"], g, *m, c["axis"], return_flags=True)
        return {"flux": flux, "flags": flags}
    if kind == "divergence":
        return T.flux_divergence(s["U0"], g, *m)
    if kind == "vjp":
        return T.flux_divergence_vjp(s["U0"], s["Lbar"], g, *m, workspace=s["ws"])
    if kind == "step_vjp":
        s["Ubar"].copy_(s["Ubar0"])
        return T.rk3_step_vjp(s["U0"], s["Ubar"], g, *m, s["dt"], workspace=s["ws"])
    U = T.rollout(s["U0"], g, *m, s["dt"], c["steps"], checkpoint=c["checkpoint"])
    loss = 0.5 * ((U[0] - s["target"]) ** 2).sum()
    (grad,) = torch.autograd.grad(loss, s["U0"])
    return {"U": U.detach(), "grad": grad}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _face_ops(case, adjoint=False):
    """Operations per face vector with every candidate smooth (the limiter's part depends on the data)."""
    nd, K, ad = case.get("ndim", 1), case["scheme"] & 0xFF, bool(case["scheme"] & T.SCHEME_ADAPTIVE)
    if adjoint:
        return opcount.adjoint_face_vector_ops(nd, K, case["limiter"], ad, rough=0, nonsmooth=0)
    system = "scalar" if case.get("system") == SCALAR else "euler"
    return opcount.face_vector_ops(system, nd, K, case["limiter"], ad, rough=0, nonsmooth=0)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        # sizes log-uniform in [lo, hi]
        cells = case["count"] * (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
        return {"bytes": 2 * 24 * cells, "flops": 3 * case["steps"] * cells * _face_ops(case)}
    n = _extents(case)
    cells = math.prod(n)
    state = 8 * cells * (1 if case["system"] == SCALAR else len(n) + 2)
    axis_ops = cells * _face_ops(case)
    if kind == "faces":
        faces = cells // n[case["axis"]] * (n[case["axis"]] + 1)
        return {"bytes": state + state * faces / cells * (1 + 2 / 8), "flops": axis_ops}
    if kind == "divergence":
        return {"bytes": 2 * state, "flops": len(n) * axis_ops}
    if kind == "step":
        return {"bytes": 2 * state, "flops": 3 * len(n) * case["steps"] * axis_ops}
    reverse = len(n) * cells * _face_ops(case, adjoint=True)
    if kind == "vjp":
        return {"bytes": 3 * state, "flops": reverse}
    if kind == "step_vjp":  # two stages forward again, three reversed
        return {"bytes": 3 * state, "flops": 2 * len(n) * axis_ops + 3 * reverse}
    return {"bytes": 3 * state, "flops": case["steps"] * 3 * (len(n) * axis_ops + reverse)}


# ---------------------------------------------------------------------------
# the same results in plain float64 torch
# ---------------------------------------------------------------------------

def exact(case, seed):
    ct, dim = _cutoff(case), case.get("ndim", 1)
    if case["kind"] == "batch":
        n = _batch_sizes(case)
        with torch.no_grad():
            lines = _Packed(n, case["bc"])
            U = _batch_initial(n, seed)
            for _ in range(case["steps"]):
                dt = CFL / lines.largest(_signal_rate(U, [lines.dx]))
                U = _rk3(U, dt[lines.prob], lambda V: lines.divergence(V, case, ct))
        return U
    U = _initial(case, seed)
    n = _extents(case)
    dx = [length / m for length, m in zip(_lengths(case), n)]

    def rhs(V):
        out = 0.0
        for ax in range(dim):
            F, _ = _axis_faces(V, ax, case, ct)
            d = V.dim() - 1 - ax
            out = out - (F.narrow(d, 1, n[ax]) - F.narrow(d, 0, n[ax])) / dx[ax]
        return out

    kind = case["kind"]
    if kind == "step":
        with torch.no_grad():
            dt = _fixed_dt(case, U) if case["call"] == "fixed" else None
            for _ in range(case["steps"]):
                U = _rk3(U, dt if dt is not None else CFL / _rate(U, n, dx, case["system"]), rhs)
        return U
    if kind == "faces":
        with torch.no_grad():
            F, flags = _axis_faces(U, case["axis"], case, ct)
        return {"flux": F, "flags": flags}
    if kind == "divergence":
        with torch.no_grad():
            return rhs(U)

    def pullback(f, V, bar):
        V = V.detach().requires_grad_(True)
        return torch.autograd.grad(f(V), V, bar)[0]

    if kind == "vjp":
        return pullback(rhs, U, _cotangent(U, seed))
    dt = _fixed_dt(case, U)

    def step(V):
        return _rk3(V, dt, rhs)

    if kind == "step_vjp":
        return pullback(step, U, _cotangent(U, seed))
    states = [U]
    with torch.no_grad():
        for _ in range(case["steps"]):
            states.append(step(states[-1]))
    bar = torch.zeros_like(U)
    bar[0] = states[-1][0] - _target(case, seed)
    for V in reversed(states[:-1]):
        bar = pullback(step, V, bar)
    return {"U": states[-1], "grad": bar}


def _rk3(U, dt, rhs):
    U1 = U + dt * rhs(U)
    U2 = 0.75 * U + 0.25 * (U1 + dt * rhs(U1))
    return U / 3.0 + 2.0 / 3.0 * (U2 + dt * rhs(U2))


def _signal_rate(U, dx):
    nd = len(dx)
    vel = [U[1 + d] / U[0] for d in range(nd)]
    p = (GAMMA - 1.0) * (U[-1] - 0.5 * U[0] * sum(v * v for v in vel))
    c = torch.sqrt(GAMMA * p / U[0])
    return sum((vel[d].abs() + c) / dx[d] for d in range(nd))


def _rate(U, n, dx, system):
    if system == SCALAR:
        return torch.tensor(sum(abs(a) / h for a, h in zip((1.0, -0.7, 0.4), dx)), dtype=torch.float64)
    return _signal_rate(U, dx).max()


def _axis_faces(U, ax, case, ct):
    """Fluxes and smoothness bytes at faces 0 .. n of one axis (U: [field][z][y][x])."""
    dim = U.dim() - 1 - ax
    n, K = U.shape[dim], case["scheme"] & 0xFF
    cells = []
    for m in range(K):
        j = torch.arange(n + 1, device=U.device) - K // 2 + m
        j = j % n if case["bc"][ax] == "p" else j.clamp(0, n - 1)
        cells.append(U.index_select(dim, j))
    return _face_fluxes(cells, ax, case, ct)


class _Packed:
    """1D problems packed end to end: stencils and reductions per problem."""

    def __init__(self, n, bc):
        nt = torch.from_numpy(n).to(DEV)
        count = len(n)
        self.bc, self.count = bc, count
        self.prob = torch.repeat_interleave(torch.arange(count, device=DEV), nt)
        self.dx = (1.0 / nt.double())[self.prob]
        first = torch.cumsum(nt, 0) - nt
        self.fprob = torch.repeat_interleave(torch.arange(count, device=DEV), nt + 1)
        self.face = torch.arange(int(n.sum()) + count, device=DEV) - (first + torch.arange(count, device=DEV))[self.fprob]
        self.fn, self.fbase = nt[self.fprob], first[self.fprob]
        self.left = torch.arange(int(n.sum()), device=DEV) + self.prob  # face left of each cell

    def divergence(self, U, case, ct):
        K = case["scheme"] & 0xFF
        cells = []
        for m in range(K):
            j = self.face - K // 2 + m
            j = j % self.fn if self.bc == "p" else torch.minimum(j.clamp(min=0), self.fn - 1)
            cells.append(U[:, self.fbase + j])
        F, _ = _face_fluxes(cells, 0, {**case, "system": EULER}, ct)
        return -(F[:, self.left + 1] - F[:, self.left]) / self.dx

    def largest(self, r):
        out = torch.zeros(self.count, dtype=torch.float64, device=r.device)
        return out.scatter_reduce_(0, self.prob, r, "amax")


def _min(a, b):
    return torch.where(a <= b, a, b)


def _max(a, b):
    return torch.where(a >= b, a, b)


def _minmod(*v):
    lo, hi = functools.reduce(_min, v), functools.reduce(_max, v)
    zero = torch.zeros_like(lo)
    return torch.where(lo > 0, lo, torch.where(hi < 0, hi, zero))


def _face_fluxes(cells, ax, case, ct):
    """Flux and smoothness bytes from the K stencil states cells[m] = [field, ...]."""
    K = len(cells)
    if case["system"] == SCALAR:
        a = (1.0, -0.7, 0.4)[ax]
        fields = [([a * c[0] for c in cells], [abs(a) * c[0] for c in cells])]
        R = None
    else:
        nd = cells[0].shape[0] - 2
        order = [0, 1 + ax] + [1 + t for t in range(nd) if t != ax] + [nd + 1]
        states = [[c[q] for q in order] for c in cells]
        prims = [_primitive(X) for X in states]
        alpha = torch.zeros_like(states[0][0])
        for _, p, u in prims:
            lam = u["n"].abs() + torch.sqrt(GAMMA * p / u["rho"])
            alpha = torch.where(lam > alpha, lam, alpha)
        L, R = _eigenvectors(states[K // 2 - 1], states[K // 2])
        W = [L(X) for X in states]
        G = [L(F) for F, _, _ in prims]
        fields = [([G[m][q] for m in range(K)], [alpha * W[m][q] for m in range(K)]) for q in range(nd + 2)]
    values, flags = [], [[], []]
    for g, w in fields:
        plus, fp = _reconstruct([0.5 * (g[m] + w[m]) for m in range(K)], case, ct)
        minus, fm = _reconstruct([0.5 * (g[K - 1 - m] - w[K - 1 - m]) for m in range(K)], case, ct)
        values.append(plus + minus)
        flags[0].append(fp)
        flags[1].append(fm)
    flags = torch.stack([torch.stack(f) for f in flags])
    if R is None:
        return torch.stack(values), flags
    F = R(values)
    back = [order.index(f) for f in range(len(order))]
    return torch.stack([F[b] for b in back]), flags


def _primitive(X):
    """Flux along the normal, pressure and velocities of a state (density, normal momentum, tangential ones, energy)."""
    rho, E = X[0], X[-1]
    vel = [m / rho for m in X[1:-1]]
    p = (GAMMA - 1.0) * (E - 0.5 * rho * sum(v * v for v in vel))
    F = [X[1], X[1] * vel[0] + p] + [m * vel[0] for m in X[2:-1]] + [(E + p) * vel[0]]
    return F, p, {"n": vel[0], "all": vel, "rho": rho}


def _eigenvectors(XL, XR):
    """Left and right eigenvectors of the flux Jacobian at the Roe average, as functions of a vector."""
    def roe(X):
        _, p, u = _primitive(X)
        return torch.sqrt(X[0]), u["all"], (X[-1] + p) / X[0]

    (sl, ul, Hl), (sr, ur, Hr) = roe(XL), roe(XR)
    u = [(sl * a + sr * b) / (sl + sr) for a, b in zip(ul, ur)]
    H = (sl * Hl + sr * Hr) / (sl + sr)
    q2 = sum(v * v for v in u)
    c = torch.sqrt((GAMMA - 1.0) * (H - 0.5 * q2))
    b1 = (GAMMA - 1.0) / (c * c)

    def L(Y):
        A = 0.5 * q2 * b1 * Y[0] + b1 * (Y[-1] - sum(v * m for v, m in zip(u, Y[1:-1])))
        B = (u[0] * Y[0] - Y[1]) / c
        return [0.5 * (A + B), Y[0] - A] + [m - v * Y[0] for v, m in zip(u[1:], Y[2:-1])] + [0.5 * (A - B)]

    def R(w):
        s, d = w[0] + w[1] + w[-1], w[-1] - w[0]
        e = H * (w[0] + w[-1]) + u[0] * c * d + 0.5 * q2 * w[1] + sum(v * x for v, x in zip(u[1:], w[2:-1]))
        return [s, u[0] * s + c * d] + [v * s + x for v, x in zip(u[1:], w[2:-1])] + [e]

    return L, R


@functools.lru_cache(maxsize=None)
def _stencil(lo, hi):
    """The polynomial whose cell averages over cells lo .. hi (unit cells about 0) are given: its value at 1/2 as
    weights of the adjacent differences after cell 0's value, and the smoothness measure sum_l int (p^(l))^2 over
    cell 0 as rows y = rows @ differences, beta = sum y^2."""
    r = hi - lo + 1
    half = Fraction(1, 2)
    # averages of the monomials
    A = [[((c + half) ** (k + 1) - (c - half) ** (k + 1)) / (k + 1) for k in range(r)] for c in range(lo, hi + 1)]
    M = [row[:] + [Fraction(int(i == j)) for j in range(r)] for i, row in enumerate(A)]
    for i in range(r):
        piv = next(k for k in range(i, r) if M[k][i] != 0)
        M[i], M[piv] = M[piv], M[i]
        M[i] = [v / M[i][i] for v in M[i]]
        for k in range(r):
            if k != i:
                M[k] = [a - M[k][i] * b for a, b in zip(M[k], M[i])]
    coef = [row[r:] for row in M]  # coefficient k of p in the cell values
    # a step from cell j on: difference j is 1, the others 0
    steps = [[Fraction(int(i > j)) for i in range(r)] for j in range(r - 1)]
    d = [[sum(a * b for a, b in zip(row, s)) for s in steps] for row in coef]
    base = -lo  # cell 0 among lo .. hi
    at_half = [sum(d[k][j] * half ** k for k in range(r)) - steps[j][base] for j in range(r - 1)]
    # Gram matrix of the derivatives' inner products over cell 0 in the coefficients
    gram = [[Fraction(0)] * r for _ in range(r)]
    for a in range(1, r):
        for b in range(1, r):
            for order in range(1, min(a, b) + 1):
                fa = math.prod(range(a - order + 1, a + 1))
                fb = math.prod(range(b - order + 1, b + 1))
                e = a + b - 2 * order
                gram[a][b] += fa * fb * (half ** (e + 1) - (-half) ** (e + 1)) / (e + 1)
    Q = [[sum(d[a][i] * gram[a][b] * d[b][j] for a in range(r) for b in range(r)) for j in range(r - 1)]
         for i in range(r - 1)]
    chol = np.linalg.cholesky(np.array([[float(v) for v in row] for row in Q]))
    return [float(v) for v in at_half], chol.T.tolist()


_CANDIDATES = {6: ((-1, 1), (0, 2), (-2, 0), (0, 3)),
               8: ((-1, 1), (0, 2), (-2, 0), (0, 3), (-3, 0), (0, 4))}
_WEIGHTS = {6: (9 / 20, 3 / 10, 1 / 20, 1 / 5), 8: (3 / 7, 9 / 35, 2 / 35, 6 / 35, 1 / 70, 1 / 14)}


def _reconstruct(v, case, ct):
    """One reconstruction at the face right of cell 0 = v[K/2 - 1]: its value and the byte of smooth candidates."""
    K, lim = len(v), case["limiter"]
    c0 = K // 2 - 1
    D = [v[j + 1] - v[j] for j in range(K - 1)]

    def beta(lo, hi):
        out = 0.0
        for row in _stencil(lo, hi)[1]:
            y = sum(w * D[c0 + lo + j] for j, w in enumerate(row) if w != 0.0)
            out = out + y * y
        return out

    with torch.no_grad():
        b = [beta(*s) for s in _CANDIDATES[K]]
        tau = (beta(1 - K // 2, K // 2) - (b[1] + b[2] + 4.0 * b[0]) / 6.0).abs()
        gam = [(1.0 + tau / (x + 1e-40)) ** 6 for x in b]
        cut = (_adaptive_cutoff(D, c0) if case["scheme"] & T.SCHEME_ADAPTIVE else ct) * sum(gam)
        smooth = [~(x < cut) for x in gam]
        flags = sum(s.to(torch.uint8) << k for k, s in enumerate(smooth))
        del b, tau, gam, cut
    cand = [sum(w * D[c0 + lo + j] for j, w in enumerate(_stencil(lo, hi)[0])) for lo, hi in _CANDIDATES[K]]
    d = _WEIGHTS[K]
    if lim == T.LIM_TENO:
        w = [x * s.double() for s, x in zip(smooth, d)]
        return v[c0] + sum(x * c for x, c in zip(w, cand)) / sum(w), flags
    limited = _limit(D, c0, cand, lim)
    return v[c0] + sum(x * torch.where(s, c, m) for x, s, c, m in zip(d, smooth, cand, limited)), flags


def _adaptive_cutoff(D, c0):
    eps = 0.9 * 0.23 / (1.0 - 0.9 * 0.23) * 1e-6
    eta = functools.reduce(torch.minimum, [((2.0 * D[j] * D[j - 1]).abs() + eps) / (D[j] ** 2 + D[j - 1] ** 2 + eps)
                                           for j in range(c0 - 1, c0 + 3)])
    m = 1.0 - (eta / 0.23).clamp(max=1.0)
    g = (1.0 - m) ** 4 * (1.0 + 4.0 * m)
    return torch.pow(10.0, -torch.floor(10.5 - 3.5 * (1.0 - g)))


def _limit(D, c0, cand, lim):
    """What replaces each nonsmooth candidate, relative to cell 0's value."""
    dm, dp = D[c0 - 1], D[c0]
    zero = torch.zeros_like(dm)
    if lim == T.LIM_TVD_MINMOD:
        f = 0.5 * _minmod(dm, dp)
    elif lim == T.LIM_TVD5:
        B = (-2.0 * D[c0 - 2] + 11.0 * dm + 24.0 * dp - 3.0 * D[c0 + 1]) / 30.0
        up = _max(zero, _min(_min(2.0 * dm, 2.0 * dp), B))
        down = _min(zero, _max(_max(2.0 * dm, 2.0 * dp), B))
        f = 0.5 * torch.where(dm > 0, up, torch.where(dm < 0, down, zero))
    elif lim == T.LIM_VA:
        den = dp * dp + dm * dm
        live = den > 0
        phi = torch.where(live, 2.0 * dp * dm / torch.where(live, den, 1.0), zero)
        f = 0.25 * phi * ((1.0 - phi / 3.0) * dm + (1.0 + phi / 3.0) * dp)
    else:
        beta = {T.LIM_MP: 4.0, T.LIM_MP_M4_B2: 2.0, T.LIM_MP_MM_B4: 4.0, T.LIM_MP_MM_B2: 2.0, T.LIM_MP_MM_B1: 1.0}[lim]
        e = [D[c0 + j] - D[c0 + j - 1] for j in (-1, 0, 1)]  # curvatures at cells -1, 0, 1

        def measure(a, b):
            if lim in (T.LIM_MP, T.LIM_MP_M4_B2):
                return _minmod(4.0 * a - b, 4.0 * b - a, a, b)
            return _minmod(a, b)

        upper = 1.25 * dm
        median = 0.5 * dp - 0.5 * measure(e[1], e[2])
        large = 0.5 * dm + beta / 3.0 * measure(e[0], e[1])
        lo = _max(_min(_min(zero, dp), median), _min(_min(zero, upper), large))
        hi = _min(_max(_max(zero, dp), median), _max(_max(zero, upper), large))
        return [_min(_max(c, lo), hi) for c in cand]
    return [f] * len(cand)
