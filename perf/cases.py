"""The work that users of this library have it do, as cases that can be timed.

A case is a dict of plain values.  ``prepare`` builds what a solver program
holds before the call (the grid handle or server, and its state on the
device), ``run`` advances (or evaluates) it once through the public Python
entry points, ``exact`` gives the same result from a plain torch solver in 64
bits that shares no code with the library, and ``work`` counts the bytes and
operations the method cannot do without.

Keys of a case
  op       "step"      set a state, take ``steps`` steps, read the state back
           "residual"  one residual evaluation of the state the grid holds
           "noalloc"   steps on the caller's own state, without a workspace
           "serve"     a batch of solves through the continuous-batching server
  grid     "vortex"    2D uniform periodic block (isentropic vortex)
           "inlet"     2D curvilinear blocks, inflow to outflow, slip walls
           "viscous"   the inlet grid with no-slip walls and a viscosity
           "blobs"     3D uniform block, density blobs in a Mach 2 stream
           "curved"    3D curvilinear blocks linked around in i
  blocks, ni, nj, nk   blocks along i, cells of each block
  fp32     reconstruction and flux in FP32 (state and sums stay in FP64)
  limiter  0 minmod, 1 none
  rk       3 (SSP-RK3), 2 or 4 (the 2- and 4-stage schemes)
  source   the grid carries a cell-averaged source
  walls    "curved": slip walls at the k-faces (else periodic)
"""
import math
import time

import numpy as np
import torch

from paper_2305_18057_amd import cases as C
from paper_2305_18057_amd import fv

G = C.GAMMA
DEV = "cuda" if torch.cuda.is_available() else "cpu"
F64 = torch.float64


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _case(name, op, grid, blocks, ni, nj, nk=1, steps=1, fp32=False, limiter=0, rk=3, source=False,
          walls=False):
    return dict(name=name, op=op, grid=grid, blocks=blocks, ni=ni, nj=nj, nk=nk, steps=steps,
                fp32=fp32, limiter=limiter, rk=rk, source=source, walls=walls)


def listed():
    return [
        # one time step of a small unsteady problem, the loop of a coupled or
        # time-accurate program that looks at every step: latency and launches
        _case("vortex_one_step", "step", "vortex", 1, 128, 64),
        # residual evaluations, as an outer (implicit or adjoint) solver calls
        # them; ragged blocks (201 columns leave a 9-column tile)
        _case("residual_ragged", "residual", "inlet", 3, 201, 131),
        # the allocation-free entry point of a serving loop, 2-stage scheme
        _case("noalloc_small", "noalloc", "inlet", 2, 160, 121, steps=5, rk=2),
        # the headline workload: the 4 x 512 x 256 inlet in FP64
        _case("inlet_fp64", "step", "inlet", 4, 512, 256, steps=20),
        # a large 2D grid in the mixed-precision mode, 4-stage scheme
        _case("inlet_large_fp32flux", "step", "inlet", 8, 512, 1024, steps=4, fp32=True, rk=4),
        # viscous flow on the headline grid (no-slip walls, FP64)
        _case("viscous_fp64", "step", "viscous", 4, 512, 256, steps=10),
        # a smaller viscous run with a source term, ragged, mixed precision
        _case("viscous_source_ragged", "step", "viscous", 2, 301, 167, steps=10, fp32=True,
              source=True),
        # the 3D headline workload: 256^3 in FP64
        _case("blobs_256_fp64", "step", "blobs", 1, 256, 256, 256, steps=3),
        # a served 3D solve's size (32^3 .. 192^3), ragged, mixed precision
        _case("blobs_ragged_fp32flux", "step", "blobs", 1, 99, 90, 77, steps=10, fp32=True),
        # curvilinear 3D with a source (manufactured-solution style), 192^3
        _case("curved_192_fp64", "step", "curved", 2, 96, 192, 192, steps=2, source=True),
        # a mid-size body-fitted 3D grid with slip walls, unlimited scheme
        _case("curved_walls_ragged", "step", "curved", 3, 41, 50, 45, steps=5, limiter=1, walls=True),
        # a batch of uneven 2D solves through the server (64..1024 x 64..512
        # cells, mixed precision), submission to last result
        _case("serve_batch", "serve", "inlet", 12, 1024, 512, steps=50, fp32=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["vortex", "inlet", "inlet", "viscous", "blobs", "curved", "residual",
                       "noalloc", "serve"])
    fp32 = rng.random() < 0.4
    lim = 1 if rng.random() < 0.15 else 0  # unlimited: smooth flows only
    rk = rng.choice([3, 3, 3, 2, 4])
    if kind == "serve":
        return _nameless(_case("", "serve", "inlet", rng.randint(2, 12), _log(rng, 128, 1024),
                               _log(rng, 64, 512), steps=rng.randint(10, 50), fp32=fp32))
    if kind == "vortex":
        return _nameless(_case("", "step", "vortex", 1, _log(rng, 48, 600), _log(rng, 32, 400),
                               steps=_log(rng, 1, 20), fp32=fp32, limiter=lim, rk=rk))
    if kind in ("inlet", "viscous", "residual", "noalloc"):
        blocks = rng.randint(1, 4)
        ni, nj = _log(rng, 48, 700), _log(rng, 40, 600)
        if kind == "noalloc":  # the static scratch holds about 700 k cells
            ni, nj = _log(rng, 48, 400), _log(rng, 40, 300)
        op = kind if kind in ("residual", "noalloc") else "step"
        grid = "viscous" if kind == "viscous" else "inlet"
        return _nameless(_case("", op, grid, blocks, ni, nj, steps=1 if op == "residual" else _log(rng, 1, 12),
                               fp32=fp32, rk=rk,
                               source=grid == "viscous" and rng.random() < 0.3))
    if kind == "blobs":
        return _nameless(_case("", "step", "blobs", 1, _log(rng, 32, 200), _log(rng, 32, 200),
                               _log(rng, 32, 200), steps=_log(rng, 1, 6), fp32=fp32, limiter=lim, rk=rk))
    return _nameless(_case("", "step", "curved", rng.randint(1, 3), _log(rng, 24, 90), _log(rng, 24, 140),
                           _log(rng, 24, 140), steps=_log(rng, 1, 4), fp32=fp32, limiter=lim, rk=rk,
                           source=rng.random() < 0.5, walls=rng.random() < 0.5))


def _nameless(c):
    del c["name"]
    return c


# --------------------------------------------------------------------------
# inputs: grids, boundary rules, states
# --------------------------------------------------------------------------
def _waves(seed, count, ndim):
    """``count`` smooth fields of three random modes each, with values of
    order one, on unit coordinates."""
    r = np.random.default_rng(seed)
    k = r.integers(1, 5, size=(count, 3, ndim))
    ph = r.uniform(0.0, 2.0 * math.pi, size=(count, 3, ndim))
    a = r.uniform(0.3, 0.6, size=(count, 3))

    def field(f, xs):
        out = 0.0
        for m in range(3):
            t = a[f, m]
            for d in range(ndim):
                t = t * torch.sin(2.0 * math.pi * float(k[f, m, d]) * xs[d] + float(ph[f, m, d]))
            out = out + t
        return out
    return field


def _noise(seed, shape):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return torch.randn(shape, generator=g, device=DEV, dtype=F64)


def _conserved(rho, vel, p):
    ke = sum(v * v for v in vel)
    return torch.stack([rho] + [rho * v for v in vel] + [p / (G - 1.0) + 0.5 * rho * ke])


def _unit(n, dims, axis):
    c = (torch.arange(n, device=DEV, dtype=F64) + 0.5) / n
    return c.reshape([n if a == axis else 1 for a in range(dims)])


def _grid_2d(c, seed):
    nb, ni, nj = c["blocks"], c["ni"], c["nj"]
    N = nb * ni
    w = _waves(seed, 4, 2)
    xs = [_unit(N, 2, 1), _unit(nj, 2, 0)]
    rho_n = 1.0 + 2e-3 * _noise(seed, (nj, N))
    if c["grid"] == "vortex":
        hx, hy = 20.0 / N, 10.0 / nj
        X, Y = xs[0] * 20.0 - 10.0, xs[1] * 10.0 - 5.0
        e = 5.0 / (2.0 * math.pi) * torch.exp(0.5 * (1.0 - X * X - Y * Y))
        T = 1.0 - (G - 1.0) / (2.0 * G) * e * e
        rho = T ** (1.0 / (G - 1.0)) * (1.0 + 0.02 * w(0, xs))
        u, v = 0.5 * math.sqrt(G) - e * Y + 0.02 * w(1, xs), e * X + 0.02 * w(2, xs)
        U = _conserved(rho * rho_n, [u, v], T ** (G / (G - 1.0)) * (1.0 + 0.02 * w(3, xs)))
        blk = [C.Block(N, nj, 1, None, None, (0.0, 0.0, 0.0), (hx, hy, 1.0),
                       [C.BC(C.PERIODIC) for _ in range(6)])]
        return blk, [U], C.qref_of((1.0, 0.5 * math.sqrt(G), 0.0, 0.0, 1.0), 2), 0.0
    prim = C.inlet_freestream()
    rho0, u0, _, _, p0 = prim
    c0 = math.sqrt(G * p0 / rho0)
    rho = rho0 * (1.0 + 0.05 * w(0, xs)) * rho_n
    u = u0 * (1.0 + 0.02 * w(1, xs))
    v = 0.1 * c0 * w(2, xs) * torch.sin(math.pi * xs[1])
    U = _conserved(rho, [u, v], p0 * (1.0 + 0.05 * w(3, xs)))
    X, Y = C.inlet_mesh(N, nj)
    wall = C.NOSLIP if c["grid"] == "viscous" else C.SLIPWALL
    blk, Us = [], []
    for b in range(nb):
        lo = C.BC(C.BLOCK, b - 1, C.IMAX) if b else C.BC(C.INFLOW, prim=prim)
        hi = C.BC(C.BLOCK, b + 1, C.IMIN) if b < nb - 1 else C.BC(C.EXTRAP)
        s = slice(b * ni, (b + 1) * ni + 1)
        blk.append(C.Block(ni, nj, 1, X[:, s].copy(), Y[:, s].copy(), (0.0, 0.0, 0.0), (1.0, 1.0, 1.0),
                           [lo, hi, C.BC(wall), C.BC(wall), C.BC(C.PERIODIC), C.BC(C.PERIODIC)]))
        Us.append(U[:, :, b * ni:(b + 1) * ni])
    mu = 1.5e-2 if c["grid"] == "viscous" else 0.0
    return blk, Us, C.qref_of(prim, 2), mu


def _grid_3d(c, seed):
    nb, ni, nj, nk = c["blocks"], c["ni"], c["nj"], c["nk"]
    N = nb * ni
    xs = [_unit(N, 3, 2), _unit(nj, 3, 1), _unit(nk, 3, 0)]
    rho_n = 1.0 + 2e-3 * _noise(seed, (nk, nj, N))
    if c["grid"] == "blobs":
        prim = C.inlet_freestream(2.0)
        r = np.random.default_rng(seed)
        rho = torch.ones((nk, nj, N), device=DEV, dtype=F64)
        for centre in r.uniform(0.0, 1.0, size=(16, 3)):
            t = 0.05
            for d in range(3):
                x = xs[d] - float(centre[d])
                x = x - torch.round(x) if d else x
                t = t * torch.exp(-x * x / (2.0 * 0.06 ** 2))
            rho = rho + t
        w = _waves(seed, 1, 3)
        U = _conserved(prim[0] * rho * rho_n, [torch.full_like(rho, prim[1]), torch.zeros_like(rho),
                                               torch.zeros_like(rho)],
                       prim[4] * (1.0 + 0.02 * w(0, xs)))
        h = (1.0 / N, 1.0 / nj, 1.0 / nk)
        bcs = [C.BC(C.INFLOW, prim=prim), C.BC(C.EXTRAP)] + [C.BC(C.PERIODIC) for _ in range(4)]
        return [C.Block(N, nj, nk, None, None, (0.0, 0.0, 0.0), h, bcs)], [U], C.qref_of(prim, 3), 0.0
    prim = (1.0, 0.6, 0.3, 0.0, 1.0 / G)
    w = _waves(seed, 5, 3)
    rho = (1.0 + 0.08 * w(0, xs)) * rho_n
    vel = [prim[1 + a] + 0.08 * w(1 + a, xs) for a in range(3)]
    U = _conserved(rho, vel, prim[4] * (1.0 + 0.08 * w(4, xs)))
    x, y, z = C.curv3d_nodes(N, nj, nk, amp=0.04, walls_k=c["walls"])
    kbc = C.SLIPWALL if c["walls"] else C.PERIODIC
    blk, Us = [], []
    for b in range(nb):
        lo = C.BC(C.BLOCK, (b - 1) % nb, C.IMAX) if nb > 1 else C.BC(C.PERIODIC)
        hi = C.BC(C.BLOCK, (b + 1) % nb, C.IMIN) if nb > 1 else C.BC(C.PERIODIC)
        s = (slice(None), slice(None), slice(b * ni, (b + 1) * ni + 1))
        blk.append(C.Block(ni, nj, nk, x[s].copy(), y[s].copy(), (0.0, 0.0, 0.0), (1.0, 1.0, 1.0),
                           [lo, hi, C.BC(C.PERIODIC), C.BC(C.PERIODIC), C.BC(kbc), C.BC(kbc)], z[s].copy()))
        Us.append(U[:, :, :, b * ni:(b + 1) * ni])
    return blk, Us, C.qref_of(prim, 3), 0.0


def _problem(c, seed):
    """The library's case object, with the state and source of each block as
    torch tensors (var, [k,] j, i)."""
    ndim = 3 if c["grid"] in ("blobs", "curved") else 2
    blk, U, qref, mu = _grid_3d(c, seed) if ndim == 3 else _grid_2d(c, seed)
    prm = C.Params(precision=C.FP32_FLUX if c["fp32"] else C.FP64, limiter=c["limiter"], qref=qref,
                   rk=c["rk"], mu=mu)
    src = None
    if c["source"]:
        # a smooth forcing: a tenth of the state's magnitude per flow-through
        w = _waves(seed + 1000, ndim + 2, ndim)
        tau = 0.1 * qref[1] / qref[0]
        src = []
        for u in U:
            xs = [_unit(n, ndim, ndim - 1 - d) for d, n in enumerate(reversed(u.shape[1:]))]
            src.append(torch.stack([tau * qref[v] * w(v, xs).expand(u.shape[1:])
                                    for v in range(ndim + 2)]))
    case = C.Case(c["grid"], ndim, blk, [], prm,
                  source=None if src is None else [s.reshape(s.shape[0], -1).cpu().numpy() for s in src])
    return case, U, src


def _flat(parts):
    return torch.cat([p.reshape(-1) for p in parts])


def _requests(c, seed):
    """The uneven grids of a served batch (sizes from the case alone, so that
    every seed has the same work): fractions of the largest, ragged."""
    out = []
    for r in range(c["blocks"]):
        f, g = 1.0 / (1 + r % 4), 1.0 / (1 + (r // 2) % 3)
        ni, nj = max(64, int(c["ni"] * f) - r), max(40, int(c["nj"] * g) - 3 * r)
        nb = 1 + r % 3
        out.append((dict(c, op="step", blocks=nb, ni=max(24, ni // nb), nj=nj), seed * 31 + r))
    return out


def prepare(case, seed):
    c = case
    if c["op"] == "serve":
        probs, cells = [], 0
        for q, s in _requests(c, seed):
            p, U, _ = _problem(q, s)
            p.U0 = [u.cpu().numpy() for u in U]
            probs.append(p)
            cells += p.ncells
        srv = fv.Server((256 << 20) + 160 * cells, max_instances=16, precision=probs[0].params.precision)
        return dict(c=c, probs=probs, srv=srv)
    p, U, _ = _problem(c, seed)
    U0 = _flat(U)
    if c["op"] == "noalloc":
        return dict(c=c, p=p, U0=U0)
    g = fv.Grid(p)
    out = torch.empty_like(U0)
    if c["op"] == "residual":
        g.set_state(U0)
    return dict(c=c, p=p, g=g, U0=U0, out=out)


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(state):
    c = state["c"]
    if c["op"] == "serve":
        srv = state["srv"]
        tickets = [srv.submit(p, drop_tol=0.0, max_steps=c["steps"]) for p in state["probs"]]
        done = {}
        while len(done) < len(tickets):
            for t in tickets:
                if t not in done:
                    r = srv.poll(t)
                    if r is not None:
                        done[t] = r
            if len(done) < len(tickets):
                time.sleep(2e-4)
        return [{"U": done[t][1], "steps": done[t][2]["steps"], "t": done[t][2]["t"],
                 "norms": done[t][2]["norms"]} for t in tickets]
    if c["op"] == "noalloc":
        U = state["U0"].clone()
        info = fv.step_noalloc(state["p"], U, nsteps=c["steps"])
        return {"U": U, "steps": info["steps"], "t": info["t"], "norms": info["norms"]}
    g = state["g"]
    if c["op"] == "residual":
        R, norms = g.residual(out=state["out"])
        return {"R": R, "norms": norms}
    g.set_state(state["U0"])
    info = g.step(nsteps=c["steps"])
    U = g.get_state(state["out"])
    return {"U": U, "steps": info["steps"], "t": info["t"], "norms": info["norms"]}


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _cells(c):
    return c["blocks"] * c["ni"] * c["nj"] * c["nk"]


def work(case):
    """Per stage: the stage's input state, U^n where the stage is not the
    first, the node coordinates (about one node per cell) and the source read
    once, the new state written once.  Operations per cell and stage counted
    from the formulas: reconstruction, one flux per face and direction,
    divergence, update."""
    c = case
    if c["op"] == "serve":
        w = [work(dict(q, op="step")) for q, _ in _requests(c, 0)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    nd = 3 if c["grid"] in ("blobs", "curved") else 2
    nv = nd + 2
    curved = c["grid"] not in ("vortex", "blobs")
    fixed = (8 * nd if curved else 0) + (8 * nv if c["source"] else 0)
    flops = 605 if nd == 3 else 393
    flops += (158 if nd == 3 else 0) if curved else 0
    flops += 120 if c["grid"] == "viscous" else 0
    if c["op"] == "residual":
        return {"bytes": _cells(c) * (16 * nv + fixed), "flops": _cells(c) * flops}
    stages = c["rk"]
    per_step = 8 * nv * (3 * stages - 1) + stages * fixed
    return {"bytes": _cells(c) * c["steps"] * per_step, "flops": _cells(c) * c["steps"] * stages * flops}


# --------------------------------------------------------------------------
# the method in plain torch, 64 bits: ghost-padded blocks, MUSCL and Roe's
# flux as a sum over waves, the viscous flux by the diamond gradient, explicit
# stages
# --------------------------------------------------------------------------
def _take(A, d, i):
    """Slice of index i along direction d (0: i, 1: j, 2: k), kept as an axis."""
    n = A.shape[-1 - d]
    return A.narrow(A.dim() - 1 - d, i % n, 1)


def _mirror(q, S):
    m = q[1:-1]
    f = 2.0 * (m * S).sum(0) / (S * S).sum(0)
    return torch.cat([q[:1], m - f * S, q[-1:]])


def _noslip(q):
    return torch.cat([q[:1], -q[1:-1], q[-1:]])


class _Exact:
    def __init__(self, case, src):
        self.p, self.nd, self.blocks, self.src = case.params, case.ndim, case.blocks, src
        self.visc = case.params.mu > 0.0
        self.S, self.vol, self.xy = [], [], []
        for B in case.blocks:
            S, vol, xy = self._metrics(B)
            self.S.append(S)
            self.vol.append(vol)
            self.xy.append(xy)

    def _metrics(self, B):
        nd, dims = self.nd, [B.ni, B.nj, B.nk][:self.nd]
        if B.x is None:
            S = []
            for d in range(nd):
                shape = [n + (1 if a == d else 0) for a, n in enumerate(dims)][::-1]
                s = torch.zeros([nd] + shape, device=DEV, dtype=F64)
                s[d] = math.prod(B.h[:nd]) / B.h[d]
                S.append(s)
            return S, torch.tensor(math.prod(B.h[:nd]), device=DEV, dtype=F64), None
        xyz = [torch.as_tensor(a, device=DEV) for a in (B.x, B.y, B.z)[:nd]]
        X = torch.stack(xyz)
        if nd == 2:
            ei, ej = X[:, 1:, :] - X[:, :-1, :], X[:, :, 1:] - X[:, :, :-1]
            S = [torch.stack([ei[1], -ei[0]]), torch.stack([-ej[1], ej[0]])]
            a, b, c, d = X[:, :-1, :-1], X[:, :-1, 1:], X[:, 1:, :-1], X[:, 1:, 1:]
            vol = 0.5 * ((d[0] - a[0]) * (c[1] - b[1]) - (c[0] - b[0]) * (d[1] - a[1]))
            return S, vol, X
        S, vol = [], 0.0
        for d in range(3):
            t1, t2 = [a for a in range(3) if a != d]

            def corner(o1, o2):
                A = X
                for t, o in ((t1, o1), (t2, o2)):
                    A = A.narrow(3 - t, o, A.shape[3 - t] - 1)
                return A
            p0, p1, p2, p3 = corner(0, 0), corner(1, 0), corner(1, 1), corner(0, 1)
            s = 0.5 * torch.cross(p2 - p0, p3 - p1, dim=0) * (-1.0 if d == 1 else 1.0)
            cs = (0.25 * (p0 + p1 + p2 + p3) * s).sum(0)
            n = cs.shape[-1 - d]
            vol = vol + cs.narrow(2 - d, 1, n - 1) - cs.narrow(2 - d, 0, n - 1)
            S.append(s)
        return S, vol / 3.0, None

    def _inflow(self, bc):
        rho, u, v, w, p = bc.prim
        vel = (u, v, w)[:self.nd]
        return torch.tensor([rho] + [rho * a for a in vel] + [p / (G - 1.0) + 0.5 * rho * sum(a * a for a in vel)],
                            device=DEV, dtype=F64)

    def pad(self, U):
        """Two ghost layers on every side, the last direction first, so that a
        corner follows the i-face rule and then the j-face rule."""
        for d in range(self.nd - 1, -1, -1):
            new = []
            for b, B in enumerate(self.blocks):
                sides = []
                for side in (0, 1):
                    bc = B.bc[2 * d + side]
                    layers = []
                    for g in (1, 2):
                        k = bc.kind
                        if k in (C.PERIODIC, C.BLOCK):
                            q = _take(U[bc.nbr_block if k == C.BLOCK else b], d, -g if side == 0 else g - 1)
                        elif k == C.EXTRAP:
                            q = _take(U[b], d, 0 if side == 0 else -1)
                        elif k == C.INFLOW:
                            q = _take(U[b], d, 0)
                            q = self._inflow(bc).reshape([-1] + [1] * self.nd).expand_as(q)
                        else:
                            q = _take(U[b], d, g - 1 if side == 0 else -g)
                            if k == C.NOSLIP:
                                q = _noslip(q)
                            else:
                                q = _mirror(q, self._wall(b, d, side, q))
                        layers.append(q)
                    sides.append(layers)
                new.append(torch.cat([sides[0][1], sides[0][0], U[b], sides[1][0], sides[1][1]],
                                     dim=U[b].dim() - 1 - d))
            U = new
        return U

    def _wall(self, b, d, side, q):
        """The wall faces' area vectors; where q is padded in the later
        directions already, those of the nearest faces (corners, not read by
        the inviscid flux)."""
        S = _take(self.S[b][d], d, 0 if side == 0 else -1)
        for a in range(self.nd):
            n = q.shape[-1 - a]
            if S.shape[-1 - a] != n:
                i = torch.arange(n, device=DEV) - (n - S.shape[-1 - a]) // 2
                S = S.index_select(S.dim() - 1 - a, i.clamp(0, S.shape[-1 - a] - 1))
        return S

    def _sides(self, P, d):
        """The left and right states of every face normal to d, from the
        padded block P with the other directions' ghosts cut off."""
        for a in range(self.nd):
            if a != d:
                P = P.narrow(P.dim() - 1 - a, 2, P.shape[-1 - a] - 4)
        ax = P.dim() - 1 - d
        n = P.shape[ax]
        dq = P.narrow(ax, 1, n - 1) - P.narrow(ax, 0, n - 1)
        dm, dp = dq.narrow(ax, 0, n - 2), dq.narrow(ax, 1, n - 2)  # of cells 1 .. n-2
        e, k = self.p.eps, self.p.kappa
        if self.p.limiter == C.MINMOD:
            s = 0.25 * e * (torch.sign(dm) + torch.sign(dp)) * torch.minimum(dm.abs(), dp.abs())
            ep = em = s
        else:
            ep = 0.25 * e * ((1.0 - k) * dm + (1.0 + k) * dp)
            em = 0.25 * e * ((1.0 - k) * dp + (1.0 + k) * dm)
        Q = P.narrow(ax, 1, n - 2)
        return (Q + ep).narrow(ax, 0, n - 3), (Q - em).narrow(ax, 1, n - 3)

    def _prim(self, q):
        vel = q[1:-1] / q[0]
        p = (G - 1.0) * (q[-1] - 0.5 * q[0] * (vel * vel).sum(0))
        return q[0], vel, p

    def _roe(self, L, R, S):
        A = torch.sqrt((S * S).sum(0))
        n = S / A
        (rL, vL, pL), (rR, vR, pR) = self._prim(L), self._prim(R)
        HL, HR = (L[-1] + pL) / rL, (R[-1] + pR) / rR
        wl, wr = torch.sqrt(rL), torch.sqrt(rR)
        r = wl * wr
        v = (wl * vL + wr * vR) / (wl + wr)
        H = (wl * HL + wr * HR) / (wl + wr)
        c = torch.sqrt((G - 1.0) * (H - 0.5 * (v * v).sum(0)))
        un, uL, uR = (v * n).sum(0), (vL * n).sum(0), (vR * n).sum(0)
        one, zero = torch.ones_like(r), torch.zeros_like(r)

        def lam(x):
            a, dl = x.abs(), self.p.entropy_fix * c
            return torch.where(a < dl, 0.5 * (a * a / dl + dl), a) if self.p.entropy_fix > 0.0 else a

        def vec(first, mom, last):
            return torch.cat([first[None], mom, last[None]])
        dr, dv, dp, du = rR - rL, vR - vL, pR - pL, uR - uL
        a1 = (dp - r * c * du) / (2.0 * c * c)
        a3 = (dp + r * c * du) / (2.0 * c * c)
        D = lam(un - c) * a1 * vec(one, v - c * n, H - c * un)
        D = D + lam(un + c) * a3 * vec(one, v + c * n, H + c * un)
        D = D + un.abs() * (dr - dp / (c * c)) * vec(one, v, 0.5 * (v * v).sum(0))
        D = D + un.abs() * r * vec(zero, dv - du * n, (v * dv).sum(0) - un * du)
        FL = vec(rL * uL, L[1:-1] * uL + pL * n, (L[-1] + pL) * uL)
        FR = vec(rR * uR, R[1:-1] * uR + pR * n, (R[-1] + pR) * uR)
        return 0.5 * A * (FL + FR - D)

    def _centres(self):
        """Cell centres with one ghost ring (corners unused)."""
        inner = [0.25 * (X[:, :-1, :-1] + X[:, :-1, 1:] + X[:, 1:, :-1] + X[:, 1:, 1:]) for X in self.xy]
        out = []
        for b, B in enumerate(self.blocks):
            P = torch.zeros((2, B.nj + 2, B.ni + 2), device=DEV, dtype=F64)
            P[:, 1:-1, 1:-1] = inner[b]
            for d in (0, 1):
                for side in (0, 1):
                    bc = B.bc[2 * d + side]
                    if bc.kind == C.BLOCK:
                        g = _take(inner[bc.nbr_block], d, -1 if side == 0 else 0)
                    else:
                        X = _take(self.xy[b], d, 0 if side == 0 else -1)
                        t = X.dim() - 2 + d  # the axis along the face
                        m = 0.5 * (X.narrow(t, 0, X.shape[t] - 1) + X.narrow(t, 1, X.shape[t] - 1))
                        g = 2.0 * m - _take(inner[b], d, 0 if side == 0 else -1)
                    if d == 0:
                        P[:, 1:-1, 0 if side == 0 else -1] = g[:, :, 0]
                    else:
                        P[:, 0 if side == 0 else -1, 1:-1] = g[:, 0, :]
            out.append(P)
        return out

    def _viscous(self, b, P, d):
        """F_nu . S of the faces normal to d (2D)."""
        rho, vel, p = self._prim(P[:, 1:-1, 1:-1])  # the cells and one ring
        w = torch.cat([vel, (p / rho)[None]])
        node = 0.25 * (w[:, :-1, :-1] + w[:, :-1, 1:] + w[:, 1:, :-1] + w[:, 1:, 1:])
        S, ctr = self.S[b][d], self.ctr[b]
        if d == 0:
            wL, wR = w[:, 1:-1, :-1], w[:, 1:-1, 1:]
            t = node[:, 1:, :] - node[:, :-1, :]
            dx = ctr[:, 1:-1, 1:] - ctr[:, 1:-1, :-1]
        else:
            wL, wR = w[:, :-1, 1:-1], w[:, 1:, 1:-1]
            t = node[:, :, :-1] - node[:, :, 1:]
            dx = ctr[:, 1:, 1:-1] - ctr[:, :-1, 1:-1]
        a, D = wR - wL, (dx * S).sum(0)
        gx, gy = (a * S[0] - t * dx[1]) / D, (a * S[1] + t * dx[0]) / D
        mu, div = self.p.mu, gx[0] + gy[1]
        txx, tyy = mu * (2.0 * gx[0] - 2.0 / 3.0 * div), mu * (2.0 * gy[1] - 2.0 / 3.0 * div)
        txy = mu * (gy[0] + gx[1])
        kq = mu / self.p.prandtl * G / (G - 1.0)
        u, v = 0.5 * (wL[0] + wR[0]), 0.5 * (wL[1] + wR[1])
        hx, hy = u * txx + v * txy + kq * gx[2], u * txy + v * tyy + kq * gy[2]
        return torch.stack([torch.zeros_like(u), txx * S[0] + txy * S[1], txy * S[0] + tyy * S[1],
                            hx * S[0] + hy * S[1]])

    def residual(self, U):
        out = []
        for b, P in enumerate(self.pad(U)):
            R = 0.0
            for d in range(self.nd):
                L, Rt = self._sides(P, d)
                F = self._roe(L, Rt, self.S[b][d])
                if self.visc:
                    F = F - self._viscous(b, P, d)
                ax = F.dim() - 1 - d
                R = R + F.narrow(ax, 1, F.shape[ax] - 1) - F.narrow(ax, 0, F.shape[ax] - 1)
            if self.src is not None:
                R = R - self.vol[b] * self.src[b]
            out.append(R)
        return out

    def dt(self, U):
        m = math.inf
        for b, u in enumerate(U):
            rho, vel, p = self._prim(u)
            c = torch.sqrt(G * p / rho)
            lam, ss = 0.0, 0.0
            for d in range(self.nd):
                S = self.S[b][d]
                ax = S.dim() - 1 - d
                Sb = 0.5 * (S.narrow(ax, 0, S.shape[ax] - 1) + S.narrow(ax, 1, S.shape[ax] - 1))
                s2 = (Sb * Sb).sum(0)
                lam = lam + (vel * Sb).sum(0).abs() + c * torch.sqrt(s2)
                ss = ss + s2
            if self.visc:
                lam = lam + 2.0 * max(4.0 / 3.0, G / self.p.prandtl) * (self.p.mu / rho) * ss / self.vol[b]
            m = min(m, float((self.vol[b] / lam).min()))
        return self.p.cfl * m

    def norms(self, R):
        n = sum(r[0].numel() for r in R)
        s = sum(((r / v) ** 2).reshape(r.shape[0], -1).sum(1) for r, v in zip(R, self.vol))
        return np.array([math.sqrt(float(x) / n) for x in s] + [0.0] * (5 - len(s)))

    def advance(self, U, steps):
        t, norms = 0.0, None
        for _ in range(steps):
            dt = self.dt(U)

            def stage(V, base, f):
                R = self.residual(V)
                return R, [u - f * dt / v * r for u, v, r in zip(base, self.vol, R)]
            if self.p.rk == 3:
                R, A = stage(U, U, 1.0)
                _, B = stage(A, A, 1.0)
                B = [0.75 * u + 0.25 * x for u, x in zip(U, B)]
                _, D = stage(B, B, 1.0)
                new = [u / 3.0 + 2.0 / 3.0 * x for u, x in zip(U, D)]
            else:
                new = U
                for k, f in enumerate((0.5, 1.0) if self.p.rk == 2 else (0.25, 1.0 / 3.0, 0.5, 1.0)):
                    r, new = stage(new, U, f)
                    R = r if k == 0 else R
            norms = self.norms(R)
            U, t = new, t + dt
        return U, t, norms


def exact(case, seed):
    c = case
    if c["op"] == "serve":
        return [exact(q, s) for q, s in _requests(c, seed)]
    p, U, src = _problem(c, seed)
    E = _Exact(p, src)
    if E.visc:
        E.ctr = E._centres()
    if c["op"] == "residual":
        R = E.residual(U)
        return {"R": _flat(R), "norms": E.norms(R)}
    V, t, norms = E.advance(U, c["steps"])
    return {"U": _flat(V), "steps": c["steps"], "t": t, "norms": norms}
