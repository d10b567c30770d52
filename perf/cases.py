"""Timed workloads of the lattice-Boltzmann library, run through its public entry points.

A case is one simulation as a user's program runs it: a lattice made once (geometry, fluid,
options), then passes of a number of time steps after which the macroscopic fields are read
into device arrays; or one evaluation of the channel objective with its gradients.

    listed()            the workloads that stand for the range
    draw(rng)           one more workload of the same ranges
    prepare(case, seed) lattice, initial state and output arrays of one workload
    run(state)          one pass: steps and fields (or objective and gradients)
    work(case)          bytes and operations one pass cannot do without
    exact(case, seed)   the same outputs in 64-bit arithmetic with plain torch operations
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.utils.checkpoint

import paper_2108_13241_amd as lbm

# ------------------------------------------------------------------ workloads --


def listed():
    return [
        # A small channel driven by a body force, double precision: the launch-bound end,
        # where a step is a few microseconds of GPU work (256 x 64, the smallest
        # benchmark configuration).
        _case2("channel_256x64_f64", 256, 64, "f64", "channel", steps=200, tau=0.8),
        # A lid-driven cavity of odd size with a moving lid (open-boundary nodes), walls
        # on three sides, and the two-relaxation-time collision: validation runs.
        _case2("cavity_257_f64_trt", 257, 257, "f64", "cavity", steps=100, tau=0.6,
               collision="trt"),
        # A mid-size flow around random discs, ragged row length, an odd number of steps,
        # multiple-relaxation-time collision, single precision.
        _case2("discs_1500x1001_f32_mrt", 1500, 1001, "f32", "discs", steps=51, tau=0.7,
               phi=0.9, collision="mrt"),
        # The pressure-driven open channel at 4096 x 512, single precision.
        _case2("chan_p_4096x512_f32", 4096, 512, "f32", "open", steps=100, tau=1.25),
        # Taylor-Green vortex 2048^2 with 16-bit storage (the reduced-precision study).
        _case2("tgv_2048_f16", 2048, 2048, "f16s", "vortex", steps=50, tau=0.8),
        # The dense headline: Taylor-Green vortex 4096^2, double precision, two lattices.
        _case2("tgv_4096_f64", 4096, 4096, "f64", "vortex", steps=50, tau=0.8),
        # The same mesh in place (half the memory), single precision, odd step count.
        _case2("tgv_4096_f32_aa", 4096, 4096, "f32", "vortex", steps=51, tau=0.8,
               layout="dense_aa"),
        # Porous medium of random discs at fluid fraction 0.5, compacted 16 x 16 tiles.
        _case2("discs_4096_f32_tiled", 4096, 4096, "f32", "discs", steps=30, tau=0.8,
               phi=0.5, layout="tiled16"),
        # The same medium on the list of fluid nodes, double precision.
        _case2("discs_4096_f64_list", 4096, 4096, "f64", "discs", steps=30, tau=0.8,
               phi=0.5, layout="indirect"),
        # Objective of a 1024 x 256 channel with a drag field after 500 steps, and its
        # gradients (forward and backward through checkpoints): one optimisation step.
        dict(name="objective_1024x256_f32", kind="objective", nx=1024, ny=256, dtype="f32",
             steps=500, tau=0.8),
        # Three-dimensional Taylor-Green vortex 256^3, single precision, two lattices.
        _case3("d3q19_vortex_256_f32", 256, 256, 256, "f32", "vortex", steps=20),
        # Flow through a packing of spheres at fluid fraction 0.4 on the list of fluid
        # nodes, double precision.
        _case3("d3q19_spheres_256_f64_list", 256, 256, 256, "f64", "spheres", steps=20,
               phi=0.4, layout="indirect"),
    ]


def _case2(name, nx, ny, dtype, flow, *, steps, tau, layout="dense_ab", phi=1.0,
           collision="bgk"):
    c = dict(kind="d2q9", nx=nx, ny=ny, dtype=dtype, layout=layout, flow=flow, phi=phi,
             collision=collision, steps=steps, tau=tau)
    return dict(name=name, **c) if name else c


def _case3(name, nx, ny, nz, dtype, flow, *, steps, tau=0.8, layout="dense_ab", phi=1.0,
           collision="bgk"):
    c = dict(kind="d3q19", nx=nx, ny=ny, nz=nz, dtype=dtype, layout=layout, flow=flow, phi=phi,
             collision=collision, steps=steps, tau=tau)
    return dict(name=name, **c) if name else c


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more workload: sizes spread over their logarithm, odd ones among them; layouts,
    storage types, collisions and flows as users combine them."""
    kind = rng.choices(["d2q9", "d3q19", "objective"], [7, 2, 1])[0]
    tau = round(rng.uniform(0.55, 1.2), 3)
    collision = rng.choice(["bgk", "bgk", "trt", "mrt"])
    if kind == "objective":
        return dict(kind=kind, nx=_log_uniform(rng, 200, 1100), ny=_log_uniform(rng, 60, 300),
                    dtype=rng.choice(["f32", "f32", "f64"]), steps=rng.randint(60, 300),
                    tau=round(rng.uniform(0.6, 1.0), 3))
    if kind == "d3q19":
        layout = rng.choice(["dense_ab", "dense_ab", "dense_aa", "indirect", "tiled16"])
        n = [_log_uniform(rng, 24, 250) for _ in range(3)]
        if layout == "tiled16":
            n = [4 * max(1, v // 4) for v in n]
        flow = "spheres" if layout in ("indirect", "tiled16") else rng.choice(["vortex", "spheres"])
        phi = 1.0 if flow == "vortex" else round(rng.uniform(0.3, 0.8), 2)
        return _case3(None, *n, rng.choice(["f64", "f32", "f32", "f16s"]), flow,
                      steps=rng.randint(5, 16), tau=tau, layout=layout, phi=phi,
                      collision=collision)
    layout = rng.choice(["dense_ab", "dense_ab", "dense_ab", "dense_aa", "tiled16", "indirect"])
    nx, ny = _log_uniform(rng, 60, 4000), _log_uniform(rng, 40, 4000)
    if layout == "tiled16":
        nx, ny = 16 * max(2, nx // 16), 16 * max(2, ny // 16)
    if layout in ("tiled16", "indirect"):
        flow = rng.choice(["discs", "discs", "channel"])
    else:
        flow = rng.choice(["vortex", "vortex", "channel", "open", "cavity", "discs"])
    phi = round(rng.uniform(0.2, 0.95), 2) if flow == "discs" else 1.0
    most = max(4, min(100, int(4e8 / (nx * ny))))
    return _case2(None, nx, ny, rng.choice(["f64", "f64", "f32", "f32", "f16s", "bf16s"]), flow,
                  steps=rng.randint(max(2, most // 3), most), tau=tau, layout=layout, phi=phi,
                  collision=collision)


# -------------------------------------------------------------------- inputs --

_FORCE2 = (1e-6, 2e-7)
_FORCE3 = (1e-6, 5e-7, -2e-7)


def _forced(case):
    return case["flow"] in ("channel", "discs", "spheres")


def _mask2(case, seed):
    """uint8 [ny, nx]: 1 = solid."""
    nx, ny, flow = case["nx"], case["ny"], case["flow"]
    m = np.zeros((ny, nx), dtype=np.uint8)
    if flow in ("channel", "discs", "open"):
        m[0] = m[-1] = 1
    elif flow == "cavity":
        m[0] = 1
        m[:, 0] = m[:, -1] = 1
    if flow == "discs":
        rng = np.random.default_rng(seed)
        small = min(nx, ny)
        rmin, rmax = max(2, min(8, small // 16)), max(4, min(64, small // 6))
        while m.size - np.count_nonzero(m) > case["phi"] * m.size:
            for _ in range(16):
                r = int(rng.integers(rmin, rmax + 1))
                cx, cy = int(rng.integers(0, nx)), int(rng.integers(1, ny - 1))
                y0, y1 = max(0, cy - r), min(ny, cy + r + 1)
                x0, x1 = max(0, cx - r), min(nx, cx + r + 1)
                dy = np.arange(y0, y1)[:, None] - cy
                dx = np.arange(x0, x1)[None, :] - cx
                m[y0:y1, x0:x1] |= (dx * dx + dy * dy <= r * r).astype(np.uint8)
    return m


def _mask3(case, seed):
    """uint8 [nz, ny, nx]: 1 = solid."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    m = np.zeros((nz, ny, nx), dtype=np.uint8)
    if case["flow"] == "spheres":
        m[0] = m[-1] = 1
        rng = np.random.default_rng(seed)
        small = min(nx, ny, nz)
        rmin, rmax = max(2, min(8, small // 10)), max(3, min(24, small // 4))
        while m.size - np.count_nonzero(m) > case["phi"] * m.size:
            for _ in range(4):
                r = int(rng.integers(rmin, rmax + 1))
                c = [int(rng.integers(0, n)) for n in (nz, ny, nx)]
                lo = [max(0, a - r) for a in c]
                hi = [min(n, a + r + 1) for a, n in zip(c, (nz, ny, nx))]
                d = [np.arange(a, b) - k for a, b, k in zip(lo, hi, c)]
                d2 = (d[0][:, None, None] ** 2 + d[1][None, :, None] ** 2
                      + d[2][None, None, :] ** 2)
                m[lo[0]:hi[0], lo[1]:hi[1], lo[2]:hi[2]] |= (d2 <= r * r).astype(np.uint8)
    return m


def _boundaries(case):
    """Open-boundary codes and values of the open channel and the cavity, or None."""
    nx, ny = case["nx"], case["ny"]
    bc = np.zeros((ny, nx), dtype=np.uint8)
    val = np.zeros((2, ny, nx))
    if case["flow"] == "open":  # pressure inlet at x = 0, pressure outlet at x = nx - 1
        bc[1:-1, 0], bc[1:-1, -1] = 5, 6
        val[0, 1:-1, 0], val[0, 1:-1, -1] = 1.016, 1.0
    elif case["flow"] == "cavity":  # lid at the top row, moving along +x
        bc[-1, 1:-1] = 4
        val[0, -1, 1:-1] = 0.1
    else:
        return None
    return bc, val


def _fields(shape, seed, amp):
    """Smooth random initial fields on the GPU, float64: density near 1 and one velocity
    component per axis, sums of a few seeded Fourier modes with long wavelengths."""
    rng = np.random.default_rng(seed + 1000)
    out = []
    for k in range(1 + len(shape)):
        f = torch.zeros(shape, dtype=torch.float64, device="cuda")
        for _ in range(3):
            term = None
            for ax, n in enumerate(shape):
                x = torch.arange(n, dtype=torch.float64, device="cuda")
                m, ph = int(rng.integers(1, 4)), float(rng.uniform(0, 2 * math.pi))
                w = torch.sin(2 * math.pi * m / n * x + ph)
                w = w.reshape([-1 if a == ax else 1 for a in range(len(shape))])
                term = w if term is None else term * w
            f += float(rng.uniform(0.3, 1.0)) * term
        f *= amp / 3.0
        out.append(1.0 + 0.1 * f if k == 0 else f)
    return out


def _initial(case, seed, mask):
    """(rho, velocity components) as device float64 arrays; zero velocity at solid nodes."""
    if case["kind"] == "objective":
        return None
    f = _fields(mask.shape, seed, 0.02 if case["flow"] == "cavity" else 0.05)
    fluid = torch.from_numpy(mask == 0).cuda()
    return [f[0]] + [u * fluid for u in f[1:]]


def _drag(case, seed):
    """Smooth drag coefficients in [0, 1] (float32 [ny, nx], GPU)."""
    f = _fields((case["ny"], case["nx"]), seed, 3.0)[1]
    return (0.5 * (1.0 + torch.tanh(2.0 * f))).float()


_MRT2 = (1.64, 1.54, 1.9)
_MRT3 = (1.19, 1.4, 1.2, 1.4, 1.98)
_MAGIC = 3.0 / 16.0


def prepare(case, seed):
    if case["kind"] == "objective":
        m = np.zeros((case["ny"], case["nx"]), dtype=np.uint8)
        m[0] = m[-1] = 1
        alpha = _drag(case, seed).requires_grad_(True)
        g = torch.tensor([1e-5, 1e-6], dtype=torch.float64, device="cuda", requires_grad=True)
        spec = dict(mask=m, tau=case["tau"], steps=case["steps"], x_out=case["nx"] - 1,
                    dtype=case["dtype"])
        return dict(kind="objective", alpha=alpha, g=g, spec=spec)
    three = case["kind"] == "d3q19"
    mask = (_mask3 if three else _mask2)(case, seed)
    if three:
        lat = lbm.Lattice3D(mask, case["tau"], force=_FORCE3 if _forced(case) else (0., 0., 0.),
                            dtype=case["dtype"], layout=case["layout"])
    else:
        lat = lbm.Lattice(mask, case["tau"], force=_FORCE2 if _forced(case) else (0., 0.),
                          dtype=case["dtype"], layout=case["layout"])
        if (b := _boundaries(case)) is not None:
            lat.set_boundaries(*b)
    if case["collision"] == "trt":
        lat.set_trt(_MAGIC)
    elif case["collision"] == "mrt":
        lat.set_mrt(_MRT3 if three else _MRT2)
    init = _initial(case, seed, mask)
    lat.init_equilibrium(*[f.cpu().numpy() for f in init])
    del init
    out = [torch.empty(mask.shape, dtype=torch.float64, device="cuda")
           for _ in range(1 + mask.ndim)]
    return dict(kind=case["kind"], lat=lat, steps=case["steps"], out=out)


def run(state):
    if state["kind"] == "objective":
        alpha, g = state["alpha"], state["g"]
        J = lbm.ChannelObjective.apply(alpha, g, state["spec"])
        ga, gg = torch.autograd.grad(J, (alpha, g))
        return {"J": J.detach(), "grad_alpha": ga, "grad_g": gg}
    lat = state["lat"]
    lat.step(state["steps"])
    lat.macroscopic_device(*state["out"])
    return {n: f for n, f in zip(("rho", "ux", "uy", "uz"), state["out"])}


def work(case):
    """State read once and written once, node types once, output fields once; the
    collisions of all steps (about 130 operations a node in D2Q9, 300 in D3Q19; the
    backward pass of the objective does about three times a forward step)."""
    s = {"f64": 8, "f32": 4}.get(case["dtype"], 2)
    n = case["nx"] * case["ny"] * case.get("nz", 1)
    if case["kind"] == "objective":
        # drag field in, its gradient out; forward, recomputation and reverse collisions
        return {"bytes": 8.0 * n, "flops": 130.0 * 5 * n * case["steps"]}
    q, ops, fields = (19, 300.0, 4) if case["kind"] == "d3q19" else (9, 130.0, 3)
    fluid = n * case["phi"]
    return {"bytes": 2.0 * q * s * fluid + n + 8.0 * fields * n,
            "flops": ops * fluid * case["steps"]}


# ------------------------------------------------------- 64-bit reference values --

_C2 = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
_W2 = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
_C3 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
       (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
       (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
_W3 = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12


def _dot(c, v):
    """c . v for a velocity of components -1, 0, 1 (None for the rest velocity)."""
    s = None
    for a, x in zip(c, v):
        if a:
            s = (x if a > 0 else -x) if s is None else (s + x if a > 0 else s - x)
    return s


def _relaxation_matrix(C, W, tau, collision):
    """A with f* = f - A (f - f^eq) + (1 - A / 2) S for the chosen collision."""
    q = len(C)
    om = 1.0 / tau
    if collision == "bgk":
        return om * np.eye(q)
    if collision == "trt":
        om_m = 1.0 / (0.5 + _MAGIC / (tau - 0.5))
        opp = [C.index(tuple(-a for a in c)) for c in C]
        P = np.zeros((q, q))
        P[np.arange(q), opp] = 1.0
        return om * 0.5 * (np.eye(q) + P) + om_m * 0.5 * (np.eye(q) - P)
    c = np.array(C, dtype=float)
    if q == 9:
        x, y = c.T
        r2 = x * x + y * y
        M = [np.ones(9), -4 + 3 * r2, 4 - 10.5 * r2 + 4.5 * r2 * r2, x, (-5 + 3 * r2) * x, y,
             (-5 + 3 * r2) * y, x * x - y * y, x * y]
        se, sp, sq = _MRT2
        s = [1.0, se, sp, 1.0, sq, 1.0, sq, om, om]
    else:
        x, y, z = c.T
        r2 = x * x + y * y + z * z
        xx = 3 * x * x - r2
        ww = y * y - z * z
        M = [np.ones(19), -30 + 19 * r2, (24 - 53 * r2 + 21 * r2 * r2) / 2,
             x, (5 * r2 - 9) * x, y, (5 * r2 - 9) * y, z, (5 * r2 - 9) * z,
             xx, (3 * r2 - 5) * xx, ww, (3 * r2 - 5) * ww, x * y, y * z, x * z,
             (y * y - z * z) * x, (z * z - x * x) * y, (x * x - y * y) * z]
        se, sp, sq, spi, sm = _MRT3
        s = [1.0, se, sp, 1.0, sq, 1.0, sq, 1.0, sq, om, spi, om, spi, om, om, om, sm, sm, sm]
    M = np.array(M)
    return np.linalg.inv(M) @ np.diag(s) @ M


def _moments(f, C, g, invD):
    rho = sum(f[1:], f[0])
    u = []
    for a in range(len(C[0])):
        m = sum(fi if c[a] > 0 else -fi for c, fi in zip(C, f) if c[a])
        v = m / rho + 0.5 * g[a]
        u.append(v if invD is None else v * invD)
    return rho, u


def _open(f, C, bc, val):
    """Rebuild of the populations entering across open boundaries (Zou and He)."""
    for code in range(1, 9):
        at = bc == code
        if not at.any():
            continue
        at = torch.from_numpy(at).cuda()
        n = [(1, 0), (-1, 0), (0, 1), (0, -1)][(code - 1) % 4]
        t = (-n[1], n[0])
        fl = [fi[at] for fi in f]
        dn = [c[0] * n[0] + c[1] * n[1] for c in C]
        dt = [c[0] * t[0] + c[1] * t[1] for c in C]
        S = sum(x for x, d in zip(fl, dn) if d == 0) + 2 * sum(x for x, d in zip(fl, dn) if d < 0)
        T = sum(s * x for x, d, s in zip(fl, dn, dt) if d == 0 and s)
        v = [torch.from_numpy(a).cuda()[at] for a in val]
        if code <= 4:
            un, ut = v[0] * n[0] + v[1] * n[1], v[0] * t[0] + v[1] * t[1]
            rho = S / (1 - un)
            run, rut = rho * un, rho * ut
        else:
            run, rut = v[0] - S, 0.0 * S
        for i, c in enumerate(C):
            if dn[i] > 0:
                o = fl[C.index((-c[0], -c[1]))]
                inc = 2 / 3 * run if dt[i] == 0 else run / 6 + dt[i] * 0.5 * (rut - T)
                f[i][at] = o + inc


class _Reference:
    """Collide and stream over full arrays, halfway bounce-back at solid nodes."""

    def __init__(self, mask, tau, g, collision, bc=None, alpha=None):
        three = mask.ndim == 3
        self.C, self.W = (_C3, _W3) if three else (_C2, _W2)
        self.opp = [self.C.index(tuple(-a for a in c)) for c in self.C]
        self.g, self.bc = g, bc
        self.A = _relaxation_matrix(self.C, self.W, tau, collision)
        self.plain = collision == "bgk"
        self.fluid = torch.from_numpy(mask == 0).cuda()
        self.dims = tuple(range(mask.ndim))[::-1]  # x is the last axis
        self.alpha = alpha
        self.invD = None if alpha is None else 1.0 / (1.0 + 0.5 * alpha)
        self.has_solid = bool(mask.any())
        if self.has_solid:
            self.from_solid = [~torch.roll(self.fluid, c, self.dims) for c in self.C]

    def equilibrium(self, i, rho, u, usq):
        cu = _dot(self.C[i], u)
        e = 1.0 - usq
        return self.W[i] * rho * (e if cu is None else e + 3.0 * cu + 4.5 * cu * cu)

    def init(self, rho, u):
        usq = 1.5 * sum(v * v for v in u)
        f = [self.equilibrium(i, rho, u, usq) for i in range(len(self.C))]
        if self.bc is not None:
            _open(f, self.C, *self.bc)
        return f

    def step(self, f):
        rho, u = _moments(f, self.C, self.g, self.invD)
        forced = self.alpha is not None or any(self.g)
        if forced:
            F = [rho * (a if self.alpha is None else a - self.alpha * v)
                 for a, v in zip(self.g, u)]
            uF = sum(a * b for a, b in zip(u, F))
        usq = 1.5 * sum(v * v for v in u)

        def neq(i):  # (f - f^eq, S) of direction i
            d = f[i] - self.equilibrium(i, rho, u, usq)
            if not forced:
                return d, None
            cF = _dot(self.C[i], F)
            if cF is None:
                return d, self.W[i] * -3.0 * uF
            return d, self.W[i] * (3.0 * (cF - uF) + 9.0 * _dot(self.C[i], u) * cF)

        q = len(self.C)
        post = []
        if self.plain:
            om = float(self.A[0, 0])
            for i in range(q):
                d, s = neq(i)
                p = f[i] - om * d
                post.append(p if s is None else p + (1.0 - 0.5 * om) * s)
        else:
            all_neq = [neq(i) for i in range(q)]
            shape = f[0].shape
            A = torch.from_numpy(self.A).cuda()
            D = torch.stack([d for d, _ in all_neq]).reshape(q, -1)
            relax = A @ D
            if forced:
                S = torch.stack([s for _, s in all_neq]).reshape(q, -1)
                relax = relax - S + 0.5 * (A @ S)
            post = [f[i] - relax[i].reshape(shape) for i in range(q)]
        new = []
        for i in range(q):
            v = torch.roll(post[i], self.C[i], self.dims) if i else post[i]
            if self.has_solid and i:
                v = torch.where(self.from_solid[i], post[self.opp[i]], v)
            new.append(v)
        if self.bc is not None:
            _open(new, self.C, *self.bc)
        return new


def _exact_objective(case, seed):
    m = np.zeros((case["ny"], case["nx"]), dtype=np.uint8)
    m[0] = m[-1] = 1
    alpha = _drag(case, seed).double().requires_grad_(True)
    g = torch.tensor([1e-5, 1e-6], dtype=torch.float64, device="cuda", requires_grad=True)
    fluid = torch.from_numpy(m == 0).cuda()

    def steps(alpha, g, k, *f):
        # at solid nodes the populations stay at rest, so their values are finite
        ref = _Reference(m, case["tau"], (0.0, 0.0), "bgk", None, alpha)
        ref.g = (g[0], g[1])
        f = list(f)
        for _ in range(k):
            f = [torch.where(fluid, v, torch.full_like(v, w)) for v, w in zip(f, _W2)]
            f = ref.step(f)
        return tuple(f)

    f = tuple(torch.full(m.shape, w, dtype=torch.float64, device="cuda") for w in _W2)
    left = case["steps"]
    while left > 0:
        k = min(25, left)
        f = torch.utils.checkpoint.checkpoint(steps, alpha, g, k, *f, use_reentrant=False)
        left -= k
    _, u = _moments(list(f), _C2, (g[0], g[1]), 1.0 / (1.0 + 0.5 * alpha))
    col = fluid[:, case["nx"] - 1]
    J = u[0][:, case["nx"] - 1][col].mean()
    ga, gg = torch.autograd.grad(J, (alpha, g))
    return {"J": J.detach(), "grad_alpha": ga, "grad_g": gg}


def exact(case, seed):
    if case["kind"] == "objective":
        return _exact_objective(case, seed)
    three = case["kind"] == "d3q19"
    mask = (_mask3 if three else _mask2)(case, seed)
    g = (0.0,) * mask.ndim
    if _forced(case):
        g = _FORCE3 if three else _FORCE2
    ref = _Reference(mask, case["tau"], g, case["collision"],
                     None if three else _boundaries(case))
    init = _initial(case, seed, mask)
    with torch.no_grad():
        f = ref.init(init[0], init[1:])
        for _ in range(case["steps"]):
            f = ref.step(f)
        rho, u = _moments(f, ref.C, g, None)
    out = [torch.where(ref.fluid, v, torch.zeros_like(v)) for v in [rho] + u]
    return {n: v for n, v in zip(("rho", "ux", "uy", "uz"), out)}
