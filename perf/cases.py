"""Performance cases of the IB-LBM framework: whole runs through its public
entry points (Sim, Batch, Server), as a program that uses it makes them.

A pass queues a few hundred to a few thousand time steps and reads back what
such a program keeps: the body history of those steps (forces, motion,
boundary fidelity) and the final fields.  A pass continues the flow where
the previous one left it.

Kinds of case
  cylinder      fixed cylinder in a uniform stream, velocity faces on three
                sides, zero-gradient outlet (drag and shedding runs)
  channel       fixed cylinder between bounce-back walls, parabolic inlet,
                zero-gradient outlet (the parameter-sweep geometry)
  oscillating   cylinder driven across the stream by a sine
  settling      one or two free disks falling in a closed box with Zou-He
                walls (Velocity-Verlet, explicit internal-mass correction)
  batch         many channel cases of a sweep stepped by shared launches
  serve         a burst of channel cases through the request server
"""
import math

import numpy as np
import torch

import paper_2609_02298_amd as ib

SCHEMES = {"DF": ib.DF, "MDF": ib.MDF, "DFC": ib.DFC}
KERNELS = {"hat": ib.HAT, "P4": ib.PESKIN4}
COLLISIONS = {"BGK": ib.BGK, "TRT": ib.TRT, "CMMRT": ib.CMMRT}
PRECISIONS = {"fp32": ib.FP32_SHIFTED, "fp64": ib.FP64}

# ------------------------------------------------------------------ the cases


def listed():
    """The listed cases; the comment above each says what it stands for."""
    return [
        # The smallest run in use: the 25 % blockage channel of the unit
        # checks, in double precision.  A step moves 2.3 MB, so launches and
        # latency are all of it.
        dict(name="channel-200x80-DF-hat-BGK-fp64", kind="channel", nx=200, ny=80, diameter=20.0,
             markers=63, scheme="DF", kernel="hat", collision="BGK", precision="fp64", re=20.0,
             u=0.05, steps=1000),
        # The benchmark's run: vortex shedding at Re 100 with five MDF passes.
        dict(name="cylinder-2000x800-MDF-P4-TRT-fp32", kind="cylinder", nx=2000, ny=800,
             diameter=80.0, markers=0, scheme="MDF", kernel="P4", collision="TRT",
             precision="fp32", re=100.0, u=0.1, steps=2000),
        # The same run in double precision, its accuracy reference.
        dict(name="cylinder-2000x800-MDF-P4-TRT-fp64", kind="cylinder", nx=2000, ny=800,
             diameter=80.0, markers=0, scheme="MDF", kernel="P4", collision="TRT",
             precision="fp64", re=100.0, u=0.1, steps=1500),
        # The published fixed-cylinder setup: odd sizes, marker spacing 2/3,
        # adaptive MDF (5 to 20 passes, tolerance 1e-4).
        dict(name="cylinder-2001x1601-adaptive-MDF-P4-BGK-fp32", kind="cylinder", nx=2001, ny=1601,
             diameter=40.0, markers=188, scheme="MDF", kernel="P4", collision="BGK",
             precision="fp32", re=100.0, u=0.1, steps=1000, adaptive=True),
        # A fixed body of a scheme/collision study: distribution-function
        # correction with the central-moment collision on a ragged lattice.
        dict(name="cylinder-1531x617-DFC-hat-CMMRT-fp32", kind="cylinder", nx=1531, ny=617,
             diameter=61.0, markers=0, scheme="DFC", kernel="hat", collision="CMMRT",
             precision="fp32", re=100.0, u=0.1, steps=1000),
        # A driven body: transverse oscillation below the shedding frequency.
        dict(name="oscillating-1200x600-MDF-P4-TRT-fp32", kind="oscillating", nx=1200, ny=600,
             diameter=40.0, markers=0, scheme="MDF", kernel="P4", collision="TRT",
             precision="fp32", re=100.0, u=0.1, steps=1000),
        # One sedimenting disk in a tall closed box (DFC, central moments).
        dict(name="settling-400x2000-DFC-P4-CMMRT-fp64", kind="settling", nx=400, ny=2000,
             diameter=20.0, markers=0, scheme="DFC", kernel="P4", collision="CMMRT",
             precision="fp64", ar=1000.0, nu=0.02, bodies=1, steps=600),
        # Two disks of different density, one above the other.
        dict(name="settling-pair-400x2000-DFC-P4-CMMRT-fp32", kind="settling", nx=400, ny=2000,
             diameter=20.0, markers=0, scheme="DFC", kernel="P4", collision="CMMRT",
             precision="fp32", ar=1000.0, nu=0.02, bodies=2, steps=600),
        # The published settling channel: a large free disk (754 markers) on
        # a lattice beyond the on-chip caches.
        dict(name="settling-1281x3841-DF-P4-BGK-fp32", kind="settling", nx=1281, ny=3841,
             diameter=160.0, markers=754, scheme="DF", kernel="P4", collision="BGK",
             precision="fp32", ar=76562.5, nu=0.0214, bodies=1, steps=400),
        # The largest lattice of the parameter sweep: memory bandwidth.
        dict(name="channel-7175x2014-DF-hat-BGK-fp32", kind="channel", nx=7175, ny=2014,
             diameter=201.4, markers=0, scheme="DF", kernel="hat", collision="BGK",
             precision="fp32", re=150.0, u=0.1, steps=600),
        # A resident set of sweep cases, all schemes, kernels and collisions.
        dict(name="batch-12-fp32", kind="batch", count=12, width_min=128, width_max=512, mix=1,
             precision="fp32", steps=400),
        # A burst of requests: admission, stepping and retirement included.
        dict(name="serve-12-fp32", kind="serve", count=12, width_min=128, width_max=384, mix=2,
             precision="fp32", steps=300),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def loguni(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    precision = rng.choice(["fp32", "fp32", "fp64"])
    kind = rng.choice(["cylinder", "channel", "oscillating", "settling", "settling", "batch",
                       "serve"])
    if kind in ("batch", "serve"):
        return dict(kind=kind, count=rng.randint(6, 12), width_min=128, width_max=loguni(200, 512),
                    mix=rng.randint(3, 10 ** 6), precision=precision,
                    steps=rng.randint(150, 300))
    c = dict(kind=kind, markers=0, scheme=rng.choice(list(SCHEMES)),
             kernel=rng.choice(list(KERNELS)), collision=rng.choice(list(COLLISIONS)),
             precision=precision)
    if kind == "settling":
        nx = loguni(200, 1000)
        d = round(nx * rng.uniform(0.06, 0.125), 1)
        ny = int(nx * rng.uniform(3.0, 5.0))
        c.update(nx=nx, ny=ny, diameter=d, ar=round(rng.uniform(300.0, 1000.0), 1), nu=0.02,
                 bodies=rng.choice([1, 1, 2]), steps=rng.randint(200, 400))
    else:
        ny = loguni(96, 1600)
        nx = int(ny * rng.uniform(1.25, 3.5))
        d = round(max(8.0, ny * rng.uniform(0.05, 0.125)), 1)
        c.update(nx=nx, ny=ny, diameter=d, re=round(rng.uniform(20.0, 100.0), 1), u=0.08,
                 steps=rng.randint(300, 600))
        if c["scheme"] == "MDF" and rng.random() < 0.4:
            c["adaptive"] = True
    return c


# -------------------------------------------------- a case's workload in full


def _tau(u, d, re):
    tau = 0.5 + 3.0 * u * d / re
    # the collision operators are used between tau 0.53 and 1.75
    return min(max(tau, 0.53), 1.75)


def _workloads(case, seed):
    """The lattice and body descriptions of the case's runs (one, or one per
    member of a batch).  The seed moves the bodies against the lattice by a
    fraction of a node and shifts the phase of the start disturbance."""
    rng = np.random.default_rng([0x1B, int(seed)])
    if case["kind"] in ("batch", "serve"):
        mix = np.random.default_rng([0x5EED, int(case["mix"])])
        combos = [(s, k, c) for s in SCHEMES for k in KERNELS for c in COLLISIONS]
        order = mix.permutation(len(combos))
        out = []
        for i in range(case["count"]):
            w = int(round(math.exp(mix.uniform(math.log(case["width_min"]),
                                               math.log(case["width_max"])))))
            a, re = mix.uniform(2.0, 4.0), mix.uniform(20.0, 100.0)
            s, k, c = combos[int(order[i % len(combos)])]
            one = dict(kind="channel", nx=int(round(a * w)), ny=w, diameter=w / 10.0, markers=0,
                       scheme=s, kernel=k, collision=c, precision=case["precision"], re=re, u=0.1,
                       steps=case["steps"])
            out.append(_workload(one, rng))
        return out
    return [_workload(case, rng)]


def _workload(case, rng):
    kind, nx, ny, d = case["kind"], case["nx"], case["ny"], case["diameter"]
    dx, dy, phase = rng.uniform(-0.5, 0.5, 3)
    body = dict(diameter=d, n_markers=case["markers"], scheme=SCHEMES[case["scheme"]],
                kernel=KERNELS[case["kernel"]], mdf_iters=5, motion=ib.FIXED)
    if case.get("adaptive"):
        body.update(mdf_nmin=5, mdf_iters=20, mdf_tol=1e-4)
    w = dict(nx=nx, ny=ny, collision=COLLISIONS[case["collision"]], trt_magic=0.25, cm_s_q=1.2,
             cm_s_eps=1.4, rho0=1.0, phase=2.0 * math.pi * float(phase))
    if kind == "settling":
        nu, ar = case["nu"], case["ar"]
        g = ar * nu * nu / (0.5 * d ** 3)
        body.update(motion=ib.FREE, internal_mass=ib.IM_FENG, integrator=ib.VERLET)
        y = max(ny - 10.0 * d, 0.62 * ny)
        bodies = [dict(body, xc=0.5 * nx + dx, yc=y + dy, density_ratio=1.5)]
        if case["bodies"] == 2:
            gap = d + 2.0 * 4 + 8.0
            bodies[0]["yc"] = y - 0.5 * gap + dy
            bodies.append(dict(body, xc=0.5 * nx - dx, yc=y + 0.5 * gap + dy, density_ratio=1.25))
        w.update(tau=0.5 + 3.0 * nu, bc=(ib.ZOU_HE,) * 4, u_bc=0.0, gravity=(0.0, -g), u0=0.0,
                 bodies=bodies)
        return w
    u = case["u"]
    far = kind != "channel"
    w.update(tau=_tau(u, d, case["re"]), u_bc=u, u0=u,
             bc=(ib.VEL_UNIFORM, ib.ZERO_GRADIENT, ib.VEL_UNIFORM, ib.VEL_UNIFORM) if far else
             (ib.VEL_PARABOLIC, ib.ZERO_GRADIENT, ib.BOUNCE_BACK, ib.BOUNCE_BACK))
    body.update(xc=0.25 * nx + dx, yc=0.5 * ny + dy)
    if kind == "oscillating":
        body.update(motion=ib.PRESCRIBED_SIN, amp=(0.0, 0.2 * d), freq=0.8 * 0.165 * u / d,
                    phase=0.0)
    w["bodies"] = [body]
    return w


def _start_velocity(w):
    """The start state's velocity: the inlet's own profile with a smooth
    two per cent disturbance whose phase the seed sets (a rest state is
    disturbed by 1e-4)."""
    nx, ny = w["nx"], w["ny"]
    x = np.arange(nx) / nx
    y = (np.arange(ny) + 0.5) / ny
    base = np.full(ny, w["u0"])
    if w["bc"][0] == ib.VEL_PARABOLIC:
        base = 4.0 * w["u0"] * y * (1.0 - y)
    amp = 0.02 * w["u0"] if w["u0"] else 1e-4
    sy = np.sin(math.pi * y) * amp
    ux = base[:, None] + sy[:, None] * np.cos(4.0 * math.pi * x + w["phase"])[None, :]
    uy = (sy * np.cos(2.0 * math.pi * y))[:, None] * np.sin(4.0 * math.pi * x + w["phase"])[None, :]
    return ux, uy


# ---------------------------------------------------------- prepare and run


def prepare(case, seed):
    precision = PRECISIONS[case["precision"]]
    works = _workloads(case, seed)
    st = dict(case=case, works=works, done=0)
    if case["kind"] == "serve":
        st["server"] = ib.Server(precision=precision, quantum=128)
        return st
    st["sims"] = [_start(w, precision) for w in works]
    if case["kind"] == "batch":
        st["batch"] = ib.Batch(precision=precision)
        for sim in st["sims"]:
            st["batch"].attach(sim)
    return st


def _start(w, precision):
    sim = ib.Sim(w, precision=precision)
    sim.set_equilibrium(*_start_velocity(w))
    return sim


def _fall_steps(case, w):
    """Steps after which a settling run ends, well before the disk could
    reach the floor: half the way down at u_g = (0.5 g D)^(1/2)."""
    d = case["diameter"]
    ug = math.sqrt(case["ar"]) * case["nu"] / d
    return int(0.5 * (min(b["yc"] for b in w["bodies"]) - d) / ug)


def run(state):
    case, steps = state["case"], state["case"]["steps"]
    if case["kind"] == "serve":
        server = state["server"]
        ids = [server.submit(w, steps, fields=True) for w in state["works"]]
        out = {}
        for i, rid in enumerate(ids):
            r = server.wait(rid)
            if r["status"] != 0:
                raise RuntimeError(f"request {i}: status {r['status']}")
            b = r["bodies"][0]
            out[f"{i}.force"] = np.array([b["fx"], b["fy"], b["torque"]])
            out[f"{i}.rho"], out[f"{i}.ux"], out[f"{i}.uy"] = r["rho"], r["ux"], r["uy"]
        return out
    if case["kind"] == "settling" and \
            state["done"] + steps > max(steps, _fall_steps(case, state["works"][0])):
        # the disk has fallen its way: the next run of the study begins
        state["sims"][0].close()
        state["sims"] = [_start(state["works"][0], PRECISIONS[case["precision"]])]
        state["done"] = 0
    if case["kind"] == "batch":
        state["batch"].step(steps)
    else:
        state["sims"][0].step(steps)
    first = state["done"] + 1
    state["done"] += steps
    out = {}
    for i, sim in enumerate(state["sims"]):
        for b in range(len(state["works"][i]["bodies"])):
            h = sim.history(b, first, steps)
            out.update(_split_history(f"{i}.{b}", h, short=case["kind"] == "batch"))
        rho, ux, uy = sim.fields()
        out[f"{i}.rho"] = rho
        out[f"{i}.ux"] = ux
        out[f"{i}.uy"] = uy
    return out


def _split_history(tag, h, short=False):
    """The history rows by what they hold, so that each part is compared at
    its own scale: (force, torque), (slip mean and max, MDF residual) and,
    unless short (the fixed bodies of a batch), (position), (velocity, spin),
    (step, passes, flags)."""
    out = {f"{tag}.force": h[:, 1:4].copy(), f"{tag}.fidelity": h[:, 9:12].copy()}
    if not short:
        out.update({f"{tag}.position": h[:, 4:6].copy(), f"{tag}.motion": h[:, 6:9].copy(),
                    f"{tag}.counts": h[:, [0, 12, 13]].copy()})
    return out


# -------------------------------------------------------- work and tolerance


def work(case):
    """Every step reads and writes the nine populations of every node once;
    a collision takes about 100 (BGK), 110 (TRT) or 200 (central moments)
    operations; the read-back reads the populations and the two force
    components and writes three fields of doubles (and the history rows)."""
    size = 4 if case["precision"] == "fp32" else 8
    nbytes = flops = 0
    for w in _workloads(case, 0):
        nodes = w["nx"] * w["ny"]
        per = {ib.BGK: 100, ib.TRT: 110, ib.CMMRT: 200}[w["collision"]]
        nbytes += nodes * 18 * size * case["steps"] + nodes * (11 * size + 24)
        flops += nodes * per * case["steps"]
        nbytes += len(w["bodies"]) * 128 * case["steps"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Rounding differences between correct implementations, grown over the
    steps of a pass: against exact() the transverse velocity, the smallest
    of the outputs, is the furthest off, 1.3e-5 in fp32 and 2e-12 in fp64."""
    if case["precision"] == "fp64":
        return {"rel": 1e-10, "max": 1e-7}
    return {"rel": 1e-4, "max": 1e-2}


# ------------------------------------------------------- the exact reference

_EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
_EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
_OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)
_W = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4


def exact(case, seed):
    """What the first run() on prepare(case, seed) returns, computed in
    float64 with plain torch; None where that would take too long."""
    works = _workloads(case, seed)
    cost = sum(case["steps"] * (2.0e-3 * (1 + 2 * bool(case.get("adaptive"))) * len(w["bodies"]) +
                                1.1e-9 * w["nx"] * w["ny"] *
                                (2 if w["collision"] == ib.CMMRT else 1)) for w in works)
    if cost > 14.0:
        return None
    out = {}
    for i, w in enumerate(works):
        ref = _Reference(w, rest=case["kind"] == "serve")
        hist = ref.run(case["steps"])
        rho, ux, uy = ref.fields()
        if case["kind"] == "serve":
            out[f"{i}.force"] = hist[0][-1, 1:4]
        else:
            for b, h in enumerate(hist):
                out.update(_split_history(f"{i}.{b}", h, short=case["kind"] == "batch"))
        out[f"{i}.rho"], out[f"{i}.ux"], out[f"{i}.uy"] = rho, ux, uy
    return out


def _delta(kernel, r):
    a = r.abs()
    if kernel == ib.HAT:
        return (1.0 - a).clamp(min=0.0)
    near = 0.125 * (3.0 - 2.0 * a + (1.0 + 4.0 * a - 4.0 * a * a).clamp(min=0.0).sqrt())
    far = 0.125 * (5.0 - 2.0 * a - (-7.0 + 12.0 * a - 4.0 * a * a).clamp(min=0.0).sqrt())
    return torch.where(a <= 1.0, near, torch.where(a <= 2.0, far, torch.zeros_like(a)))


class _RefBody:
    """A disk of the reference run: markers on a patch of the lattice."""

    def __init__(self, ref, b):
        self.ref, self.b = ref, b
        self.R = 0.5 * b["diameter"]
        self.nb = b["n_markers"] or int(round(math.pi * b["diameter"]))
        self.ds = math.pi * b["diameter"] / self.nb
        th = 2.0 * math.pi * torch.arange(self.nb, dtype=torch.float64, device=ref.dev) / self.nb
        self.cos, self.sin = th.cos(), th.sin()
        self.ns = 2 if b["kernel"] == ib.HAT else 4
        area = math.pi * self.R ** 2
        self.mf = area
        self.ms = b.get("density_ratio", 1.0) * area
        self.Is = 0.5 * self.ms * self.R ** 2
        self.x, self.y = float(b["xc"]), float(b["yc"])
        self.v, self.vp, self.om = [0.0, 0.0], [0.0, 0.0], 0.0
        self.f, self.tq = [0.0, 0.0], 0.0
        self.place()
        if b["scheme"] == ib.MDF:
            one = torch.ones(self.nb, dtype=torch.float64, device=ref.dev)
            self.omega = 1.0 / (self.ds * float(self.interp(self.spread(one)).max()))

    def place(self):
        """Stencils and weights of the markers about the current centre."""
        s = self.ns // 2
        X, Y = self.x + self.R * self.cos, self.y + self.R * self.sin
        self.px0 = int(math.floor(self.x - self.R)) - self.ns
        self.py0 = int(math.floor(self.y - self.R)) - self.ns
        self.pw = int(math.ceil(2 * self.R)) + 2 * self.ns + 4
        off = torch.arange(self.ns, device=X.device)
        ix = X.floor().long()[:, None] - (s - 1) + off
        iy = Y.floor().long()[:, None] - (s - 1) + off
        self.wx, self.wy = _delta(self.b["kernel"], ix - X[:, None]), _delta(self.b["kernel"],
                                                                           iy - Y[:, None])
        w = self.wy[:, :, None] * self.wx[:, None, :]
        self.w = w.reshape(self.nb, -1)
        idx = (iy - self.py0)[:, :, None] * self.pw + (ix - self.px0)[:, None, :]
        self.idx = idx.reshape(self.nb, -1)
        self.X, self.Y = X, Y

    def interp(self, field):
        return (field.reshape(*field.shape[:-2], -1)[..., self.idx] * self.w).sum(-1)

    def spread(self, v):
        """sum_k v_k D_h(x - X_k) on the patch (v: [..., nb])."""
        lead = v.shape[:-1]
        src = (v[..., None] * self.w).reshape(*lead, -1)
        out = torch.zeros(*lead, self.pw * self.pw, dtype=torch.float64, device=v.device)
        out.index_add_(-1, self.idx.reshape(-1), src)
        return out.reshape(*lead, self.pw, self.pw)

    def advance(self, step):
        """Kinematics to the end of the step; sets the markers' velocity."""
        b = self.b
        if b["motion"] == ib.FIXED:
            vel, om = (0.0, 0.0), 0.0
        elif b["motion"] == ib.PRESCRIBED_SIN:
            w = 2.0 * math.pi * b["freq"]
            ph = w * (step + 1) + b["phase"]
            self.x = b["xc"] + b["amp"][0] * math.sin(ph)
            self.y = b["yc"] + b["amp"][1] * math.sin(ph)
            vel, om = (b["amp"][0] * w * math.cos(ph), b["amp"][1] * w * math.cos(ph)), 0.0
            self.v = list(vel)
            self.place()
        else:
            g = self.ref.w["gravity"]
            self.fg = [(self.ms - self.mf) * g[0], (self.ms - self.mf) * g[1]]
            self.dim = [self.mf * (self.v[i] - self.vp[i]) for i in (0, 1)]
            self.vp = list(self.v)
            self.vh = [self.v[i] + (self.f[i] + self.fg[i] + self.dim[i]) / (2.0 * self.ms)
                       for i in (0, 1)]
            self.x += self.vh[0]
            self.y += self.vh[1]
            self.omh = self.om + self.tq / (2.0 * self.Is)
            vel, om = tuple(self.v), self.om
            self.place()
        self.ud = torch.stack((vel[0] - om * (self.Y - self.y), vel[1] + om * (self.X - self.x)))

    def patch(self, t):
        return t[..., self.py0:self.py0 + self.pw, self.px0:self.px0 + self.pw]

    def enforce(self, step):
        """The scheme on the new populations; the step's history row."""
        b, ds = self.b, self.ds
        f = self.patch(self.ref.f)
        ex, ey = self.ref.ex, self.ref.ey
        rho = f.sum(0)
        u = torch.stack(((f * ex).sum(0), (f * ey).sum(0))) / rho
        res, passes = 0.0, 1
        if b["scheme"] == ib.DFC:
            g = self.interp(f)
            lam = 1.0 / (2.0 * ds * self.interp(self.spread(torch.ones_like(self.X))))
            wq = self.ref.wq[:, None]
            eud = ex.reshape(9, 1) * self.ud[0] + ey.reshape(9, 1) * self.ud[1]
            dl = lam * (g[list(_OPP)] - g + 6.0 * wq * eud)
            f += self.spread(dl) * ds
            F = -ds * torch.stack(((ex.reshape(9, 1) * dl).sum(0), (ey.reshape(9, 1) * dl).sum(0)))
            rho = f.sum(0)
            u = torch.stack(((f * ex).sum(0), (f * ey).sum(0))) / rho
            fx, fy = F.sum(1).tolist()
            tq = float(((self.X - self.x) * F[1] - (self.Y - self.y) * F[0]).sum())
            passes = 0
        else:
            rX = self.interp(rho)
            if b["scheme"] == ib.DF:
                F = 2.0 * rX * (self.ud - self.interp(u))
                u = u + self.spread(F) * ds / (2.0 * rho)
            else:
                F = torch.zeros_like(self.ud)
                tol, prev, passes = b.get("mdf_tol", 0.0), 0.0, 0
                for n in range(1, b["mdf_iters"] + 1):
                    e = self.ud - self.interp(u)
                    if tol > 0.0 or n == b["mdf_iters"]:
                        res = float((e * e).sum(0).sqrt().max())
                    if tol > 0.0:
                        if (n > b["mdf_nmin"] and res < tol) or (n > 1 and res > 1.5 * prev):
                            break
                        prev = res
                    dF = self.omega * 2.0 * rX * e
                    u = u + self.spread(dF) * ds / (2.0 * rho)
                    F += dF
                    passes = n
            self.patch(self.ref.force).add_(self.spread(F) * ds)
            ws = self.wx.sum(1) * self.wy.sum(1)
            fx, fy = (-(F * ws).sum(1) * ds).tolist()
            tq = float(-((self.X - self.x) * F[1] - (self.Y - self.y) * F[0]).sum() * ds)
        slip = self.interp(u) - self.ud
        slip = (slip * slip).sum(0).sqrt()
        if b["motion"] == ib.FREE:
            self.v = [self.vh[i] + ((fx, fy)[i] + self.fg[i] + self.dim[i]) / (2.0 * self.ms)
                      for i in (0, 1)]
            self.om = self.omh + tq / (2.0 * self.Is)
        self.f, self.tq = [fx, fy], tq
        return [step + 1, fx, fy, tq, self.x, self.y, self.v[0], self.v[1], self.om,
                float(slip.mean()), float(slip.max()), res, passes, 0, 0, 0]


class _Reference:
    """D2Q9 run of one workload in float64 (populations f[9, ny, nx])."""

    def __init__(self, w, rest):
        self.w = w
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        t = dict(dtype=torch.float64, device=self.dev)
        self.ex = torch.tensor(_EX, **t).reshape(9, 1, 1)
        self.ey = torch.tensor(_EY, **t).reshape(9, 1, 1)
        self.wq = torch.tensor(_W, **t)
        nx, ny = w["nx"], w["ny"]
        y = (torch.arange(ny, **t) + 0.5) / ny
        if rest:
            # a request starts from the inlet's own equilibrium
            ux = (4.0 * w["u_bc"] * y * (1.0 - y))[:, None].expand(ny, nx)
            uy = torch.zeros(ny, nx, **t)
        else:
            ux, uy = (torch.as_tensor(np.ascontiguousarray(a), **t) for a in _start_velocity(w))
        eu = self.ex * ux + self.ey * uy
        self.f = self.wq.reshape(9, 1, 1) * (1.0 + 3.0 * eu + 4.5 * eu * eu -
                                             1.5 * (ux * ux + uy * uy))
        self.force = torch.zeros(2, ny, nx, **t)
        self.bodies = [_RefBody(self, b) for b in w["bodies"]]
        yl = torch.arange(ny, **t)
        # wall velocity at the mid-points of the links through the west face
        self.uw = {i: (4.0 * w["u_bc"] * (yl + 0.5 * _EY[i] + 0.5) * (ny - 0.5 - yl - 0.5 * _EY[i]) /
                       ny ** 2 if w["bc"][0] == ib.VEL_PARABOLIC else
                       torch.full((ny,), w["u_bc"], **t)) for i in (3, 6, 7)}

    def run(self, steps):
        hist = [np.zeros((steps, 16)) for _ in self.bodies]
        for n in range(steps):
            for b in self.bodies:
                b.advance(n)
            self.collide()
            self.force.zero_()
            self.stream()
            for b, h in zip(self.bodies, hist):
                h[n] = b.enforce(n)
        return hist

    def fields(self):
        f, F = self.f, self.force
        rho = f.sum(0)
        ux = ((f * self.ex).sum(0) + 0.5 * F[0]) / rho
        uy = ((f * self.ey).sum(0) + 0.5 * F[1]) / rho
        return rho.cpu().numpy(), ux.cpu().numpy(), uy.cpu().numpy()

    def collide(self):
        w, f = self.w, self.f
        Fx, Fy = self.force
        rho = f.sum(0)
        ux = (f[1] - f[3] + f[5] - f[6] - f[7] + f[8] + 0.5 * Fx) / rho
        uy = (f[2] - f[4] + f[5] + f[6] - f[7] - f[8] + 0.5 * Fy) / rho
        if w["collision"] == ib.CMMRT:
            return self.collide_central(rho, ux, uy, Fx, Fy)
        se = so = 1.0 / w["tau"]
        if w["collision"] == ib.TRT:
            so = 1.0 / (w["trt_magic"] / (w["tau"] - 0.5) + 0.5)
        uu, uF = 1.5 * (ux * ux + uy * uy), 3.0 * (ux * Fx + uy * Fy)
        for i, j in ((0, 0), (1, 3), (2, 4), (5, 7), (6, 8)):
            a = _EX[i] * ux + _EY[i] * uy
            b = _EX[i] * Fx + _EY[i] * Fy
            even = se * (_W[i] * rho * (1.0 + 4.5 * a * a - uu) - 0.5 * (f[i] + f[j])) + \
                (1.0 - 0.5 * se) * _W[i] * (9.0 * a * b - uF)
            if i == 0:
                f[0] += even
                continue
            odd = so * (3.0 * _W[i] * rho * a - 0.5 * (f[i] - f[j])) + \
                (1.0 - 0.5 * so) * 3.0 * _W[i] * b
            f[i] += even + odd
            f[j] += even - odd

    def collide_central(self, rho, ux, uy, Fx, Fy):
        w, f = self.w, self.f
        # k_pq = sum_i f_i (e_x - u_x)^p (e_y - u_y)^q by rows, then columns
        grid = [[f[7], f[4], f[8]], [f[3], f[0], f[1]], [f[6], f[2], f[5]]]
        rows = []
        for m, z, p in grid:
            s0, s1, s2 = m + z + p, p - m, p + m
            rows.append((s0, s1 - ux * s0, s2 - 2.0 * ux * s1 + ux * ux * s0))
        k = []
        for c in range(3):
            m, z, p = rows[0][c], rows[1][c], rows[2][c]
            s0, s1, s2 = m + z + p, p - m, p + m
            k.append([s0, s1 - uy * s0, s2 - 2.0 * uy * s1 + uy * uy * s0])
        om, sq, se = 1.0 / w["tau"], w["cm_s_q"], w["cm_s_eps"]
        k[1][0] = k[1][0] + Fx
        k[0][1] = k[0][1] + Fy
        k[2][0] = k[2][0] - om * (k[2][0] - rho / 3.0)
        k[0][2] = k[0][2] - om * (k[0][2] - rho / 3.0)
        k[1][1] = k[1][1] * (1.0 - om)
        k[2][1] = k[2][1] * (1.0 - sq) + (1.0 - 0.5 * sq) * Fy / 3.0
        k[1][2] = k[1][2] * (1.0 - sq) + (1.0 - 0.5 * sq) * Fx / 3.0
        k[2][2] = k[2][2] - se * (k[2][2] - rho / 9.0)

        def back(u, k0, k1, k2):
            m1, m2 = k1 + u * k0, k2 + 2.0 * u * k1 + u * u * k0
            return 0.5 * (m2 - m1), k0 - m2, 0.5 * (m2 + m1)

        cols = [back(uy, *k[c]) for c in range(3)]
        names = ((7, 4, 8), (3, 0, 1), (6, 2, 5))
        for r in range(3):
            for i, v in zip(names[r], back(ux, cols[0][r], cols[1][r], cols[2][r])):
                f[i] = v

    def stream(self):
        w, f = self.w, self.f
        nx, ny, bc = w["nx"], w["ny"], w["bc"]
        new = torch.stack([torch.roll(f[i], (_EY[i], _EX[i]), (0, 1)) for i in range(9)])
        if bc[0] == ib.ZOU_HE:
            self.f = new
            return self.zou_he()
        # links through the south and north faces: walls, or velocity faces
        # (the west face's velocity closure goes first at its corners)
        u = w["u_bc"]
        for i, row in ((4, 0), (7, 0), (8, 0), (2, ny - 1), (5, ny - 1), (6, ny - 1)):
            v = f[i, row]
            if bc[2] != ib.BOUNCE_BACK:
                v = v - 6.0 * _W[i] * _EX[i] * u
            new[_OPP[i], row] = v
        for i in (3, 6, 7):
            v = f[i, :, 0] + 6.0 * _W[i] * self.uw[i]
            if bc[2] == ib.BOUNCE_BACK and _EY[i]:
                corner = 0 if _EY[i] < 0 else ny - 1
                v[corner] = f[i, corner, 0]
            new[_OPP[i], :, 0] = v
        # zero-gradient outlet: the entering populations of the column inside
        for i in (3, 6, 7):
            new[i, :, nx - 1] = new[i, :, nx - 2]
        self.f = new

    def zou_he(self):
        f = self.f
        ny, nx = f.shape[1:]
        for row, n, d1, d2 in ((0, 2, 5, 6), (ny - 1, 4, 8, 7)):
            v = f[:, row, 1:-1]
            t = 0.5 * (v[1] - v[3])
            v[n] = v[_OPP[n]]
            v[d1] = v[_OPP[d1]] - t
            v[d2] = v[_OPP[d2]] + t
        for col, n, d1, d2 in ((0, 1, 5, 8), (nx - 1, 3, 6, 7)):
            v = f[:, 1:-1, col]
            t = 0.5 * (v[2] - v[4])
            v[n] = v[_OPP[n]]
            v[d1] = v[_OPP[d1]] - t
            v[d2] = v[_OPP[d2]] + t
        for x, sx in ((0, 1), (nx - 1, -1)):
            for y, sy in ((0, 1), (ny - 1, -1)):
                d = {(1, 1): 5, (1, -1): 8, (-1, 1): 6, (-1, -1): 7}[(sx, sy)]
                pair = (6, 8) if d in (5, 7) else (5, 7)
                v = f[:, y, x]
                for i in (1 if sx > 0 else 3, 2 if sy > 0 else 4, d):
                    v[i] = v[_OPP[i]]
                known = sum(v[i] for i in range(9) if i not in pair)
                v[list(pair)] = 0.5 * (f[:, y + sy, x + sx].sum() - known)
