"""What the library is timed on: calls of its public entry points as programs make them, from one
small modelling call to batched, checkpointed, time-lapse and 3D gradients.

A case is a dict of plain values.  `prepare` makes what a program holds before the call (plan,
workspace, packed inputs), `run` makes one call, `work` counts what the call cannot do without,
and `exact` evaluates the same operators in FP64 with plain torch.

Models are the benchmark's kind: flat layers 1.5-4.5 km/s with a smooth 5 % perturbation; sources
and receivers near the surface (wells for the time-lapse survey), a Ricker source of 15 Hz, time
step 0.4 h / vmax.  All inputs come from the seed alone.
"""
import math
import random

import numpy as np
import torch
import torch.nn.functional as F

import paper_2304_05592_amd as A

VMAX = 5.5        # km/s, bound of every model below
F0 = 0.015        # kHz
DAMP_R = 1e-3


def listed():
    return [
        # one quick modelling call: the smallest thing a user does, bound by launches
        dict(name="fwd_small", kind="forward", nz=101, nx=201, nbl=40, h=10.0, nt=626, nshot=1, nrec=101),
        # shot-by-shot inversion: the gradient and F^T dd of one shot, whole wavefield kept
        dict(name="grad_one_shot", kind="gradient", nz=341, nx=650, nbl=40, h=6.25, nt=1200, nshot=1, nrec=650,
             prec=0),
        # the benchmark's batched gradient (fewer time samples), launch shapes tuned once per plan
        dict(name="grad_batch", kind="gradient", nz=341, nx=650, nbl=40, h=6.25, nt=1200, nshot=16, nrec=650,
             prec=0, tune=True),
        # the training-style call: autograd through F with checkpoints, from the physical grid
        dict(name="autograd_ckpt", kind="autograd", nz=512, nx=1024, nbl=40, h=6.25, nt=500, nshot=16, nrec=1024,
             nslots=16, tune=True),
        # modelling of shots with windows and recording lengths of their own, in one batch
        dict(name="fwd_uneven", kind="forward", nz=341, nx=1024, nbl=40, h=6.25, nt=1000, nshot=24, nrec=512,
             uneven=True),
        # one time-lapse iteration: wavespeed gradients of every vintage, crosswell
        dict(name="timelapse_iter", kind="timelapse", nz=256, nx=512, nbl=40, h=6.25, nt=600, nvint=6, nshot=24,
             nrec=960),
        # linearised data of the batch
        dict(name="born_batch", kind="born", nz=341, nx=650, nbl=40, h=6.25, nt=600, nshot=16, nrec=650),
        # the gradient from probes of the time axis, where memory is short
        dict(name="probed_batch", kind="probed", nz=341, nx=650, nbl=40, h=6.25, nt=400, nshot=8, nrec=650,
             nprobe=8),
        # a 3D gradient at full size, 16-bit wavefield
        dict(name="grad_3d", kind="gradient", nz=256, ny=256, nx=256, nbl=40, h=12.5, nt=160, nshot=1, nrec=1024,
             prec=1),
        # 3D modelling of a cut-out of that model
        dict(name="fwd_3d_crop", kind="forward", nz=64, ny=64, nx=64, nbl=40, h=12.5, nt=300, nshot=1, nrec=1024),
        # a small survey with odd sizes and a 16-bit wavefield
        dict(name="grad_odd_16bit", kind="gradient", nz=151, nx=227, nbl=17, h=10.0, nt=501, nshot=3, nrec=113,
             prec=1),
        # rock physics of 15 vintages and its pullback
        dict(name="rock_physics", kind="rock", nz=256, nx=512, nvint=15),
    ]


def draw(rng: random.Random):
    lu = lambda a, b: int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))
    kind = rng.choice(["forward", "gradient", "gradient", "autograd", "timelapse", "born", "probed", "rock", "3d"])
    if kind == "rock":
        return dict(kind="rock", nz=lu(60, 400), nx=lu(100, 800), nvint=rng.randint(1, 20))
    if kind == "3d":
        c = dict(kind=rng.choice(["forward", "gradient"]), nz=lu(40, 200), ny=lu(40, 200),
                 nx=lu(40, 200), nbl=rng.choice([8, 20, 40]), h=12.5, nshot=rng.randint(1, 2), nrec=lu(16, 2000), prec=rng.choice([0, 1, 2]))
    else:
        c = dict(kind=kind, nz=lu(60, 512), nx=lu(90, 1100), nbl=rng.choice([12, 17, 40, 40, 50]),
                 h=rng.choice([6.25, 10.0]), nshot=lu(1, 32), nrec=lu(20, 1000))
        if kind == "gradient":
            c["prec"] = rng.choice([0, 0, 0, 1, 2])
        if kind == "autograd":
            c["nslots"] = rng.randint(4, 24)
        if kind == "timelapse":
            c["nvint"] = rng.randint(1, 8)
            c["nshot"] = c["nvint"] * rng.randint(1, 4)
        if kind == "probed":
            c["nprobe"] = rng.randint(1, 12)
        if kind == "forward":
            c["uneven"] = rng.random() < 0.5 and c["nshot"] > 1
    if c["kind"] in ("forward", "gradient", "autograd", "born"):
        c["tune"] = rng.random() < 0.3
    # as many time samples as keep the call within the cost of the listed ones
    pts = c["nshot"] * math.prod(n + 2 * c["nbl"] for n in _dims(c))
    cost = {"forward": 1.0, "gradient": 2.6, "timelapse": 2.6, "autograd": 7.0, "born": 2.0, "probed": 8.0}[c["kind"]]
    if len(_dims(c)) == 3:
        cost *= 4.0
    c["nt"] = max(60, min(lu(300, 1500), int(1.2e10 / (cost * pts))))
    return c


def _dims(c):
    return [c[k] for k in ("nz", "ny", "nx") if k in c]


# ---------------------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _smooth(shape, cells, gen):
    """A smooth random field of unit scale: coarse normal noise, interpolated."""
    coarse = [max(2, n // cells + 2) for n in shape]
    x = torch.randn([1, 1] + coarse, generator=gen, device="cuda", dtype=torch.float32)
    mode = "bilinear" if len(shape) == 2 else "trilinear"
    return F.interpolate(x, size=list(shape), mode=mode, align_corners=True)[0, 0]


def _velocity(dims, gen, smooth_only=False):
    nz = dims[0]
    k = torch.arange(nz, device="cuda")
    col = 1.5 + 3.0 * torch.div(k * 8, nz, rounding_mode="floor") / 7
    if smooth_only:
        col = torch.linspace(1.5, 4.5, nz, device="cuda")
    v = col.reshape([nz] + [1] * (len(dims) - 1)) * (1.0 + 0.05 * _smooth(dims, 32, gen).clamp(-3.5, 3.5))
    return v.clamp(1.2, VMAX).to(torch.float32)


def _ricker(t):
    a = (math.pi * F0 * t) ** 2
    return (1.0 - 2.0 * a) * torch.exp(-a)


def _wavelet(nt, dt):
    t = torch.arange(nt, device="cuda", dtype=torch.float64) * dt
    return _ricker(t - 1.5 / F0).to(torch.float32)


def _traces(nt, nrec, dt, gen):
    """Residual-like traces [nt][nrec]: three Ricker arrivals per trace."""
    t = (torch.arange(nt, device="cuda", dtype=torch.float32) * dt)[:, None]
    out = torch.zeros(nt, nrec, device="cuda")
    for _ in range(3):
        amp = torch.randn(1, nrec, generator=gen, device="cuda")
        tau = torch.rand(1, nrec, generator=gen, device="cuda") * (nt * dt)
        out += amp * _ricker(t - tau)
    return out.contiguous()


def _pad(x, nbl):
    """Edge replication by indexing (differentiable)."""
    for ax in range(x.dim()):
        i = torch.arange(-nbl, x.shape[ax] + nbl, device=x.device).clamp(0, x.shape[ax] - 1)
        x = x.index_select(ax, i)
    return x


class _Survey:
    """Geometry of a case (host side) and its seeded inputs (device side)."""

    def __init__(self, c, seed):
        self.c, gen = c, _gen(seed)
        rng = random.Random(seed)
        dims, h, nbl = _dims(c), c["h"], c["nbl"]
        self.nd, self.h, self.nbl = len(dims), h, nbl
        self.dt = 0.4 * h / VMAX
        vint = c.get("nvint", 1)
        shape_rng = random.Random(1000 + c["nshot"])      # sizes belong to the case, not to the seed
        self.phys, self.nts, self.win = [], [], []
        for s in range(c["nshot"]):
            if c.get("uneven"):
                w = shape_rng.randint(min(256, max(8, dims[-1] // 2)), dims[-1])
                self.phys.append([dims[0], w])
                self.nts.append(shape_rng.randint(max(2, int(0.4 * c["nt"])), c["nt"]))
                self.win.append(s)
            else:
                self.nts.append(c["nt"])
                self.win.append(s * vint // c["nshot"])
        if not c.get("uneven"):
            self.phys = [dims] * vint
        self.src, self.rec = [], []
        for s in range(c["nshot"]):
            p = self.phys[self.win[s]]
            wx, nrec = (p[-1] - 1) * h, c["nrec"]
            if c["kind"] == "timelapse":
                self.src.append([0.45 * wx, 0.0, rng.uniform(0.1, 0.9) * (p[0] - 1) * h])
                rec = np.zeros((nrec, 3))
                rec[:, 0] = 0.6 * wx
                rec[:, 2] = np.linspace(0.05, 0.95, nrec) * (p[0] - 1) * h
            elif self.nd == 2:
                self.src.append([(s + rng.uniform(0.3, 0.7)) * wx / c["nshot"], 0.0, 2 * h])
                rec = np.zeros((min(nrec, p[-1]), 3))
                rec[:, 0] = np.floor(np.linspace(0, p[-1] - 1, len(rec))) * h
                rec[:, 2] = 2 * h
            else:
                wy = (p[1] - 1) * h
                self.src.append([rng.uniform(0.4, 0.6) * wx, rng.uniform(0.4, 0.6) * wy, 2 * h])
                n = max(2, int(math.sqrt(nrec)))
                X, Y = np.meshgrid(np.linspace(0.05, 0.95, n) * wx, np.linspace(0.05, 0.95, n) * wy)
                rec = np.zeros((n * n, 3))
                rec[:, 0], rec[:, 1], rec[:, 2] = X.ravel(), Y.ravel(), 2 * h
            self.rec.append(rec)
        base = [_velocity(p, gen) for p in (self.phys if c.get("uneven") else self.phys[:1])]
        if not c.get("uneven"):
            # vintages: a growing slow patch in the middle of the baseline
            z = torch.linspace(0, 1, dims[0], device="cuda").reshape([-1] + [1] * (self.nd - 1))
            x = torch.linspace(0, 1, dims[-1], device="cuda")
            base = [base[0] * (1 - 0.05 * i / max(vint, 1) * torch.exp(-40 * ((z - 0.6) ** 2 + (x - 0.5) ** 2)))
                    for i in range(vint)]
        self.v = base
        ext = [b if c["kind"] in ("autograd", "timelapse") else _pad(b, nbl) for b in base]
        self.q = torch.cat([_wavelet(n, self.dt) for n in self.nts])
        self.m = torch.cat([(1.0 / e.double() ** 2).float().reshape(-1) for e in ext])
        if c["kind"] in ("gradient", "probed", "autograd", "timelapse"):
            self.dd = torch.cat([_traces(n, len(r), self.dt, gen).reshape(-1) for n, r in zip(self.nts, self.rec)])
            if c["kind"] in ("autograd", "timelapse"):
                self.dd *= 0.02
        if c["kind"] == "born":
            self.dm = torch.cat([(0.02 * _smooth(e.shape, 16, gen)).reshape(-1) for e in ext])
        if c["kind"] == "probed":
            r = c["nprobe"]
            C = torch.where(torch.rand(r, c["nt"], generator=gen, device="cuda") < 0.5, -1.0, 1.0)
            C[:, 0] = 0
            self.C, self.s = C.contiguous(), np.full(r, 1.0 / r)

    def comp(self, w):
        return tuple(n + 2 * self.nbl for n in self.phys[w])

    def plan(self, storage):
        geoms = [A.ShotGeometry(self.win[s], self.nts[s], self.src[s], self.rec[s]) for s in range(self.c["nshot"])]
        return A.Plan(self.nd, self.h, self.dt, self.nbl, VMAX, [self.comp(w) for w in range(len(self.phys))], geoms,
                      storage=storage, damp_vref=VMAX, damp_R=DAMP_R)


def _storage(c):
    k = c["kind"]
    if k in ("gradient", "timelapse"):
        return A.Storage(A.STORE_FULL, 0, c.get("prec", 0))
    if k == "autograd":
        return A.Storage(A.STORE_CHECKPOINT, c["nslots"])
    if k == "probed":
        return A.Storage(A.STORE_PROBED, c["nprobe"])
    return A.Storage()


def _rock_inputs(c, seed):
    gen = _gen(seed)
    shape = _dims(c)
    sat = torch.stack([(_smooth(shape, 24, gen) * 0.7 + 0.3).clamp(0, 1) for _ in range(c["nvint"])])
    rock = []
    for lo, hi in ((3.1, 3.8), (2250.0, 2450.0), (0.20, 0.30)):
        f = lo + (hi - lo) * 0.5 * (1 + torch.tanh(_smooth(shape, 16, gen)))
        rock.append(f.expand(c["nvint"], *shape).contiguous())
    gv = torch.randn(sat.shape, generator=gen, device="cuda")
    gr = torch.randn(sat.shape, generator=gen, device="cuda") * 1e-3
    return sat.contiguous(), rock, gv, gr


def prepare(case, seed):
    if case["kind"] == "rock":
        sat, rock, gv, gr = _rock_inputs(case, seed)
        return dict(c=case, sat=sat.requires_grad_(True), rock=rock, g=[gv, gr])
    S = _Survey(case, seed)
    plan = S.plan(_storage(case))
    st = dict(c=case, plan=plan, q=S.q)
    if case["kind"] in ("autograd", "timelapse"):
        st["nbl"] = S.nbl
        st["d_obs"] = S.dd
        if case["kind"] == "timelapse":
            st["v"] = [v.clone().requires_grad_(True) for v in S.v]
        else:
            st["m_phys"] = S.m.reshape(S.phys[0]).clone().requires_grad_(True)
            m_ext = A.extend_edge(st["m_phys"].detach(), S.nbl).reshape(-1).contiguous()
    else:
        st["m"] = m_ext = S.m
        st["ws"] = plan.workspace()
    for k in ("dm", "C", "s") + (("dd",) if case["kind"] in ("gradient", "probed") else ()):
        if hasattr(S, k):
            st[k] = getattr(S, k)
    if case.get("tune"):
        plan.autotune(m_ext, S.q, getattr(S, "dd", None), probe_steps=24, ws=st.get("ws"))
    return st


def run(st):
    k = st["c"]["kind"]
    if k == "rock":
        st["sat"].grad = None
        vp, rho = A.patchy_rock_physics(st["sat"], *st["rock"])
        torch.autograd.backward([vp, rho], st["g"])
        return vp.detach(), rho.detach(), st["sat"].grad
    plan, q = st["plan"], st["q"]
    if k == "forward":
        return plan.forward(st["m"], q, ws=st["ws"])
    if k == "gradient":
        return plan.gradient(st["m"], q, st["dd"], v=True, d=True, ws=st["ws"])
    if k == "born":
        return plan.born(st["m"], q, st["dm"], ws=st["ws"])
    if k == "probed":
        return plan.gradient_probed(st["m"], q, st["dd"], st["C"], st["s"], d=True, ws=st["ws"])[::2]
    if k == "autograd":
        x = st["m_phys"]
        x.grad = None
        phi = A.misfit(A.wave_forward(A.extend_edge(x, st["nbl"]).reshape(-1), q, plan), st["d_obs"])
        phi.backward()
        return phi.detach(), x.grad
    for v in st["v"]:
        v.grad = None
    m = torch.cat([A.extend_edge(A.slowness2_from_velocity(v), st["nbl"]).reshape(-1) for v in st["v"]])
    phi = A.misfit(A.wave_forward(m, q, plan), st["d_obs"])
    phi.backward()
    return [phi.detach()] + [v.grad for v in st["v"]]


def _cells(c):
    if c["kind"] == "rock":
        return c["nvint"] * math.prod(_dims(c)), 1
    if c.get("uneven"):
        r = random.Random(1000 + c["nshot"])
        upd = pts = 0
        for _ in range(c["nshot"]):
            w = r.randint(min(256, max(8, c["nx"] // 2)), c["nx"])
            n = r.randint(max(2, int(0.4 * c["nt"])), c["nt"])
            p = (w + 2 * c["nbl"]) * (c["nz"] + 2 * c["nbl"])
            pts, upd = pts + p, upd + p * (n - 1)
        return pts, upd
    p = c["nshot"] * math.prod(n + 2 * c["nbl"] for n in _dims(c))
    return p, p * (c["nt"] - 1)


def work(case):
    """Stencil arithmetic per point and level; as memory traffic the model, the traces and the
    results once, the kept wavefield (FULL) once out and once in, the probe sums once."""
    pts, upd = _cells(case)
    k = case["kind"]
    if k == "rock":
        return {"bytes": pts * 4 * (4 + 2 + 4 + 2 + 1), "flops": pts * 60}
    per = 40 if len(_dims(case)) == 2 else 56
    data = 4 * case["nt"] * case["nshot"] * case["nrec"]
    grid = pts // case["nshot"] * case.get("nvint", 1) if not case.get("uneven") else pts
    nbytes, flops = 4 * grid + data, upd * per
    if k in ("gradient", "timelapse"):
        nbytes += 2 * upd * (2 if case.get("prec", 0) else 4) + data + 8 * grid
        flops = upd * (2 * per + 2)
    elif k == "autograd":
        nbytes += data + 8 * grid
        flops = upd * (2 * per + 2)
    elif k == "born":
        nbytes += 4 * grid
        flops = upd * (2 * per + 2)
    elif k == "probed":
        nbytes += data + 8 * grid + 2 * 8 * case["nprobe"] * pts
        flops = upd * (2 * per + 4 * case["nprobe"])
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------------------- FP64
_W = (-205.0 / 72.0, 8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0, -1.0 / 560.0)


def _band(n, h):
    B = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    for r, w in enumerate(_W):
        for s in {r, -r}:
            if abs(s) < n:
                B += torch.diag(torch.full((n - abs(s),), w / h ** 2, dtype=torch.float64, device="cuda"), s)
    return B


class _Wave64:
    """The discrete operators of one window for a batch of its shots, in FP64."""

    def __init__(self, S, w, shots, m):
        self.shape = S.comp(w)
        self.S, self.shots, self.nt, self.dt = S, shots, S.nts[shots[0]], S.dt
        h, nbl, nd = S.h, S.nbl, S.nd
        eta = torch.zeros(self.shape, dtype=torch.float64, device="cuda")
        amp = 3.0 * math.log(1.0 / DAMP_R) / (2.0 * nbl * h * VMAX)
        for ax, n in enumerate(self.shape):
            i = torch.arange(n, dtype=torch.float64, device="cuda")
            d = torch.clamp(torch.maximum(nbl - i, i - (n - 1 - nbl)), min=0.0) / nbl
            eta += (amp * d ** 2).reshape([-1 if a == ax else 1 for a in range(nd)])
        m = m.double().reshape(self.shape)
        dt = self.dt
        self.den = m / dt ** 2 + eta / (2 * dt)
        self.a1 = 2 * m / dt ** 2 / self.den
        self.a2 = -(m / dt ** 2 - eta / (2 * dt)) / self.den
        self.inv = 1.0 / self.den
        self.L = [_band(n, h) for n in self.shape]
        self.src = [self._interp([S.src[s]]) for s in shots]
        self.rec = [self._interp(S.rec[s]) for s in shots]

    def _interp(self, pos):
        """(flat node indices [n][2^d], weights) of the bi- / trilinear interpolation."""
        pos = np.asarray(pos, dtype=np.float64).reshape(-1, 3)
        axes = [2, 0] if len(self.shape) == 2 else [2, 1, 0]
        idx, wt = [np.zeros(len(pos), dtype=np.int64)], [np.ones(len(pos))]
        for ax, n in zip(axes, self.shape):
            g = pos[:, ax] / self.S.h + self.S.nbl
            b = np.floor(g).astype(np.int64)
            f = g - b
            idx, wt = ([i * n + np.minimum(b + o, n - 1) for i in idx for o in (0, 1)],
                       [x * (f if o else 1 - f) for x in wt for o in (0, 1)])
        return torch.from_numpy(np.stack(idx, 1)).cuda(), torch.from_numpy(np.stack(wt, 1)).cuda()

    def zeros(self):
        return torch.zeros((len(self.shots),) + self.shape, dtype=torch.float64, device="cuda")

    def lap(self, u):
        n = self.shape
        out = torch.matmul(u.reshape(-1, n[-1]), self.L[-1]).reshape(u.shape)
        b = len(self.shots)
        if len(n) == 3:
            out += torch.matmul(self.L[1], u.reshape(b * n[0], n[1], n[2])).reshape(u.shape)
        out += torch.matmul(self.L[0], u.reshape(b, n[0], -1)).reshape(u.shape)
        return out

    def step(self, u1, u2, s=None):
        x = self.lap(u1)
        if s is not None:
            x += s
        x *= self.inv
        x.addcmul_(self.a1, u1).addcmul_(self.a2, u2)
        return x

    def inject(self, x, ops, vals):
        for b, ((i, w), v) in enumerate(zip(ops, vals)):
            x[b].view(-1).index_add_(0, i.reshape(-1), (w * v.reshape(-1, 1)).reshape(-1))

    def sample(self, u, ops):
        return [(u[b].reshape(-1)[i] * w).sum(1) for b, (i, w) in enumerate(ops)]

    def forward(self, q, b_out=None, dm=None, C=None):
        """Traces per shot; with b_out the second differences, with dm the Born traces, with C
        the probe sums of the second differences."""
        S, hd = self.S, self.S.h ** self.S.nd
        u1, u2 = self.zeros(), self.zeros()
        if dm is not None:
            p1, p2 = self.zeros(), self.zeros()
        nd = [torch.zeros(self.nt, len(S.rec[s]), dtype=torch.float64, device="cuda") for s in self.shots]
        B = None if C is None else [self.zeros() for _ in range(len(C))]
        for k in range(1, self.nt):
            x = self.lap(u1)
            self.inject(x, self.src, [x_[k - 1:k] / hd for x_ in q])
            x *= self.inv
            x.addcmul_(self.a1, u1).addcmul_(self.a2, u2)
            if b_out is not None or dm is not None or C is not None:
                b = x - 2 * u1 + u2
                if b_out is not None:
                    b_out[k] = b
                if C is not None:
                    for j in range(len(C)):
                        B[j].add_(b, alpha=float(C[j][k]))
                if dm is not None:
                    y = self.step(p1, p2, -dm * b / self.dt ** 2)
                    p2, p1 = p1, y
            u2, u1 = u1, x
            for t, s in zip(nd, self.sample(u1 if dm is None else p1, self.rec)):
                t[k] = s
        return (nd, B) if C is not None else nd

    def adjoint(self, dd, b_in=None, C=None):
        """(sum over levels of w b per shot, F^T dd per shot, probe sums of w)."""
        S, hd = self.S, self.S.h ** self.S.nd
        w1, w2 = self.zeros(), self.zeros()
        acc = self.zeros()
        v = [torch.zeros(self.nt, dtype=torch.float64, device="cuda") for _ in self.shots]
        B = None if C is None else [self.zeros() for _ in range(len(C))]
        for j in range(self.nt - 1, 0, -1):
            x = self.lap(w1)
            self.inject(x, self.rec, [d[j] for d in dd])
            x *= self.inv
            x.addcmul_(self.a1, w1).addcmul_(self.a2, w2)
            w2, w1 = w1, x
            if b_in is not None:
                acc.addcmul_(w1, b_in[j])
            if C is not None:
                for p in range(len(C)):
                    B[p].add_(w1, alpha=float(C[p][j]))
            for t, s in zip(v, self.sample(w1, self.src)):
                t[j - 1] = s[0] / hd
        return acc, v, B


def exact(case, seed):
    """What run returns, in FP64."""
    if case["kind"] == "rock":
        sat, (vp, rho, phi), gv, gr = _rock_inputs(case, seed)
        s = sat.double().requires_grad_(True)
        vp, rho, phi = vp.double(), rho.double(), phi.double()
        km, kb, kc, rc, rb = 36.6e9, 2.735e9, 0.125e9, 700.0, 1000.0
        p1 = rho * (vp * 1e3) ** 2
        mu = p1 / 3
        k1 = p1 - 4 * mu / 3
        ratio = lambda k: k / (km - k)
        x = ratio(k1) - ratio(kb) / phi + ratio(kc) / phi
        p2 = x * km / (1 + x) + 4 * mu / 3
        M = 1.0 / ((1 - s) / p1 + s / p2)
        rn = rho + phi * s * (rc - rb)
        vn = torch.sqrt(M / rn) / 1e3
        torch.autograd.backward([vn, rn], [gv.double(), gr.double()])
        return vn.detach(), rn.detach(), s.grad
    S = _Survey(case, seed)
    c, kind = case, case["kind"]
    # seconds this takes, about: launches per window, level and shot, and the FP64 products
    pts, upd = _cells(c)
    both = 1 if kind in ("forward", "born") else 2
    levels = sum(S.nts) if c.get("uneven") else c["nt"] * len(S.phys)
    flop = 2 * upd * sum(n + 2 * c["nbl"] for n in _dims(c))
    if both * (3e-4 * levels + 6e-5 * sum(S.nts) + flop / 2e13) > 12 or \
            (kind in ("gradient", "autograd", "timelapse") and 8 * pts * c["nt"] > 120e9):
        return None
    if kind in ("autograd", "timelapse"):
        leaf = [v.double().requires_grad_(True) for v in S.v] if kind == "timelapse" else \
            [S.m.double().reshape(S.phys[0]).requires_grad_(True)]
        # the library rounds m to float32 once before the solve
        ms = [x.detach().float().double() + (x - x.detach()) for x in
              [_pad(1.0 / v ** 2 if kind == "timelapse" else v, S.nbl) for v in leaf]]
    else:
        off, ms = 0, []
        for w in range(len(S.phys)):
            n = math.prod(S.comp(w))
            ms.append(S.m[off:off + n].double().reshape(S.comp(w)))
            off += n
    qo = np.concatenate([[0], np.cumsum(S.nts)])
    do = np.concatenate([[0], np.cumsum([n * len(r) for n, r in zip(S.nts, S.rec)])])
    q = [S.q[qo[s]:qo[s + 1]].double() for s in range(c["nshot"])]
    dd = [S.dd[do[s]:do[s + 1]].double().reshape(S.nts[s], -1) if hasattr(S, "dd") else None for s in range(c["nshot"])]
    d_out, v_out = [None] * c["nshot"], [None] * c["nshot"]
    g_out = [torch.zeros(S.comp(w), dtype=torch.float64, device="cuda") for w in range(len(S.phys))]
    phi = torch.zeros((), dtype=torch.float64, device="cuda")
    for w in range(len(S.phys)):
        shots = [s for s in range(c["nshot"]) if S.win[s] == w]
        if not shots:
            continue
        op = _Wave64(S, w, shots, ms[w].detach())
        qs, ds = [q[s] for s in shots], [dd[s] for s in shots]
        if kind == "forward":
            out = op.forward(qs)
        elif kind == "born":
            out = op.forward(qs, dm=S.dm.double().reshape(S.comp(w)))
        elif kind == "probed":
            out, B = op.forward(qs, C=S.C.cpu().numpy())
            _, _, W = op.adjoint(ds, C=S.C.cpu().numpy())
            for j in range(len(S.s)):
                g_out[w] -= S.s[j] * (W[j] * B[j]).sum(0) / S.dt ** 2
        else:
            b = torch.zeros((op.nt,) + tuple(op.zeros().shape), dtype=torch.float64, device="cuda")
            out = op.forward(qs, b_out=b)
            if kind in ("autograd", "timelapse"):
                ds = [o - d for o, d in zip(out, ds)]
                phi += sum(0.5 * (r ** 2).sum() for r in ds)
            acc, v, _ = op.adjoint(ds, b_in=b)
            g_out[w] -= acc.sum(0) / S.dt ** 2
            for s, x in zip(shots, v):
                v_out[s] = x
        for s, x in zip(shots, out):
            d_out[s] = x.reshape(-1)
    d = torch.cat(d_out)
    if kind in ("forward", "born"):
        return d
    g = torch.cat([x.reshape(-1) for x in g_out])
    if kind == "gradient":
        return g, torch.cat(v_out), d
    if kind == "probed":
        return g, d
    torch.autograd.backward(ms, g_out)
    return (phi, leaf[0].grad) if kind == "autograd" else [phi] + [x.grad for x in leaf]
