"""Workloads on which this framework's speed is measured.

Each case is one call that a flow solver or a solve service makes: a direct
Poisson or Helmholtz solve in place (FP64, or FP32 with FP64 refinement), a
batch of independent solves, a stream of requests to the server, a
pressure-correction step, a whole Runge-Kutta time step.  Sizes, boundary pairs
and stretching are those of the paper's validation cases (Table 3), of the
benchmark and of the served and batched mixes in ``inputs``.

The solves work in place, so a second pass on a state solves for the first
pass's result.  Boxes are therefore scaled so that the smallest eigenvalue of
the operator (in modulus, the null space aside) is 1: the field keeps its size
over any number of passes.
"""
import math
import random

import numpy as np
import torch

from paper_1802_10323_amd import poisson
from paper_1802_10323_amd.inputs import BATCH_SIZES, BC_NAMES, Problem, smooth_sizes, tanh_widths, uniform_widths

BETA = 1.8                                   # tanh clustering toward both walls
ALPHA = (8.0 / 15.0, 5.0 / 12.0, 3.0 / 4.0)  # Runge-Kutta coefficients, Eq. (up)
RKBETA = (0.0, -17.0 / 60.0, -5.0 / 12.0)


def listed():
    return [
        # a call so small that launches and latency are all of it
        dict(name="solve small 32", kind="solve", nx=32, ny=32, nz=32, bcs="P,P,NN",
             stretch=False, box="unit", refined=False),
        # lid-driven cavity (Table 3): walls on every side, singular, an ordinary small 3D run
        dict(name="solve cavity 128", kind="solve", nx=128, ny=128, nz=128, bcs="NN,NN,NN",
             stretch=False, box="unit", refined=False),
        # plane channel (Table 3): the solve of a wall-turbulence run, 144 stretched cells between the walls
        dict(name="solve channel 512x256x144", kind="solve", nx=512, ny=256, nz=144, bcs="P,P,NN",
             stretch=True, box="channel", refined=False),
        # lengths with factors 3 and 5, as a user picks them by resolution and not by power of two
        dict(name="solve ragged 270x150x162", kind="solve", nx=270, ny=150, nz=162, bcs="NN,P,ND",
             stretch=True, box="unit", refined=False),
        # the benchmark's cube: the elimination along x, both transforms along strided axes
        dict(name="solve cube 512", kind="solve", nx=512, ny=512, nz=512, bcs="DD,ND,P",
             stretch=False, box="unit", refined=False),
        # a finer channel, up to the longest transforms: the largest solve
        dict(name="solve channel 1024x640x320", kind="solve", nx=1024, ny=640, nz=320, bcs="P,P,NN",
             stretch=True, box="channel", refined=False),
        # the mixed-precision option on the benchmark's channel
        dict(name="refined channel 512x256x192", kind="solve", nx=512, ny=256, nz=192, bcs="P,P,NN",
             stretch=True, box="channel", refined=True),
        # implicit diffusion of a channel's wall-normal velocity: unknowns on the 191 inner nodes
        dict(name="helmholtz 512x256x191", kind="helmholtz", nx=512, ny=256, nz=191, bcs="P,P,DDn",
             stretch=False, box="channel", refined=False),
        # many independent uneven problems in one persistent launch, replayed as a graph
        dict(name="batch of 32", kind="batch", count=32, mix=0, refined=False),
        # a burst of requests of all sizes, pairs and both precisions to the solve server
        dict(name="served burst of 40", kind="served", count=40, mix=0),
        # the square duct (Table 3) with the steps around the solve
        dict(name="correction duct 512x128x128", kind="correction", nx=512, ny=128, nz=128,
             bcs="P,NN,NN", stretch=False, box="unit"),
        # Taylor-Green vortex (Table 3): one whole time step, the largest call
        dict(name="step vortex 512", kind="step", nx=512, ny=512, nz=512),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _smooth(rng, lo, hi):
    sizes = smooth_sizes(lo, hi)
    x = _log_uniform(rng, lo, hi)
    return min(sizes, key=lambda s: (abs(s - x), s))


def draw(rng):
    """One more case: any smooth transformed lengths up to 1024, any
    elimination length up to 512, every boundary pair and option."""
    kind = rng.choice(("solve", "solve", "solve", "solve", "helmholtz", "batch", "served",
                       "correction", "step"))
    if kind in ("batch", "served"):
        case = dict(kind=kind, count=rng.randint(4, 32), mix=rng.randint(1, 10 ** 6))
        if kind == "batch":
            case["refined"] = rng.random() < 0.3
        return case
    if kind == "step":
        while True:
            n = [_smooth(rng, 48, 512) for _ in range(3)]
            if n[0] * n[1] * n[2] <= 1 << 26:
                return dict(kind=kind, nx=n[0], ny=n[1], nz=n[2])
    names = BC_NAMES if kind != "correction" else ("P", "NN", "NN", "ND")
    while True:
        bcs = [rng.choice(names) for _ in range(3)]
        if rng.random() < 0.5:               # channel-like: the commonest runs
            bcs = ["P", "P", "NN"]
        stretch = kind != "helmholtz" and bcs[2] != "P" and rng.random() < 0.5
        if kind == "helmholtz":
            bcs[rng.randrange(3)] = rng.choice(("DDn", "DD", "NN"))
        nx, ny = _smooth(rng, 24, 1024), _smooth(rng, 24, 1024)
        nz = round(_log_uniform(rng, 24, 512))
        # the axes that the plan transforms need smooth lengths; the others are free
        if bcs[2] == "P" and not stretch:
            nz = _smooth(rng, 24, 512)
        if bcs[2] == "P" and (bcs[0] != "P" or bcs[1] == "P") and nx > 512:
            continue
        if bcs[2] == "P" and bcs[0] == "P" and bcs[1] != "P" and ny > 512:
            continue
        dims = (nx, ny, nz)
        sizes = smooth_sizes(2, 1024)
        for a in (0, 1, 2):
            if bcs[a] == "DDn" and a != 2:
                n = min(sizes, key=lambda s: abs(s - 2 * (dims[a] + 1))) // 2 - 1
                dims = dims[:a] + (n,) + dims[a + 1:]
        if dims[0] * dims[1] * dims[2] > 1 << 26 or dims[0] * dims[1] * dims[2] < 20000:
            continue
        case = dict(kind=kind, nx=dims[0], ny=dims[1], nz=dims[2], bcs=",".join(bcs), stretch=stretch,
                    box=rng.choice(("unit", "channel")))
        if kind != "correction":
            case["refined"] = rng.random() < 0.3
        return case


# ---- grids ----

def _lowest(bc, n, h):
    """Smallest and smallest non-zero eigenvalue (modulus) of one uniform axis."""
    length = n * h
    k0, k1 = {"P": (0.0, 2 * math.pi / length), "NN": (0.0, math.pi / length),
              "DD": (math.pi / length,) * 2, "ND": (0.5 * math.pi / length,) * 2,
              "DN": (0.5 * math.pi / length,) * 2, "DDn": (math.pi / (length + h),) * 2,
              "NNn": (0.0, math.pi / max(length - h, h))}[bc]
    return tuple(4.0 / (h * h) * math.sin(min(0.5 * k * h, 0.5 * math.pi)) ** 2 for k in (k0, k1))


def _problem(nx, ny, nz, bcs, stretch, box, shift=0.0):
    """The grid of a case, scaled so that the operator's smallest eigenvalue is 1."""
    dims, lengths = (nx, ny, nz), (4 * math.pi, 2 * math.pi, 2.0) if box == "channel" else (1.0, 1.0, 1.0)
    low = [_lowest(b, n, length / n) for b, n, length in zip(bcs, dims, lengths)]
    least = sum(a for a, _ in low) + shift
    if least < 1e-9:
        least = min(b for _, b in low)
    s = math.sqrt(least)
    hz = tanh_widths(nz, s * lengths[2], BETA) if stretch else uniform_widths(nz, s * lengths[2])
    prob = Problem(uniform_widths(nx, s * lengths[0]), uniform_widths(ny, s * lengths[1]), hz, *bcs, None)
    prob.shift = -shift / least
    return prob


def _of_case(case):
    """The problems of a case, in order."""
    if case["kind"] == "step":
        return [Problem(*(uniform_widths(case[k], 2 * math.pi) for k in ("nx", "ny", "nz")), "P", "P", "P", None)]
    if case["kind"] in ("batch", "served"):
        rng, out = random.Random(1000 + case["mix"]), []
        while len(out) < case["count"]:
            if case["kind"] == "batch":
                dims = [rng.choice(BATCH_SIZES) for _ in range(3)]
            else:
                dims = [_smooth(rng, 32, 512) for _ in range(3)]
            if dims[0] * dims[1] * dims[2] > 1 << 24:
                continue
            bcs = [rng.choice(BC_NAMES) for _ in range(3)]
            out.append(_problem(*dims, bcs, bcs[2] != "P" and rng.random() < 0.5, "unit"))
            out[-1].mixed = rng.random() < 0.5
        return out
    bcs = case["bcs"].split(",")
    shift = 20000.0 if case["kind"] == "helmholtz" else 0.0   # 2 / (nu dt) of a channel step
    return [_problem(case["nx"], case["ny"], case["nz"], bcs, case["stretch"], case["box"], shift)]


def _inputs(case, seed):
    """The fields of a case, made from the seed alone."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))

    def uniform(shape):
        return torch.rand(shape, generator=gen, device=dev, dtype=torch.float64).mul_(2.0).sub_(1.0)

    probs = _of_case(case)
    p = probs[0]
    if case["kind"] == "step":
        # Taylor-Green vortex in a flow of a little noise: u = sin x cos y cos z, v = -cos x sin y cos z
        face = [torch.arange(n, device=dev, dtype=torch.float64) * (2 * math.pi / n) for n in (p.nx, p.ny, p.nz)]
        mid = [f + math.pi / n for f, n in zip(face, (p.nx, p.ny, p.nz))]

        def outer(x, y, z):
            return z[:, None, None] * y[None, :, None] * x[None, None, :]

        vel = torch.zeros((3,) + p.shape, device=dev, dtype=torch.float64)
        vel[0] = outer(torch.sin(face[0]), torch.cos(mid[1]), torch.cos(mid[2]))
        vel[1] = outer(torch.cos(mid[0]), -torch.sin(face[1]), torch.cos(mid[2]))
        for c in range(3):
            vel[c] += 1e-2 * uniform(p.shape)
        pr = (torch.cos(2 * mid[0])[None, None, :] + torch.cos(2 * mid[1])[None, :, None]) \
            * ((torch.cos(2 * mid[2]) + 2.0) / 16.0)[:, None, None]
        return vel, pr
    if case["kind"] == "correction":
        vel = []
        for axis, bc in ((2, p.bcx), (1, p.bcy), (0, p.bcz)):
            shape = list(p.shape)
            shape[axis] += bc != "P"
            t = uniform(shape)
            if bc[0] == "N":
                t.select(axis, 0).zero_()
            if bc[-1] == "N":
                t.select(axis, shape[axis] - 1).zero_()
            vel.append(t)
        return vel, uniform(p.shape)
    return [uniform(q.shape) for q in probs]


# ---- the calls ----

def prepare(case, seed):
    """Inputs on the GPU, and the plan, batch or server that a program keeps."""
    kind, probs, data = case["kind"], _of_case(case), _inputs(case, seed)
    if kind == "served":
        return dict(kind=kind, server=poisson.Server(slots=8), problems=probs, fields=data)
    plans = [poisson.Plan.from_problem(p) for p in probs]
    if case.get("refined"):
        for p in plans:
            p.set_precision(poisson.FP32_REFINED)
    state = dict(kind=kind, plan=plans[0])
    if kind == "batch":
        state.update(batch=poisson.Batch(plans), fields=data)
        state["batch"].bind(data)
    elif kind == "correction":
        state.update(vel=data[0], p=data[1], phi=torch.empty_like(data[1]), gamma_dt=1e-3)
    elif kind == "step":
        p = probs[0]
        vel, pr = data
        n = pr.numel()
        new = lambda k: torch.empty(k * n, device=pr.device, dtype=torch.float64)  # noqa: E731
        state.update(vel=vel, p=pr, phi=torch.empty_like(pr), work=new(3), ad=new(6), scratch=new(2),
                     **_time_step(p))
    else:
        state["field"] = data[0]
    return state


def _time_step(p):
    h = min(p.dx, p.dy, float(p.hz[0]))
    return dict(dt=min(0.3 * h, 0.1 * h * h * 1600.0), nu=1.0 / 1600.0)


def run(state):
    kind = state["kind"]
    if kind in ("solve", "helmholtz"):
        return state["plan"].solve(state["field"])
    if kind == "batch":
        state["batch"].launch(graph=True)
        return state["fields"]
    if kind == "served":
        server = state["server"]
        ids = [server.submit(p, f, precision=poisson.FP32_REFINED if p.mixed else poisson.FP64)
               for p, f in zip(state["problems"], state["fields"])]
        for i in ids:
            server.wait(i)
        return state["fields"]
    if kind == "correction":
        state["plan"].pressure_correction(*state["vel"], state["p"], state["gamma_dt"], state["phi"])
        return dict(u=state["vel"][0], v=state["vel"][1], w=state["vel"][2], p=state["p"], phi=state["phi"])
    state["plan"].rk3_step(state["dt"], state["nu"], state["vel"], state["work"], state["ad"], state["p"],
                           state["phi"], state["scratch"])
    return dict(vel=state["vel"], p=state["p"], phi=state["phi"])


def work(case):
    """Each input read once and each output written once; the transforms at
    2.5 log2 n operations a point and direction, the elimination at 10."""
    nbytes = flops = 0.0
    for p in _of_case(case):
        axes = sorted((p.nx, p.ny, p.nz))
        solve = p.points * (5.0 * (math.log2(axes[2]) + math.log2(axes[1])) + 10.0)
        if case["kind"] == "correction":     # u, v, w, p read and written, phi written
            nbytes, flops = nbytes + 72.0 * p.points, flops + solve + 20.0 * p.points
        elif case["kind"] == "step":         # the same fields; three predictions and solves
            nbytes, flops = nbytes + 72.0 * p.points, flops + 3 * (solve + 200.0 * p.points)
        else:
            nbytes, flops = nbytes + 16.0 * p.points, flops + solve
    return {"bytes": nbytes, "flops": flops}


# ---- the same results from dense linear algebra ----

def _rows(bc, h):
    """Lower, middle and upper entries of one axis of the operator, and the
    weights that make it symmetric."""
    n, h = len(h), np.asarray(h, dtype=np.float64)
    if bc in ("DDn", "NNn"):
        a, c, w = np.full(n, h[0] ** -2.0), np.full(n, h[0] ** -2.0), np.ones(n)
        b = -(a + c)
        if bc == "NNn" and n > 1:
            c[0], a[-1], w[0], w[-1] = 2 * c[0], 2 * a[-1], 0.5, 0.5
        a[0] = c[-1] = 0.0
        return a, b, c, w
    gap = 0.5 * (h[1:] + h[:-1])
    wrap = 0.5 * (h[0] + h[-1])
    below = np.concatenate([[wrap if bc == "P" else h[0]], gap])
    above = np.concatenate([gap, [wrap if bc == "P" else h[-1]]])
    a, c = 1.0 / (h * below), 1.0 / (h * above)
    b = -(a + c)
    if bc != "P":
        b[0] += a[0] if bc[0] == "N" else -a[0]
        b[-1] += c[-1] if bc[1] == "N" else -c[-1]
        a[0] = c[-1] = 0.0
    return a, b, c, h.copy()


class _Dense:
    """(A + shift) Phi = f in the eigenvectors of each axis, with one
    correction by the residual."""

    def __init__(self, p, dev):
        self.shift = getattr(p, "shift", 0.0)
        self.rows, self.to, self.back, values = [], [], [], []
        for bc, h in ((p.bcx, p.hx), (p.bcy, p.hy), (p.bcz, p.hz)):
            a, b, c, w = _rows(bc, h)
            n = len(b)
            m = np.diag(b)
            for k in range(n):               # += : a short periodic axis meets a neighbour twice
                m[k, (k - 1) % n] += a[k]
                m[k, (k + 1) % n] += c[k]
            r = np.sqrt(w)
            m = r[:, None] * m / r[None, :]
            lam, q = np.linalg.eigh(0.5 * (m + m.T))
            values.append(torch.from_numpy(lam).to(dev))
            self.to.append(torch.from_numpy(np.ascontiguousarray(r[:, None] * q)).to(dev))
            self.back.append(torch.from_numpy(np.ascontiguousarray(q.T / r[None, :])).to(dev))
            self.rows.append([torch.from_numpy(v).to(dev) for v in (a, b, c)])
        self.lam = values
        self.singular = self.shift == 0.0 and all(b in ("P", "NN", "NNn") for b in p.bcs)
        self.w = [torch.from_numpy(_rows(bc, h)[3]).to(dev) for bc, h in ((p.bcx, p.hx), (p.bcy, p.hy), (p.bcz, p.hz))]

    def _apply(self, f, mats):
        nz, ny, nx = f.shape
        f = (f.reshape(-1, nx) @ mats[0]).reshape(nz, ny, nx)
        f = f.transpose(1, 2).contiguous()
        f = (f.reshape(-1, ny) @ mats[1]).reshape(nz, nx, ny).transpose(1, 2).contiguous()
        return (mats[2].t().contiguous() @ f.reshape(nz, -1)).reshape(nz, ny, nx)

    def _centred(self, f):
        if not self.singular:
            return f
        m = f @ self.w[0] @ self.w[1] @ self.w[2]
        return f - m / (self.w[0].sum() * self.w[1].sum() * self.w[2].sum())

    def _once(self, f):
        g = self._apply(f, self.to)
        lam = self.lam[2][:, None, None] + self.lam[1][None, :, None] + self.lam[0][None, None, :] + self.shift
        g /= lam
        if self.singular:
            g[-1, -1, -1] = 0.0              # eigenvalues ascend: the null vector is the last
        return self._apply(g, self.back)

    def residual(self, phi, f):
        r = f - self.shift * phi
        for axis, (a, b, c) in zip((2, 1, 0), self.rows):
            s = [None, None, None]
            s[axis] = slice(None)
            r -= a[tuple(s)] * torch.roll(phi, 1, axis)
            r -= b[tuple(s)] * phi
            r -= c[tuple(s)] * torch.roll(phi, -1, axis)
        return r

    def solve(self, f):
        f = self._centred(f)
        phi = self._once(f)
        phi += self._once(self._centred(self.residual(phi, f)))
        return self._centred(phi)


def _exact_correction(p, vel, pr, gamma_dt, dev):
    axes = ((2, p.bcx, p.hx), (1, p.bcy, p.hy), (0, p.bcz, p.hz))
    div = torch.zeros_like(pr)
    for t, (axis, bc, h) in zip(vel, axes):
        n, shape = len(h), [1, 1, 1]
        shape[axis] = n
        up = torch.roll(t, -1, axis) if bc == "P" else t.narrow(axis, 1, n)
        div += (up - t.narrow(axis, 0, n)) / torch.from_numpy(h).to(dev).reshape(shape)
    phi = _Dense(p, dev).solve(div / gamma_dt)
    out = []
    for t, (axis, bc, h) in zip(vel, axes):
        n, shape = len(h), [1, 1, 1]
        gap = torch.from_numpy(0.5 * (h + np.roll(h, 1))).to(dev)
        shape[axis] = n
        grad = (phi - torch.roll(phi, 1, axis)) / gap.reshape(shape)
        if bc != "P":                        # walls: the ghost rules of the solve
            lo, hi = phi.narrow(axis, 0, 1), phi.narrow(axis, n - 1, 1)
            first = torch.zeros_like(lo) if bc[0] == "N" else 2.0 * lo / h[0]
            last = torch.zeros_like(hi) if bc[1] == "N" else -2.0 * hi / h[-1]
            grad = torch.cat([first, grad.narrow(axis, 1, n - 1), last], axis)
        out.append(t - gamma_dt * grad)
    return dict(u=out[0], v=out[1], w=out[2], p=pr + phi, phi=phi)


def _exact_step(p, vel, pr, dt, nu, dev):
    h = {2: p.dx, 1: p.dy, 0: float(p.hz[0])}
    axis_of = (2, 1, 0)                      # component -> array axis
    dense = _Dense(p, dev)
    u, before = [vel[c] for c in range(3)], None
    lo = lambda t, ax: torch.roll(t, 1, ax)   # noqa: E731  value at index - 1
    hi = lambda t, ax: torch.roll(t, -1, ax)  # noqa: E731  value at index + 1

    def rate(c):
        ax, ad = axis_of[c], None
        sq = (0.5 * (u[c] + hi(u[c], ax))) ** 2
        ad = -(sq - lo(sq, ax)) / h[ax]
        for d in range(3):
            e = axis_of[d]
            if d != c:
                cross = 0.25 * (u[c] + lo(u[c], e)) * (u[d] + lo(u[d], ax))
                ad -= (hi(cross, e) - cross) / h[e]
            ad += nu * (hi(u[c], e) - 2.0 * u[c] + lo(u[c], e)) / (h[e] * h[e])
        return ad

    for k in range(3):
        gamma = ALPHA[k] + RKBETA[k]
        ads = [rate(c) for c in range(3)]
        star = []
        for c in range(3):
            ax = axis_of[c]
            t = u[c] + dt * (ALPHA[k] * ads[c] - gamma * (pr - lo(pr, ax)) / h[ax])
            star.append(t if before is None else t + dt * RKBETA[k] * before[c])
        div = sum((hi(star[c], axis_of[c]) - star[c]) / h[axis_of[c]] for c in range(3))
        phi = dense.solve(div / (gamma * dt))
        u = [star[c] - gamma * dt * (phi - lo(phi, axis_of[c])) / h[axis_of[c]] for c in range(3)]
        pr, before = pr + phi, ads
    return dict(vel=torch.stack(u), p=pr, phi=phi)


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    probs, data = _of_case(case), _inputs(case, seed)
    if case["kind"] == "step":
        t = _time_step(probs[0])
        return _exact_step(probs[0], *data, t["dt"], t["nu"], dev)
    if case["kind"] == "correction":
        return _exact_correction(probs[0], *data, 1e-3, dev)
    out = [_Dense(p, dev).solve(f) for p, f in zip(probs, data)]
    return out if case["kind"] in ("batch", "served") else out[0]
