"""Performance cases of the RD3Q41 library: what its users run, over the sizes,
storage forms, models and directions that they run it with.

A case is one pass of a user's loop: a few time steps of a flow held in a
context (with the diagnostics that such a loop reads), building a context from
node fields on the device, or writing a state out. The held state is returned as
it lies in the context's workspace, [q][node] in the stored type, one view per
velocity shell; diagnostics as the calls return them. `exact` is the same pass in
64 bits, in plain torch.
"""
import itertools
import math

import numpy as np
import torch

from paper_1909_08406_amd import lbm, workloads

TWO_PI = 2.0 * math.pi
DTYPES = {"f64": torch.float64, "f32": torch.float32, "f32s": torch.float32, "f16s": torch.float16,
          "bf16s": torch.bfloat16}


def _case(name, kind, flow, dims, storage, steps, tau=0.6, sr=False, model="e2", entropic=False, walls=False,
          monitor="none", graph=0, boxes=1):
    nx, ny, nz = dims
    c = {"kind": kind, "flow": flow, "nx": nx, "ny": ny, "nz": nz, "storage": storage, "steps": steps, "tau": tau,
         "sr": sr, "model": model, "entropic": entropic, "walls": walls, "monitor": monitor, "graph": graph,
         "boxes": boxes}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: four steps of the 32x16x16 acoustic wave of the parity
        # tests, in the reference precision; a caller that couples every few steps
        _case("wave_f64_32x16x16", "step", "wave", (32, 16, 16), "f64", 4),
        # thermal-mode decay, 128^3 FP32 with stochastic rounding; the mode's
        # amplitude is read every ten steps
        _case("thermal_f32sr_128", "step", "thermal", (128, 128, 128), "f32", 10, sr=True, monitor="project"),
        # Taylor-Green vortex, 256^3 FP32, conservation totals read every ten steps
        _case("taylor_green_f32_256", "step", "taylor_green", (256, 256, 256), "f32", 10, tau=0.51211,
              monitor="totals"),
        # the largest: the 512^3 acoustic pulse in the benchmarked form
        _case("pulse_f16s_sr_512", "step", "pulse", (512, 512, 512), "f16s", 2, sr=True),
        # 256 uneven boxes in one context, steps replayed from a captured graph
        _case("batch256_f16s_sr", "step", "batch", (0, 0, 0), "f16s", 10, sr=True, graph=10, boxes=256),
        # the isothermal 2D pulse on 800 x 800 x 1 cells
        _case("pulse2d_f32s_iso_800", "step", "pulse", (800, 800, 1), "f32s", 10, tau=0.51, model="iso"),
        # Couette flow with viscous heating between a resting and a moving wall
        _case("couette_f32_walls_128", "step", "couette", (128, 128, 128), "f32", 10, tau=0.8, walls=True),
        # under-resolved Kida-Peltz turbulence with the entropic path length
        _case("kida_f16s_sr_entropic_128", "step", "kida", (128, 128, 128), "f16s", 10, tau=0.5005, sr=True,
              entropic=True),
        # the series equilibrium on a box with no round edge, BF16
        _case("wave_bf16s_sr_series_ragged", "step", "wave", (251, 183, 130), "bf16s", 5, sr=True, model="series"),
        # the FP64 reference run of the pulse
        _case("pulse_f64_192", "step", "pulse", (192, 192, 192), "f64", 4),
        # building a context from node fields on the device (encoding)
        _case("init_f16s_160", "init", "taylor_green", (160, 160, 160), "f16s", 0),
        # writing a run out: node moments, then the populations as a checkpoint and back (decoding)
        _case("output_f32_64", "output", "taylor_green", (64, 64, 64), "f32", 0),
    ]


def draw(rng):
    """One more case: sizes over the logarithm of the cell count, edges of any parity."""
    kind = rng.choice(["step"] * 8 + ["init", "output"])
    storage, sr = rng.choice([("f64", False), ("f32", False), ("f32", True), ("f32s", False), ("f16s", False),
                              ("f16s", True), ("f16s", True), ("bf16s", False), ("bf16s", True)])
    model, entropic, walls = rng.choice([("e2", False, False)] * 5 + [("iso", False, False), ("series", False, False),
                                        ("e2", True, False), ("e2", False, True), ("iso", False, True)])
    top = {"step": 24.0 if storage == "f64" else 25.0, "init": 23.0, "output": 19.0}[kind]
    cells = 2.0 ** rng.uniform(12.0, top)
    if rng.random() < 0.2:  # one cell deep
        a = 2.0 ** rng.uniform(-1.0, 1.0)
        dims = (max(4, round(math.sqrt(cells) * a)), max(4, round(math.sqrt(cells) / a)), 1)
    else:
        e = [2.0 ** rng.uniform(-0.7, 0.7) for _ in range(3)]
        s = (cells / (e[0] * e[1] * e[2])) ** (1.0 / 3.0)
        dims = tuple(max(4, round(s * v)) for v in e)
        if rng.random() < 0.3:  # rows of whole wavefronts, as powers of two give
            dims = (max(64, 64 * round(dims[0] / 64)),) + dims[1:]
    n = 2 * dims[0] * dims[1] * dims[2]
    steps = 0 if kind != "step" else max(1, min(20, int(4.0e7 / n))) if n > 1 << 20 else rng.choice([1, 2, 10, 20])
    flow = "couette" if walls else rng.choice(["wave", "thermal", "taylor_green", "pulse"])
    monitor = rng.choice(["none", "none", "totals", "project"]) if kind == "step" else "none"
    if kind == "step" and rng.random() < 0.15 and model == "e2" and not (entropic or walls):
        return _case(None, "step", "batch", (0, 0, 0), storage, rng.choice([2, 6, 10]), sr=sr, monitor="none",
                     graph=0, boxes=rng.randint(8, 200))
    return _case(None, kind, flow, dims, storage, steps, round(rng.uniform(0.52, 1.0), 4), sr, model, entropic, walls,
                 monitor)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _shapes(case):
    """[(nx, ny, nz, tau)] of the boxes of a case."""
    if case["flow"] == "batch":
        return [(b.nx, b.ny, b.nz, b.tau) for b in workloads.batch_specs(case["boxes"])]
    return [(case["nx"], case["ny"], case["nz"], case["tau"])]


def _axis(n, axis, half, device):
    """Node positions along one axis, shaped to broadcast over [s][z][y][x]."""
    p = torch.arange(n, dtype=torch.float64, device=device).reshape(1, n) + half.reshape(2, 1)
    return p.reshape({0: (2, 1, 1, n), 1: (2, 1, n, 1), 2: (2, n, 1, 1)}[axis])


def _fields(flow, nx, ny, nz, gen, theta0, spec=None):
    """rho, ux, uy, uz, theta as flat FP64 tensors in [s][z][y][x] order; phases,
    centres and noise are drawn from gen."""
    dev = gen.device
    shape = (2, nz, ny, nx)
    half = torch.tensor([0.0, 0.5], dtype=torch.float64, device=dev)
    off = torch.rand(3, dtype=torch.float64, generator=gen, device=dev)
    x, y, z = (_axis(n, a, half, dev) for a, n in enumerate((nx, ny, nz)))
    X, Y, Z = (TWO_PI * (p / n + o) for p, n, o in zip((x, y, z), (nx, ny, nz), off))
    full = lambda v: torch.full(shape, v, dtype=torch.float64, device=dev)  # noqa: E731
    rho, ux, uy, uz, th = full(1.0), full(0.0), full(0.0), full(0.0), full(1.0)
    if flow == "wave":
        rho += 1e-3 * torch.sin(X)
    elif flow == "batch":
        rho += spec.amp * torch.sin(spec.k * X)
    elif flow == "thermal":
        th += 1e-3 * torch.cos(Z)
        rho += 1e-4 * (2.0 * torch.rand(shape, dtype=torch.float64, generator=gen, device=dev) - 1.0)
    elif flow == "taylor_green":
        u0 = 0.1 * math.sqrt(5.0 / 3.0 * theta0)
        ux += u0 * torch.sin(X) * torch.cos(Y) * torch.cos(Z)
        uy -= u0 * torch.cos(X) * torch.sin(Y) * torch.cos(Z)
    elif flow == "kida":
        u0 = 0.3 * math.sqrt(5.0 / 3.0 * theta0)
        s, c, c3 = torch.sin, torch.cos, lambda p: torch.cos(3 * p)
        ux += u0 * s(X) * (c3(Y) * c(Z) - c(Y) * c3(Z))
        uy += u0 * s(Y) * (c3(Z) * c(X) - c(Z) * c3(X))
        uz += u0 * s(Z) * (c3(X) * c(Y) - c(X) * c3(Y))
    elif flow == "pulse":
        # Gaussian density bump around a drawn centre, minimum image
        b, g = max(2.0, min(8.0, min(v for v in (nx, ny, nz) if v > 1) / 8.0)), full(1.0)
        for p, n, o in zip((x, y, z), (nx, ny, nz), off):
            if n > 1:
                d = p - n * o
                g *= torch.exp(-math.log(2.0) * ((d - n * torch.round(d / n)) / b) ** 2)
        rho += 1e-3 * g
    elif flow == "couette":
        eta = (y + 0.25) / ny
        ux += 0.1 * eta
        th += 0.02 * eta
        rho += 1e-4 * (2.0 * torch.rand(shape, dtype=torch.float64, generator=gen, device=dev) - 1.0)
    else:
        raise ValueError(flow)
    return [t.reshape(-1) for t in (rho, ux, uy, uz, th.mul_(theta0))]


WALL_U, WALL_THETA = 0.1, 1.02  # the moving upper wall: velocity, temperature over theta0


def _all_fields(case, seed, theta0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * int(seed) + 17)
    if case["flow"] != "batch":
        return _fields(case["flow"], case["nx"], case["ny"], case["nz"], gen, theta0)
    parts = [_fields("batch", b.nx, b.ny, b.nz, gen, theta0, b) for b in workloads.batch_specs(case["boxes"])]
    return [torch.cat(p) for p in zip(*parts)]


def _options(case, seed):
    return dict(storage=case["storage"], stochastic=case["sr"], seed=seed, isothermal=case["model"] == "iso",
                series=case["model"] == "series", entropic=case["entropic"], walls=case["walls"])


# ---------------------------------------------------------------------------
# The pass
# ---------------------------------------------------------------------------
SHELL_COUNTS = (1, 6, 6, 12, 8, 8)


def _stride(nodes, eb):
    """Elements from one q-block of a box to the next in a population buffer."""
    nbytes = (nodes * eb + 255) // 256 * 256
    return (nbytes + ((1 << 20) + 256 if eb == 2 and nbytes % (1 << 20) == 0 else 0)) // eb


def _held(ctx, shapes, storage):
    """Views of the two population buffers of a context's workspace: by shell for
    one box, the flat buffer (its gaps cleared) for several."""
    dt = DTYPES[storage]
    eb = dt.itemsize
    nodes = [2 * b[0] * b[1] * b[2] for b in shapes]
    strides = [_stride(n, eb) for n in nodes]
    elems = 41 * sum(strides)
    nbytes = (elems * eb + 255) // 256 * 256
    out = []
    for i in range(2):
        flat = ctx._workspace[i * nbytes:i * nbytes + elems * eb].view(dt)
        if len(shapes) == 1:
            rows = flat.reshape(41, strides[0])[:, :nodes[0]]
            out.append(list(torch.split(rows, SHELL_COUNTS)))
        else:
            at = 0
            for n, s in zip(nodes, strides):
                if s > n:
                    flat[at:at + 41 * s].reshape(41, s)[:, n:].zero_()
                at += 41 * s
            out.append([flat])
    return out


def prepare(case, seed):
    _, _, theta0 = lbm.lattice()
    fields = _all_fields(case, seed, theta0)
    shapes = _shapes(case)
    stream = torch.cuda.Stream()
    state = {"case": case, "shapes": shapes, "stream": stream, "opts": _options(case, seed)}
    if case["kind"] == "init":
        state["fields"] = fields
        return state
    ctx = lbm.init_device(shapes, *fields, stream=stream, **state["opts"])
    if case["walls"]:
        ctx.set_walls(0, (0.0, 0.0, 0.0, theta0), (WALL_U, 0.0, 0.0, WALL_THETA * theta0))
    if case["graph"]:
        ctx.set_tuning(graph_steps=case["graph"])
    state.update(ctx=ctx, held=_held(ctx, shapes, case["storage"]), done=0)
    torch.cuda.synchronize()
    return state


def _wave_vector(case):
    """The mode that the thermal-decay run follows: the first one along z."""
    return (0.0, 0.0, TWO_PI / case["nz"])


def run(state):
    case = state["case"]
    if case["kind"] == "init":
        # a program that restarts: the old context goes when the new one is there
        ctx = lbm.init_device(state["shapes"], *state["fields"], stream=state["stream"], **state["opts"])
        state["ctx"] = ctx
        return {"populations": _held(ctx, state["shapes"], case["storage"])[0]}
    ctx = state["ctx"]
    if case["kind"] == "output":
        moments = ctx.moments()
        f = ctx.get_populations()
        ctx.set_populations(f)
        return {"moments": moments, "checkpoint": f, "populations": state["held"][0]}
    ctx.step(case["steps"])
    state["done"] += case["steps"]
    out = {"populations": state["held"][state["done"] % 2]}
    if case["monitor"] == "totals":
        out["totals"] = ctx.totals()
    elif case["monitor"] == "project":
        out["modes"] = ctx.project(0, _wave_vector(case))
    return out


def work(case):
    """Each population read once and written once per step, read once per
    diagnostic; the operations of the collision as the method states it."""
    nodes = sum(2 * b[0] * b[1] * b[2] for b in _shapes(case))
    eb = DTYPES[case["storage"]].itemsize
    one = 41 * eb * nodes
    if case["kind"] == "init":
        return {"bytes": one + 40 * nodes, "flops": 1500 * nodes}
    if case["kind"] == "output":
        # moments out; populations out as FP64, and back
        return {"bytes": (one + 40 * nodes) + (one + 328 * nodes) + (328 * nodes + one), "flops": 400 * nodes}
    reads = 0 if case["monitor"] == "none" else 1
    return {"bytes": (2 * case["steps"] + reads) * one, "flops": 1100 * case["steps"] * nodes}


# ---------------------------------------------------------------------------
# The same pass in 64 bits
# ---------------------------------------------------------------------------
def _lattice():
    """Velocities in half units, weights and theta0, shell by shell (rest, sc-1,
    sc-2, fcc-1, bcc-1, bcc-1/2), each in descending order of (cx, cy, cz)."""
    shells = [(0, 0), (4, 1), (16, 1), (8, 2), (12, 3), (3, 3)]  # 4 |c|^2, nonzero components
    printed = [None, 0.04743040745116578, 0.00165687664501576, 0.00651175327832464, 0.00454087801154440,
               0.04917980624482672]
    c, w = [], []
    for (n2, nz), wt in zip(shells, printed):
        vs = [v for v in itertools.product((4, 2, 1, 0, -1, -2, -4), repeat=3)
              if sum(a * a for a in v) == n2 and sum(a != 0 for a in v) == nz]
        c += vs
        w += [wt] * len(vs)
    w[0] = 1.0 - sum(w[1:])
    theta0 = sum(wt * 0.25 * v[0] * v[0] for v, wt in zip(c, w))
    return c, w, theta0


HALF, WEIGHT, THETA0 = _lattice()
CHUNK = 1 << 20


class _Exact:
    def __init__(self, device):
        t = lambda v: torch.tensor(v, dtype=torch.float64, device=device)  # noqa: E731
        self.c = t(HALF) * 0.5
        self.w = t(WEIGHT).reshape(41, 1)
        self.c2 = (self.c ** 2).sum(1)
        x, y, z = self.c.T
        self.phi = torch.stack([torch.ones_like(x), x, y, z, self.c2])           # 1, c, c^2
        one, c2 = torch.ones_like(x), self.c2
        psi = [x, y, z, -c2]
        self.second = torch.stack([one] + psi + [psi[a] * psi[b] for a in range(4) for b in range(a, 4)])
        self.expo = torch.stack([x, y, z, -c2], 1)

    def equilibrium(self, rho, u, th, model):
        if model == "series":
            return self.series(rho, u, th)
        n = 3 if model == "iso" else 4
        th = torch.full_like(rho, THETA0) if model == "iso" else th
        target = torch.cat([u, -((u ** 2).sum(0) + 3.0 * th).reshape(1, -1)])
        lam = torch.cat([u / th, (0.5 / th - 0.5 / THETA0).reshape(1, -1)])
        pairs = {}
        for k, (a, b) in enumerate((a, b) for a in range(4) for b in range(a, 4)):
            pairs[(a, b)] = pairs[(b, a)] = 5 + k
        for _ in range(6):
            s = self.second @ (self.w * torch.exp(self.expo @ lam))
            m = s[1:5] / s[0]
            A = [[s[pairs[(a, b)]] / s[0] - m[a] * m[b] for b in range(n)] for a in range(n)]
            r = [m[a] - target[a] for a in range(n)]
            for i in range(n):  # elimination (the matrix is a covariance)
                for j in range(i + 1, n):
                    f = A[j][i] / A[i][i]
                    for k in range(i, n):
                        A[j][k] = A[j][k] - f * A[i][k]
                    r[j] = r[j] - f * r[i]
            d = [None] * n
            for i in reversed(range(n)):
                v = r[i]
                for k in range(i + 1, n):
                    v = v - A[i][k] * d[k]
                d[i] = v / A[i][i]
            for i in range(n):
                lam[i] -= d[i]
        f = self.w * torch.exp(self.expo @ lam)
        return f * (rho / f.sum(0))

    def series(self, rho, u, th):
        eta = th / THETA0 - 1.0
        x = (self.c2 / THETA0).reshape(41, 1)
        ft = 1.0 + eta / 2 * (x - 3) + eta ** 2 / 8 * (x ** 2 - 10 * x + 15) \
            + eta ** 3 / 48 * (x ** 3 - 21 * x ** 2 + 105 * x - 105)
        wf = self.w * ft
        M2 = ((self.c2 ** 2).reshape(1, 41) @ wf)[0] / (15 * th ** 2) - 1
        M2p = (((self.c[:, 0] * self.c[:, 1]) ** 2).reshape(1, 41) @ wf)[0] / th ** 2 - 1
        A1 = 2.5 * M2 / (1 + 2.5 * M2)
        A2 = 5 * A1 * (1 - M2) - (3 + M2p - 5 * M2)
        uc, u2, c2 = self.c @ u / th, (u ** 2).sum(0), self.c2.reshape(41, 1)
        P = 1 + uc + uc ** 2 / 2 + uc ** 3 / 6 - u2 / (2 * th) * (1 - A1) - u2 * c2 * A1 / (6 * th ** 2) \
            + u2 * uc * A2 / (6 * th) - u2 * c2 * uc * A1 / (6 * th ** 2)
        return rho * wf * P

    def node_state(self, f):
        m = self.phi @ f
        rho, u = m[0], m[1:4] / m[0]
        return m, rho, u, (m[4] / rho - (u ** 2).sum(0)) / 3.0

    def path(self, f, feq):
        """Nontrivial root of H(f + a (f_eq - f)) = H(f): Newton from the right on
        the convex difference, below the positivity cap."""
        x = feq / f - 1.0
        low = x.min(0).values
        cap = torch.where(low < 0, (1.0 - 2.0 ** -10) / -low, torch.full_like(low, 1e30))
        fx = f * x
        p = (fx * torch.log1p(x)).sum(0)
        a = torch.minimum(torch.full_like(cap, 2.0), cap)
        for _ in range(8):
            log = torch.log1p(a * x)
            g = (f * ((1.0 + a * x) * log - a * x)).sum(0) - a * p
            gp = (fx * log).sum(0) - p
            step = torch.where(gp > 0, g / gp, torch.zeros_like(g))
            a = torch.minimum(torch.clamp(a - step, min=1.0), cap)
        return torch.where(x.abs().max(0).values < 1e-7, torch.full_like(a, 2.0), a)

    def collide(self, f, omega, model, entropic):
        """Collision in place, over pieces of the nodes."""
        for at in range(0, f.shape[1], CHUNK):
            g = f[:, at:at + CHUNK].clone()
            _, rho, u, th = self.node_state(g)
            feq = self.equilibrium(rho, u, th, model)
            rate = omega * 0.5 * self.path(g, feq) if entropic else omega
            f[:, at:at + CHUNK] = g + rate * (feq - g)

    def init(self, fields, model, out):
        rho, ux, uy, uz, th = fields
        for at in range(0, rho.numel(), CHUNK):
            s = slice(at, at + CHUNK)
            out[:, s] = self.equilibrium(rho[s], torch.stack([ux[s], uy[s], uz[s]]), th[s], model)

    def pull(self, f, g, nx, ny, nz):
        """g_q(node) = f_q(node - c_q), periodic on the two sublattices."""
        for q, v in enumerate(HALF):
            src, dst = f[q].reshape(2, nz, ny, nx), g[q].reshape(2, nz, ny, nx)
            for s in range(2):
                o = (s - v[0]) % 2
                shift = [(h + o - s) // 2 for h in (v[2], v[1], v[0])]
                dst[s] = torch.roll(src[o], shift, (0, 1, 2))

    def walls(self, f, g, nx, ny, nz, model, theta0):
        """Diffuse walls below and above: what a node sent through one comes back
        to it in the shape of the wall's equilibrium."""
        find = {v: q for q, v in enumerate(HALF)}
        src, dst = f.reshape(41, 2, nz, ny, nx), g.reshape(41, 2, nz, ny, nx)
        one = torch.ones(1, dtype=torch.float64, device=f.device)
        for w, (u0, t0) in enumerate(((0.0, theta0), (WALL_U, WALL_THETA * theta0))):
            u = torch.tensor([[u0], [0.0], [0.0]], dtype=torch.float64, device=f.device)
            fw = self.equilibrium(one, u, t0 * one, model)[:, 0]
            for k in range(4):  # layers counted from the wall
                L = k if w == 0 else 2 * ny - 1 - k
                if not 0 <= L < 2 * ny:
                    continue
                qs = [q for q, v in enumerate(HALF) if (v[1] if w == 0 else -v[1]) > k]
                back = [find[tuple(-a for a in HALF[q])] for q in qs]
                s, y = L % 2, L // 2
                sigma = src[back, s, :, y].sum(0) / fw[qs].sum()
                for q in qs:
                    dst[q, s, :, y] = fw[q] * sigma


def _stored(f, case, shift):
    """Populations as the storage form holds them (shift: k_amp), by shell, in place."""
    if case["storage"] in ("f64", "f32"):
        return list(torch.split(f, SHELL_COUNTS))
    for q in range(41):
        k = 0 if case["storage"] == "f32s" else round(-math.log2(WEIGHT[q])) + shift
        f[q].sub_(WEIGHT[q]).mul_(2.0 ** k)
    return list(torch.split(f, SHELL_COUNTS))


def _largest(f):
    """Largest |f - w| 2^k_shell."""
    return max(float((f[q] - WEIGHT[q]).abs().max()) * 2.0 ** round(-math.log2(WEIGHT[q])) for q in range(41))


def exact(case, seed):
    dev = torch.device("cuda")
    E = _Exact(dev)
    fields = _all_fields(case, seed, THETA0)
    shapes = _shapes(case)
    model, nodes, at = case["model"], [2 * b[0] * b[1] * b[2] for b in shapes], 0
    f0 = []
    for n in nodes:
        f = torch.empty(41, n, dtype=torch.float64, device=dev)
        E.init([v[at:at + n] for v in fields], model, f)
        f0.append(f)
        at += n
    del fields
    m = max(_largest(f) for f in f0)
    shift = max(-40, min(40, math.floor(math.log2(1024.0 / m)))) if m > 0 else 10
    if case["kind"] == "init":
        return {"populations": _stored(f0[0], case, shift)}
    if case["kind"] == "output":
        mom = E.phi @ f0[0]
        mom[4] *= 0.5
        return {"moments": mom.cpu().numpy(), "checkpoint": f0[0].reshape(-1).cpu().numpy(),
                "populations": _stored(f0[0], case, shift)}
    for i, (nx, ny, nz, tau) in enumerate(shapes):
        f, g = f0[i], torch.empty_like(f0[i])
        for _ in range(case["steps"]):
            E.pull(f, g, nx, ny, nz)
            if case["walls"]:
                E.walls(f, g, nx, ny, nz, model, THETA0)
            E.collide(g, 1.0 / tau, model, case["entropic"])
            f, g = g, f
        f0[i] = f
        del f, g
    if case["flow"] == "batch":
        eb = DTYPES[case["storage"]].itemsize
        strides = [_stride(n, eb) for n in nodes]
        flat = torch.zeros(41 * sum(strides), dtype=torch.float64, device=dev)
        at = 0
        for f, n, s in zip(f0, nodes, strides):
            flat[at:at + 41 * s].reshape(41, s)[:, :n] = torch.cat(_stored(f, case, shift))
            at += 41 * s
        return {"populations": [flat]}
    f, out = f0[0], {}
    if case["monitor"] == "totals":
        mom = sum((E.phi @ f[:, k:k + CHUNK]).sum(1) for k in range(0, f.shape[1], CHUNK))
        mom[4] *= 0.5
        out["totals"] = mom.cpu().numpy().reshape(1, 5)
    elif case["monitor"] == "project":
        out["modes"] = _modes(E, f, case)
    out["populations"] = _stored(f, case, shift)
    return out


def _modes(E, f, case):
    """Fourier amplitudes of rho, j, E and theta at the followed mode."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    half = torch.tensor([0.0, 0.5], dtype=torch.float64, device=f.device)
    ph = sum(k * _axis(n, a, half, f.device) for a, (k, n) in enumerate(zip(_wave_vector(case), (nx, ny, nz))))
    ph = ph.expand(2, nz, ny, nx).reshape(-1)
    acc = torch.zeros(6, 2, dtype=torch.float64, device=f.device)
    for at in range(0, f.shape[1], CHUNK):
        m, rho, u, th = E.node_state(f[:, at:at + CHUNK])
        v = torch.cat([m[:4], 0.5 * m[4:5], th.reshape(1, -1)])
        p = ph[at:at + CHUNK]
        acc += torch.stack([(v * torch.cos(p)).sum(1), -(v * torch.sin(p)).sum(1)], 1)
    a = (acc / f.shape[1]).cpu().numpy()
    return np.ascontiguousarray(a[:, 0] + 1j * a[:, 1])
