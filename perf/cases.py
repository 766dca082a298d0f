"""Performance cases of the micromagnetic solver: what a user's program has
it do, over the sizes and options it takes.

Every case goes through the package's public classes (Solver, Batch,
Surrogate).  prepare() makes what a program keeps (the solver with its demag
kernel, the batch, the network) and seeded inputs on the GPU; run() is one
pass; exact() computes the same results in 64-bit floats with plain torch
(zero-padded FFT convolution with the cell-averaged demagnetising tensor,
Runge-Kutta steps, the network as shifted matrix products); work() gives the
bytes and operations a pass cannot do without.

Kinds of case:
  film     a solver of any grid (2D films and 3D blocks): set m, integrate
           (fixed steps, or an embedded pair to t_end), get m
  heff     one effective-field evaluation of a caller's field
  batch    a sweep of films of uneven size advanced together
  train    one training step of the surrogate network
  predict  proposals of the network for a batch of states
  advance  speculative verification: proposals checked by the plain solver
"""
import math

import numpy as np
import torch

import paper_1102_3069_amd as llg

MU0 = 4e-7 * math.pi
GAMMA0 = MU0 * 1.7595e11
KB = 1.380649e-23
MU_B = 9.2740100783e-24
E_CHARGE = 1.602176634e-19
FIXED = ("euler", "heun", "rk3", "rk4")
LAYERS = ((9, 32), (32, 32), (32, 32), (32, 32), (32, 32), (32, 3))   # the network's (inputs, outputs)
BATCH_SIDES = (64, 96, 128, 192, 256)


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest film of the test problems, Heun steps from a random
        # state: launches and latency
        film("film32_heun", 32, 32, method="heun", dt=1e-13, steps=50, start="random", alpha=0.5, Ku=0.0, dz=4e-9),
        # one field evaluation of a small film with odd sides, the call a
        # program makes between its own steps
        dict(name="heff_100x37", kind="heff", nx=100, ny=37, nz=1, dx=4e-9, dz=3e-9),
        # standard problem 4's element at 4 nm and twice its length, with
        # every term on (cubic anisotropy, spin torque): sides that are no
        # power of two
        film("film250x63_rk4_terms", 250, 63, method="rk4", dt=1e-13, steps=40, extras=True),
        # the same problem as the paper refines it: 256 x 64 x 2 cells, the
        # Bogacki-Shampine pair
        film("film256x64x2_rk23", 256, 64, 2, method="rk23", t_end=3e-12, dx=1.953125e-9, dz=1.5e-9),
        # the headline film, adaptive Dormand-Prince
        film("film512_dp45", 512, 512, method="rkdp45", t_end=2e-11),
        # a large film of generic sides
        film("film1000x600_rk4", 1000, 600, method="rk4", dt=1e-13, steps=5),
        # the largest film, adaptive
        film("film2048_dp45", 2048, 2048, method="rkdp45", t_end=2e-12),
        # the periodic block at 300 K, Heun steps
        film("block256x256x64_heun_300K", 256, 256, 64, method="heun", dt=5e-14, steps=10, px=True, py=True, T=300.0,
             start="vortex", alpha=0.1, Ku=0.0, dx=3e-9, dz=3e-9, Ms=1.0e6, Aex=1.5e-11, field=0.0),
        # an open block of generic sides
        film("block100x60x20_rk4", 100, 60, 20, method="rk4", dt=5e-14, steps=10, dx=3e-9, dz=3e-9),
        # a parameter sweep of 64 uneven films, advanced piece by piece
        dict(name="batch64_rk4", kind="batch", films=64, ragged=False, method="rk4", dt=1e-13, steps=30),
        # surrogate training on 16 states of 256 x 256
        dict(name="train16_256", kind="train", H=256, W=256, batch=16),
        # learned proposals verified by the plain solver, two rounds of 16
        dict(name="advance256_w16", kind="advance", H=256, W=256, window=16, segments=32),
    ]


def film(name, nx, ny, nz=1, method="rk4", dt=0.0, steps=0, t_end=0.0, start="canted", alpha=0.02, Ku=5e3, dx=4e-9,
         dz=3e-9, px=False, py=False, T=0.0, extras=False, Ms=8e5, Aex=1.3e-11, field=0.025):
    c = dict(kind="film", nx=nx, ny=ny, nz=nz, method=method, dt=dt, steps=steps, t_end=t_end, start=start,
             alpha=alpha, Ku=Ku, dx=dx, dz=dz, px=px, py=py, T=T, extras=extras, Ms=Ms, Aex=Aex, field=field)
    return dict(c, name=name) if name else c


def log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def good_even(n):
    """The nearest even length from n up made of 2, 3, 5 and 7 (a periodic axis)."""
    n += n % 2
    while True:
        m = n
        for f in (2, 3, 5, 7):
            while m % f == 0:
                m //= f
        if m == 1:
            return n
        n += 2


def draw(rng):
    kind = rng.choice(["film"] * 8 + ["block"] * 4 + ["heff"] * 3 + ["batch", "train", "predict", "predict", "advance"])
    if kind in ("film", "block", "heff"):
        if kind == "block" or (kind == "heff" and rng.random() < 0.3):
            nx, ny, nz = log_int(rng, 8, 160), log_int(rng, 8, 160), log_int(rng, 2, 48)
            dx = dz = 3e-9
        else:
            nx, ny, nz = log_int(rng, 16, 1024), log_int(rng, 16, 1024), 1
            dx, dz = 4e-9, 3e-9
        cells = nx * ny * nz
        if kind == "heff":
            return dict(kind="heff", nx=nx, ny=ny, nz=nz, dx=dx, dz=dz) if cells < 200000 else \
                dict(kind="heff", nx=nx, ny=max(16, min(ny, 200000 // nx)), nz=1, dx=dx, dz=dz)
        px, py = rng.random() < 0.2, rng.random() < 0.2
        nx, ny = good_even(nx) if px else nx, good_even(ny) if py else ny
        method = rng.choice(["heun", "rk4", "rk3", "euler", "rkdp45", "rkdp45", "rk23"])
        c = film(None, nx, ny, nz, method=method, dx=dx, dz=dz, px=px, py=py, extras=rng.random() < 0.25,
                 alpha=rng.choice([0.02, 0.1, 0.5]), field=round(rng.uniform(0.0, 0.05), 4))
        if method in FIXED:
            c["dt"] = 5e-14 if nz > 1 or method == "euler" else 1e-13
            c["steps"] = int(max(3, min(50, 3e6 / cells)))
            c["T"] = 300.0 if rng.random() < 0.25 else 0.0
        else:
            c["t_end"] = 2e-12 if method == "rk23" or cells > 300000 else 1e-11
        return c
    if kind == "batch":
        return dict(kind="batch", films=log_int(rng, 2, 64), ragged=rng.random() < 0.6, method=rng.choice(["rk4", "heun", "rk3"]),
                    dt=1e-13, steps=20)
    if kind == "advance":
        return dict(kind="advance", H=log_int(rng, 32, 256), W=log_int(rng, 32, 256), window=rng.choice([4, 8, 16]),
                    segments=16)
    return dict(kind=kind, H=log_int(rng, 32, 256), W=log_int(rng, 32, 256), batch=log_int(rng, 1, 16))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def generator(seed):
    return torch.Generator(device=device()).manual_seed(int(seed))


def unit(v, dim=0):
    return v / v.norm(dim=dim, keepdim=True)


def start_state(shape, how, seed):
    """float32 (3, nz, ny, nx) unit vectors: "random" directions, a "uniform"
    direction near (1,1,1), the same with some noise ("canted"), or a
    "vortex" with a 10-cell core and noise."""
    g = generator(seed)
    noise = torch.randn(shape, generator=g, device=device(), dtype=torch.float64)
    if how == "random":
        return unit(noise).float().contiguous()
    if how == "vortex":
        _, nz, ny, nx = shape
        x = torch.arange(nx, device=device(), dtype=torch.float64) + 0.5 - nx / 2
        y = torch.arange(ny, device=device(), dtype=torch.float64) + 0.5 - ny / 2
        r = torch.hypot(x[None, :], y[:, None])
        th = 0.5 * math.pi * torch.clamp(r / 10.0, max=1.0)
        m = torch.stack([-y[:, None] / r * torch.sin(th), x[None, :] / r * torch.sin(th), torch.cos(th)])
        m = m[:, None].expand(shape)
    else:
        tilt = torch.randn(3, generator=g, device=device(), dtype=torch.float64)
        m = (unit(torch.ones(3, device=device(), dtype=torch.float64) + 0.2 * tilt)).reshape(3, 1, 1, 1).expand(shape)
    return unit(m + (0.0 if how == "uniform" else 0.02) * noise).float().contiguous()


def problem(c):
    """The problem dict of a film, block or field case (keys of Solver.set_problem)."""
    ang = math.radians(170.0)
    f = c.get("field", 0.025)
    p = dict(n=(c["nx"], c["ny"], c["nz"]), cell=(c["dx"], c["dx"], c["dz"]), pbc=(bool(c.get("px")), bool(c.get("py")), False),
             images=10, Ms=c.get("Ms", 8e5), Aex=c.get("Aex", 1.3e-11), alpha=c.get("alpha", 0.02), Ku=c.get("Ku", 5e3),
             u=(1.0, 0.0, 0.0), B=(f * math.cos(ang), f * math.sin(ang), 0.0), T=c.get("T", 0.0), seed=3)
    if c.get("extras"):
        p.update(Kc1=4e3, Kc2=2e3, j=(1e12, 2e11, 0.0), P=0.5, xi=0.05)
    return p


def sweep(c):
    """The films of a batch case: the sides and materials of a parameter
    sweep (fixed), so that inputs of another seed are other start states."""
    rng = np.random.default_rng(4)
    films = []
    for _ in range(c["films"]):
        nx = ny = int(rng.choice(BATCH_SIDES))
        if c["ragged"]:
            nx, ny = int(rng.integers(17, 257)), int(rng.integers(9, 257))
        a, b = float(rng.uniform(0.0, 2 * math.pi)), float(rng.uniform(0.0, 0.1))
        films.append(dict(n=(nx, ny, 1), cell=(4e-9, 4e-9, 3e-9), pbc=(False, False, False), Ms=float(rng.uniform(6e5, 1.2e6)),
                          Aex=1.3e-11, alpha=float(rng.uniform(0.01, 0.5)), Ku=0.0, u=(1.0, 0.0, 0.0),
                          B=(b * math.cos(a), b * math.sin(a), 0.0)))
    return films


def sweep_states(films, seed):
    return [start_state((3, 1, p["n"][1], p["n"][0]), "random", 1000 * seed + i) for i, p in enumerate(films)]


def weights():
    """Network parameters as training starts from (the same for every seed)."""
    rng = np.random.default_rng(0)
    out = []
    for li, (ci, co) in enumerate(LAYERS):
        std = math.sqrt(2.0 / (9 * ci)) * (0.1 if li == len(LAYERS) - 1 else 1.0)
        out.append(((rng.standard_normal((co, ci, 3, 3)) * std).astype(np.float32), np.zeros(co, np.float32)))
    return out


def states(c, seed):
    """(m_in, m_base, m_target, B) of a network case: states, coarse steps
    of them and states a 1e-4 correction further on."""
    n, H, W = c["batch"], c["H"], c["W"]
    g = generator(seed)
    m = torch.stack([start_state((3, 1, H, W), "canted", 1000 * seed + i)[:, 0] for i in range(n)])
    step = torch.randn((2,) + m.shape, generator=g, device=device())
    base = unit(m + 1e-3 * step[0], 1).contiguous()
    target = unit(base + 1e-4 * step[1], 1).contiguous()
    B = np.random.default_rng(seed).uniform(-0.05, 0.05, (n, 3)).astype(np.float32)
    return m.contiguous(), base, target, B


def advance_problem(c):
    return problem(dict(nx=c["W"], ny=c["H"], nz=1, dx=4e-9, dz=3e-9, field=0.03))


def prepare(case, seed):
    c = case
    if c["kind"] in ("film", "heff"):
        shape = (3, c["nz"], c["ny"], c["nx"])
        m = start_state(shape, c.get("start", "canted"), seed)
        out = torch.empty_like(m)
        s = llg.Solver(0)
        s.set_problem(problem(c))
        torch.cuda.synchronize()
        s.set_m(m)
        s.eval_heff(out)            # builds the demag kernel, which a program keeps
        return dict(c=c, s=s, m=m, out=out)
    if c["kind"] == "batch":
        films = sweep(c)
        m = sweep_states(films, seed)
        torch.cuda.synchronize()
        b = llg.Batch([(p, x.cpu().numpy()) for p, x in zip(films, m)])
        return dict(c=c, b=b, out=[torch.empty_like(x) for x in m])
    s = llg.Surrogate(c["H"], c["W"], max_batch=c.get("batch", 1))
    s.set_params(weights())
    s.set_output_scale(1e-4)
    if c["kind"] == "advance":
        m = start_state((3, 1, c["H"], c["W"]), "uniform", seed)
        buf, prob = m.clone(), advance_problem(c)
        torch.cuda.synchronize()
        s.advance(prob, buf, 1, window=c["window"])   # builds the verification batches, which a program keeps
        return dict(c=c, s=s, m=m, out=buf, prob=prob)
    m, base, target, B = states(c, seed)
    torch.cuda.synchronize()
    return dict(c=c, s=s, m=m, base=base, target=target, B=B, out=torch.empty_like(m))


def run(state):
    c, kind = state["c"], state["c"]["kind"]
    if kind == "film":
        s = state["s"]
        s.set_m(state["m"])
        if c["method"] in FIXED:
            s.step(c["method"], c["dt"], c["steps"])
        else:
            s.run(c["t_end"], 1e-5, 1e-14, method=c["method"])
        return {"m": s.get_m(state["out"])}
    if kind == "heff":
        s = state["s"]
        if c["nz"] == 1:
            return {"h": s.eval_heff_noalloc(state["m"], state["out"])}
        s.set_m(state["m"])
        return {"h": s.eval_heff(state["out"])}
    if kind == "batch":      # the films go on from where the last pass left them
        b = state["b"]
        b.step(c["method"], c["dt"], c["steps"])
        return [b.get_m(i, o) for i, o in enumerate(state["out"])]
    s = state["s"]
    if kind == "train":
        loss = s.train_step(state["m"], state["target"], state["B"], lr=1e-3, m_base=state["base"])
        return {"loss": loss, "grads": s.get_grads(), "params": s.get_params()}
    if kind == "predict":
        return {"m": s.predict(state["m"], state["B"], out=state["out"], m_base=state["base"])}
    state["out"].copy_(state["m"])
    torch.cuda.current_stream().synchronize()   # the library works on its own stream
    s.advance(state["prob"], state["out"], c["segments"], window=c["window"])
    return {"m": state["out"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def eval_work(n, pbc):
    """One field evaluation: the field read, the result written, the kernel
    spectrum read once; the transforms of the zero-padded axes (the zero
    lines skipped), the product and the local terms."""
    nx, ny, nz = n
    P = [k if p else (1 if k == 1 and a == 2 else 2 * k) for a, (k, p) in enumerate(zip(n, pbc))]
    hx, hy, hz = P[0] // 2 + 1, P[1] // 2 + 1, P[2] // 2 + 1
    lg = [math.log2(max(2, p)) for p in P]
    flops = 6 * (2.5 * P[0] * lg[0] * ny * nz + 5 * P[1] * lg[1] * hx * nz)
    if P[2] > 1:
        flops += 6 * 5 * P[2] * lg[2] * hx * P[1]
    flops += (14 if P[2] == 1 else 30) * hx * P[1] * P[2] + 80 * nx * ny * nz
    return 24.0 * nx * ny * nz + 4.0 * (4 if P[2] == 1 else 6) * hx * hy * hz, flops


STAGES = {"euler": 1, "heun": 2, "rk3": 3, "rk4": 4, "rkdp45": 6, "rk23": 3}


def evals(c, method):
    """Evaluations of a pass (an embedded pair: about 0.3 or 0.03 ps an
    attempt after the first few)."""
    if method in FIXED:
        return STAGES[method] * c["steps"]
    return STAGES[method] * (4 + c["t_end"] / (3e-13 if method == "rkdp45" else 3e-14))


def work(case):
    c = case
    if c["kind"] in ("film", "heff"):
        b, f = eval_work((c["nx"], c["ny"], c["nz"]), (c.get("px"), c.get("py"), False))
        e = 1 if c["kind"] == "heff" else evals(c, c["method"])
        return {"bytes": e * b, "flops": e * f}
    if c["kind"] == "batch":
        w = [eval_work(p["n"], p["pbc"]) for p in sweep(c)]
        e = evals(c, c["method"])
        return {"bytes": e * sum(x[0] for x in w), "flops": e * sum(x[1] for x in w)}
    px = c["H"] * c["W"]
    net = 2.0 * 9 * sum(ci * co for ci, co in LAYERS) * px     # operations of one forward pass
    if c["kind"] == "train":
        # states and targets in; the layer outputs are needed again by the
        # backward pass (written and read once, 16 bits)
        act = 2 * 2.0 * px * sum(co for _, co in LAYERS)
        return {"bytes": c["batch"] * (36.0 * px + act) + 3 * 4 * 40483.0, "flops": 3 * net * c["batch"]}
    if c["kind"] == "predict":
        return {"bytes": c["batch"] * 36.0 * px + 2 * 40483.0, "flops": net * c["batch"]}
    # a segment: four evaluations of the coarse step, 40 of the plain steps,
    # one pass of the network
    b, f = eval_work((c["W"], c["H"], 1), (False,) * 3)
    return {"bytes": c["segments"] * (44 * b + 36.0 * px), "flops": c["segments"] * (44 * f + net)}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
def newell(X, Y, Z, d):
    """xx and xy of the tensor between two cells d apart by (X, Y, Z)
    (Newell, Williams & Dunlop 1993): second differences of f and g."""
    def guarded(num, den, fn):
        return torch.where(den > 0, fn(num / torch.where(den > 0, den, torch.ones_like(den))), torch.zeros_like(num))

    def f(x, y, z):
        x, y, z = x.abs(), y.abs(), z.abs()
        R = (x * x + y * y + z * z).sqrt()
        return (0.5 * y * (z * z - x * x) * guarded(y, (x * x + z * z).sqrt(), torch.asinh)
                + 0.5 * z * (y * y - x * x) * guarded(z, (x * x + y * y).sqrt(), torch.asinh)
                - x * y * z * guarded(y * z, x * R, torch.atan) + (2 * x * x - y * y - z * z) * R / 6)

    def g(x, y, z):      # of non-negative arguments; odd in x and y, even in z
        R = (x * x + y * y + z * z).sqrt()
        return (x * y * z * guarded(z, (x * x + y * y).sqrt(), torch.asinh)
                + y / 6 * (3 * z * z - y * y) * guarded(x, (y * y + z * z).sqrt(), torch.asinh)
                + x / 6 * (3 * z * z - x * x) * guarded(y, (x * x + z * z).sqrt(), torch.asinh)
                - z ** 3 / 6 * guarded(x * y, z * R, torch.atan) - z * y * y / 2 * guarded(x * z, y * R, torch.atan)
                - z * x * x / 2 * guarded(y * z, x * R, torch.atan) - x * y * R / 3)

    out = []
    for fn in (f, g):
        acc = 0.0
        for a, wa in ((-1, -1.0), (0, 2.0), (1, -1.0)):
            for b, wb in ((-1, -1.0), (0, 2.0), (1, -1.0)):
                for e, we in ((-1, -1.0), (0, 2.0), (1, -1.0)):
                    xs, ys, zs = X + a * d[0], Y + b * d[1], Z + e * d[2]
                    if fn is g:
                        acc = acc + wa * wb * we * torch.sign(xs) * torch.sign(ys) * g(xs.abs(), ys.abs(), zs.abs())
                    else:
                        acc = acc + wa * wb * we * f(xs, ys, zs)
        out.append(acc / (4 * math.pi * d[0] * d[1] * d[2]))
    return out


def dipole(x, y, z):
    """(xx, yy, zz, xy, xz, yz) of the point-dipole tensor."""
    r2 = x * x + y * y + z * z
    a = r2.pow(-1.5) / (4 * math.pi)
    b = -3 * a / r2
    return torch.stack([a + b * x * x, a + b * y * y, a + b * z * z, b * x * y, b * x * z, b * y * z])


def tent(d):
    """Gauss-Legendre nodes (three a side) and weights of the tent d - |s|."""
    out = []
    for t, w in ((0.5 - 0.5 * math.sqrt(0.6), 5 / 18), (0.5, 8 / 18), (0.5 + 0.5 * math.sqrt(0.6), 5 / 18)):
        out += [(s * d * t, d * w * (d - d * t)) for s in (1, -1)]
    return out


class Film64:
    """One problem in 64-bit floats: field, torque and steps."""

    def __init__(self, p):
        self.p, (nx, ny, nz), d = p, p["n"], p["cell"]
        dev = device()
        s = max(d)
        e = [v / s for v in d]
        # the non-negative offsets of each axis; the rest follows from parity
        cnt = [n // 2 + 1 if q else n for n, q in zip(p["n"], p["pbc"])]
        ax = [torch.arange(k, device=dev, dtype=torch.float64) for k in cnt]
        I, J, K = ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]
        X, Y, Z = torch.broadcast_tensors(I * e[0], J * e[1], K * e[2])
        far = torch.maximum(torch.maximum(I, J), K) > 8
        N = torch.zeros((6,) + X.shape, device=dev, dtype=torch.float64)
        x, y, z = X[far], Y[far], Z[far]
        acc = 0.0
        for sx, wx in tent(e[0]):
            for sy, wy in tent(e[1]):
                for sz, wz in tent(e[2]):
                    if x.numel():
                        acc = acc + wx * wy * wz / (e[0] * e[1] * e[2]) * dipole(x + sx, y + sy, z + sz)
        if x.numel():
            N[:, far] = acc
        x, y, z = X[~far], Y[~far], Z[~far]
        xx, xy = newell(x, y, z, e)
        yy, yz = newell(y, z, x, (e[1], e[2], e[0]))
        zz, xz = newell(z, x, y, (e[2], e[0], e[1]))
        N[:, ~far] = torch.stack([xx, yy, zz, xy, xz, yz])
        im = [range(-p.get("images", 10), p.get("images", 10) + 1) if q else (0,) for q in p["pbc"]]
        for a in im[0]:
            for b in im[1]:
                if a or b:
                    N += e[0] * e[1] * e[2] * dipole(X + a * nx * e[0], Y + b * ny * e[1], Z)
        # mirror: odd components change sign; at the Nyquist offset of a
        # periodic axis the two representatives are averaged (odd ones vanish)
        odd = {0: (3, 4), 1: (3, 5), 2: (4, 5)}
        self.P = [n if q else (1 if a == 2 and n == 1 else 2 * n) for a, (n, q) in enumerate(zip(p["n"], p["pbc"]))]
        for a, dim in ((0, 3), (1, 2), (2, 1)):
            n, P = p["n"][a], self.P[a]
            if P == 1:
                continue
            sign = torch.ones(6, 1, 1, 1, device=dev, dtype=torch.float64)
            sign[list(odd[a])] = -1.0
            if p["pbc"][a] and n % 2 == 0:
                last = N.select(dim, n // 2)
                last[list(odd[a])] = 0.0
                N = torch.cat([N, sign * N.narrow(dim, 1, n // 2 - 1).flip(dim)], dim)
            elif p["pbc"][a]:
                N = torch.cat([N, sign * N.narrow(dim, 1, n // 2).flip(dim)], dim)
            else:
                gap = torch.zeros_like(N.narrow(dim, 0, 1))
                N = torch.cat([N, gap, sign * N.narrow(dim, 1, n - 1).flip(dim)], dim)
        self.K = -torch.fft.rfftn(N, dim=(1, 2, 3)).real
        self.step_index = 0

    def demag(self, m):
        P, (nx, ny, nz) = self.P, self.p["n"]
        F = torch.fft.rfftn(m, s=(P[2], P[1], P[0]), dim=(1, 2, 3))
        K = self.K
        H = torch.stack([K[0] * F[0] + K[3] * F[1] + K[4] * F[2], K[3] * F[0] + K[1] * F[1] + K[5] * F[2],
                         K[4] * F[0] + K[5] * F[1] + K[2] * F[2]])
        return self.p["Ms"] * torch.fft.irfftn(H, s=(P[2], P[1], P[0]), dim=(1, 2, 3))[:, :nz, :ny, :nx]

    def shifted(self, m, a, k):
        """m[i + k] along axis a; the cell itself where a free surface has no neighbour."""
        dim, n = 3 - a, self.p["n"][a]
        r = torch.roll(m, -k, dim)
        if not self.p["pbc"][a]:
            edge = n - 1 if k > 0 else 0
            r.select(dim, edge).copy_(m.select(dim, edge))
        return r

    def field(self, m, thermal=None):
        p = self.p
        H = self.demag(m)
        for a in range(3):
            if p["n"][a] > 1:
                H = H + 2 * p["Aex"] / (MU0 * p["Ms"] * p["cell"][a] ** 2) * (self.shifted(m, a, 1) + self.shifted(m, a, -1) - 2 * m)
        H[0] += 2 * p["Ku"] / (MU0 * p["Ms"]) * m[0]                      # easy axis x
        if p.get("Kc1"):
            q = m * m                                                    # cubic axes x, y, z
            for i, j, k in ((0, 1, 2), (1, 2, 0), (2, 0, 1)):
                H[i] -= 2 * m[i] / (MU0 * p["Ms"]) * (p["Kc1"] * (q[j] + q[k]) + p["Kc2"] * q[j] * q[k])
        H += torch.tensor(p["B"], device=m.device, dtype=torch.float64).reshape(3, 1, 1, 1) / MU0
        return H if thermal is None else H + thermal

    def rhs(self, m, thermal=None):
        p, al = self.p, self.p["alpha"]
        a = torch.cross(m, self.field(m, thermal), dim=0)
        k = -GAMMA0 / (1 + al * al) * (a + al * torch.cross(m, a, dim=0))
        if p.get("j"):
            D = sum(p["j"][a] / (2 * p["cell"][a]) * (self.shifted(m, a, 1) - self.shifted(m, a, -1))
                    for a in range(3) if p["j"][a] and p["n"][a] > 1)
            b = p["P"] * MU_B / (E_CHARGE * p["Ms"] * (1 + p["xi"] ** 2))
            a = torch.cross(m, D, dim=0)
            k = k - b / (1 + al * al) * (torch.cross(m, a, dim=0) + (p["xi"] - al) * a)
        return k

    def noise(self, dt, shape):
        """The thermal field of one step: Philox4x32-10 (Salmon et al. 2011)
        on (cell, step, 0, 0), 24-bit uniforms, Box-Muller."""
        p = self.p
        if not p.get("T"):
            return None
        n = shape[1] * shape[2] * shape[3]
        x = [torch.arange(n, device=device()), torch.full((n,), self.step_index, device=device()), 0, 0]
        x = [torch.as_tensor(v, device=device(), dtype=torch.int64).expand(n) for v in x]
        k0, k1, mask = p["seed"] & 0xFFFFFFFF, p["seed"] >> 32, 0xFFFFFFFF

        def mulhilo(c, v):       # 32 x 32 -> 64 bits in two halves (no sign bit)
            lo16, hi = c * (v & 0xFFFF), c * (v >> 16)
            mid = hi + (lo16 >> 16)
            return mid >> 16, ((mid & 0xFFFF) << 16) | (lo16 & 0xFFFF)
        for r in range(10):
            h0, l0 = mulhilo(0xD2511F53, x[0])
            h1, l1 = mulhilo(0xCD9E8D57, x[2])
            x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        u = [((v >> 8).double() + 0.5) * 2.0 ** -24 for v in x]
        a, b = torch.sqrt(-2 * torch.log(u[0])), torch.sqrt(-2 * torch.log(u[2]))
        eta = torch.stack([a * torch.cos(2 * math.pi * u[1]), a * torch.sin(2 * math.pi * u[1]), b * torch.cos(2 * math.pi * u[3])])
        V = p["cell"][0] * p["cell"][1] * p["cell"][2]
        return math.sqrt(2 * p["alpha"] * KB * p["T"] / (GAMMA0 * MU0 * p["Ms"] * V * dt)) * eta.reshape(shape)

    def stages(self, m, dt, A, k1=None):
        """The slopes of a tableau's stages; every stage input is renormalised."""
        th = self.noise(dt, m.shape)
        ks = [self.rhs(m, th) if k1 is None else k1]
        for row in A[1:]:
            ks.append(self.rhs(unit(m + dt * sum(a * k for a, k in zip(row, ks) if a)), th))
        return ks

    def fixed(self, m, method, dt, steps):
        A, b = TABLEAUX[method][:2]
        for _ in range(steps):
            ks = self.stages(m, dt, A)
            m = unit(m + dt * sum(w * k for w, k in zip(b, ks) if w))
            self.step_index += 1
        return m

    def adaptive(self, m, method, t_end, tol, dt):
        """Embedded pair: err = max over cells of the estimate, next step
        dt clamp(0.9 (tol/err)^(1/(q+1)), 0.2, 5), landing on t_end."""
        A, b, bh, q = TABLEAUX[method]
        t, k1 = 0.0, None
        while t < t_end:
            h, last = (t_end - t, True) if dt >= t_end - t else (dt, False)
            ks = self.stages(m, h, A, k1)
            err = float((h * sum((w - v) * k for w, v, k in zip(b, bh, ks) if w != v)).norm(dim=0).max())
            k1 = ks[0]
            if err <= tol:
                m = unit(m + h * sum(w * k for w, k in zip(b, ks) if w))
                t, k1 = (t_end if last else t + h), ks[-1]
            dt = h * (min(5.0, max(0.2, 0.9 * (tol / err) ** (1.0 / (q + 1)))) if err else 5.0)
        return m


TABLEAUX = {
    "euler": ([[]], [1.0]),
    "heun": ([[], [1.0]], [0.5, 0.5]),
    "rk3": ([[], [0.5], [-1.0, 2.0]], [1 / 6, 2 / 3, 1 / 6]),
    "rk4": ([[], [0.5], [0.0, 0.5], [0.0, 0.0, 1.0]], [1 / 6, 1 / 3, 1 / 3, 1 / 6]),
    # Bogacki & Shampine 3(2); Dormand & Prince 5(4)
    "rk23": ([[], [0.5], [0.0, 0.75], [2 / 9, 1 / 3, 4 / 9]], [2 / 9, 1 / 3, 4 / 9, 0.0], [7 / 24, 0.25, 1 / 3, 0.125], 2),
    "rkdp45": ([[], [1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9],
                [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
                [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656],
                [35 / 384, 0.0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]],
               [35 / 384, 0.0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84, 0.0],
               [5179 / 57600, 0.0, 7571 / 16695, 393 / 640, -92097 / 339200, 187 / 2100, 1 / 40], 4),
}


def network(flat, m, B):
    """The network's output (n, H, W, 3) for m (n, 3, H, W), differentiable
    in `flat`: six 3 x 3 convolutions as nine shifted matrix products each,
    SiLU between; inputs m as a 16-bit pair (hi, 256 (m - hi)) and B / 50 mT."""
    n, _, H, W = m.shape
    m32 = m.float()
    hi = m32.bfloat16().float()
    lo = (256 * (m32 - hi)).bfloat16()
    Bn = (torch.as_tensor(B, device=m.device, dtype=torch.float32) / 0.05).bfloat16()
    x = torch.cat([hi.double(), lo.double(), Bn.double()[:, :, None, None].expand(n, 3, H, W)], 1).permute(0, 2, 3, 1)
    o = 0
    for li, (ci, co) in enumerate(LAYERS):
        w = flat[o:o + co * ci * 9].reshape(co, ci, 9)
        b = flat[o + co * ci * 9:o + co * ci * 9 + co]
        o += co * ci * 9 + co
        pad = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        y = b.reshape(1, co)
        for u in range(3):
            for v in range(3):
                y = y + pad[:, u:u + H, v:v + W].reshape(-1, ci) @ w[:, :, 3 * u + v].t().contiguous()
        x = (y * torch.sigmoid(y) if li < len(LAYERS) - 1 else y).reshape(n, H, W, co)
    return x


def exact(case, seed):
    c = case
    flat = torch.from_numpy(np.concatenate([v.reshape(-1) for wb in weights() for v in wb])).to(device()).double()
    if c["kind"] in ("film", "heff"):
        f = Film64(problem(c))
        m = unit(start_state((3, c["nz"], c["ny"], c["nx"]), c.get("start", "canted"), seed).double())
        if c["kind"] == "heff":
            return {"h": f.field(m)}
        if c["method"] in FIXED:
            return {"m": f.fixed(m, c["method"], c["dt"], c["steps"])}
        return {"m": f.adaptive(m, c["method"], c["t_end"], 1e-5, 1e-14)}
    if c["kind"] == "batch":
        films = sweep(c)
        return [Film64(p).fixed(unit(m.double()), c["method"], c["dt"], c["steps"])
                for p, m in zip(films, sweep_states(films, seed))]
    if c["kind"] == "advance":
        f = Film64(advance_problem(c))
        m = unit(start_state((3, 1, c["H"], c["W"]), "uniform", seed).double())
        B = np.array([advance_problem(c)["B"]])
        left = c["segments"]
        while left > 0:      # a round: the chain of proposals, then the last one's plain segment
            w = min(left, c["window"])
            for _ in range(w - 1):
                z = network(flat, m[:, 0][None], B)[0].permute(2, 0, 1)[:, None]
                m = unit(f.fixed(m, "rk4", 1e-12, 1) + 1e-4 * z)
            m = f.fixed(m, "rk4", 1e-13, 10)
            left -= w
        return {"m": m}
    m, base, target, B = (v.double() if torch.is_tensor(v) else v for v in states(c, seed))
    if c["kind"] == "predict":
        return {"m": unit(base + 1e-4 * network(flat, m, B).permute(0, 3, 1, 2), 1)}
    flat.requires_grad_(True)
    loss, n = 0.0, m.shape[0]
    for i in range(0, n, 4):     # four states at a time
        z = network(flat, m[i:i + 4], B[i:i + 4]).permute(0, 3, 1, 2)
        part = ((z - (target[i:i + 4] - base[i:i + 4]) * 1e4) ** 2).sum() / m.numel()
        part.backward()
        loss += float(part.detach())
    g = flat.grad
    with torch.no_grad():        # the first Adam step from zero moments
        p = flat - 1e-3 * g / (g.abs() + 1e-8)
    return {"loss": loss, "grads": g, "params": p.detach()}
