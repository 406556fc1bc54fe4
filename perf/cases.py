"""Performance cases of the lattice Boltzmann library, through its public entry points.

listed() gives the fixed cases, draw(rng) one more case of the same ranges,
prepare(case, seed) what a user's program holds before the call, run(state) one
pass, work(case) the bytes and operations a pass cannot do without, and
exact(case, seed) the outputs as plain torch / numpy gives them in 64 bits,
from the method's own formulas (arXiv:2410.13165) and none of the package's code.

Kinds of cases:
  evolve     initial field in, `steps` time steps, phi out (Lattice);
  gradient   the same with a checkpoint tape, then the adjoint gradients of a
             final-time misfit (Lattice.tape_gradient);
  autograd   a loss through torch.autograd (autograd.Evolve);
  sweep      many periodic lattices advanced together (Batch), with the moments
             and the field of every instance;
  map        spectral radii over wave-number grids (stability_map).
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

TWO_PI = 2.0 * math.pi


def listed():
    return [
        # the smallest use: the one-dimensional plane wave of the method's first
        # check, where a step is far shorter than a launch
        {"name": "d1_periodic_256", "kind": "evolve", "dims": "256", "bc": "periodic",
         "precision": "fp64", "tau": 0.8, "steps": 1000},
        # the coarse end of the two-dimensional grid refinement study
        {"name": "d2_periodic_64", "kind": "evolve", "dims": "64x64", "bc": "periodic",
         "precision": "fp64", "tau": 0.5, "steps": 64},
        # its fine end, in float32 storage
        {"name": "d2_periodic_2048", "kind": "evolve", "dims": "2048x2048", "bc": "periodic",
         "precision": "fp32", "tau": 0.7, "steps": 64},
        # a Dirichlet problem on an odd-sized two-dimensional grid
        {"name": "d2_fullway_odd", "kind": "evolve", "dims": "333x257", "bc": "fullway",
         "precision": "fp64", "tau": 0.5, "steps": 100},
        # the size at which the three-dimensional workload first reaches a
        # relative error of 1e-6 in float64
        {"name": "d3_fullway_192", "kind": "evolve", "dims": "192x192x192", "bc": "fullway",
         "precision": "fp64", "tau": 0.5, "steps": 48},
        # half-way walls on odd, unequal sizes, an odd number of steps
        {"name": "d3_halfway_odd", "kind": "evolve", "dims": "150x133x121", "bc": "halfway",
         "precision": "fp32", "tau": 0.5, "steps": 31},
        # the benchmark workload in its headline storage mode
        {"name": "d3_fullway_512", "kind": "evolve", "dims": "512x512x512", "bc": "fullway",
         "precision": "fp32_split", "tau": 0.5, "steps": 32},
        # the four-dimensional example at benchmark size
        {"name": "d4_fullway_96", "kind": "evolve", "dims": "96x96x96x96", "bc": "fullway",
         "precision": "fp32", "tau": 0.5, "steps": 8},
        # the gradient workload: forward with checkpoints, gradients in phi0 and tau
        {"name": "gradient_d3_256", "kind": "gradient", "dims": "256x256x256",
         "precision": "fp32_split", "tau": 0.5, "steps": 64, "every": 32, "want_tau": True},
        # a small inverse problem through torch.autograd, uneven checkpoints
        {"name": "autograd_d2_128", "kind": "autograd", "dims": "128x120", "precision": "fp64",
         "tau": 0.6, "steps": 60, "every": 7},
        # the stability sweep: lattices of 64^2 to 512^2, noise initial data
        {"name": "sweep_d2_512", "kind": "sweep", "count": 512, "sizes": "64 128 256 512",
         "precision": "fp32", "steps": 100},
        # the stability-region figure: a 61^2 grid of velocities
        {"name": "map_d2_61", "kind": "map", "d": 2, "side": 61, "m": 16, "s": 2.0},
    ]


def _text(dims):
    return "x".join(map(str, dims))


def _dims(case):
    return [int(n) for n in case["dims"].split("x")]


def _sizes(case):
    return [int(n) for n in case["sizes"].split()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evolve1", "evolve2", "evolve2", "evolve3", "evolve3", "evolve3", "evolve4",
                       "gradient", "gradient", "autograd", "sweep", "map"])
    if kind.startswith("evolve"):
        d = int(kind[-1])
        lo, hi, top = {1: (64, 100000, 1 << 62), 2: (32, 2048, 1 << 62),
                       3: (24, 320, 12 << 20), 4: (10, 64, 6 << 20)}[d]
        while True:
            dims = [_log_int(rng, lo, hi) for _ in range(d)]
            if math.prod(dims) <= top:
                break
        bc = rng.choice(["periodic", "fullway", "halfway"] if d > 1 else ["periodic", "fullway"])
        precision = rng.choice({1: ["fp64", "fp32"], 2: ["fp64", "fp32", "fp32_split"],
                                3: ["fp64", "fp32", "fp32_split", "fp32_split", "fp32_hilo"],
                                4: ["fp64", "fp32"]}[d])
        tau = rng.choice([0.5, 0.7, 0.8, 1.2]) if bc == "periodic" else 0.5
        steps = _log_int(rng, *{1: (10, 1000), 2: (10, 200), 3: (4, 64), 4: (3, 12)}[d])
        return {"kind": "evolve", "dims": _text(dims), "bc": bc, "precision": precision, "tau": tau,
                "steps": steps}
    if kind == "gradient":
        dims = [_log_int(rng, 24, 160) for _ in range(3)]
        return {"kind": "gradient", "dims": _text(dims),
                "precision": rng.choice(["fp64", "fp32", "fp32_split"]),
                "tau": rng.choice([0.5, 0.6, 0.8]), "steps": _log_int(rng, 8, 64),
                "every": rng.choice([4, 7, 16, 32]), "want_tau": rng.random() < 0.75}
    if kind == "autograd":
        dims = [_log_int(rng, 40, 600) for _ in range(2)]
        return {"kind": "autograd", "dims": _text(dims), "precision": rng.choice(["fp64", "fp32"]),
                "tau": rng.choice([0.5, 0.6, 0.9]), "steps": _log_int(rng, 10, 100),
                "every": rng.choice([4, 7, 16])}
    if kind == "sweep":
        return {"kind": "sweep", "count": _log_int(rng, 8, 256),
                "sizes": " ".join(map(str, sorted(rng.sample([48, 64, 100, 128, 200, 256, 333, 512],
                                                                4)))),
                "precision": rng.choice(["fp32", "fp32", "fp64"]),
                "steps": _log_int(rng, 10, 100)}
    d = rng.choice([1, 2, 2, 3])
    side = {1: _log_int(rng, 50, 2000), 2: _log_int(rng, 9, 61), 3: _log_int(rng, 4, 13)}[d]
    m = {1: _log_int(rng, 16, 256), 2: _log_int(rng, 8, 32), 3: _log_int(rng, 5, 12)}[d]
    return {"kind": "map", "d": d, "side": side, "m": m, "s": rng.choice([2.0, 2.0, 1.25, 0.9])}


# ------------------------------------------------------------------- inputs --

_U = [0.05, 0.1, 0.08, 0.06]


def _problem(case, seed):
    """Velocity, source, field modes and grid of an evolve case: a sum of cosines
    that is periodic on periodic lattices."""
    dims, bc = _dims(case), case["bc"]
    d = len(dims)
    rng = np.random.default_rng(seed)
    modes = 1 if d == 4 else 4
    # half-way walls are run at a small velocity, where the scheme is stable
    u = [1e-3 * v / 0.05 if bc == "halfway" else v for v in _U[:d]]
    R = 1.0 if bc != "periodic" and d < 4 else 0.0
    lengthen = 2.0 if d == 4 else 1.0
    dx = lengthen / (dims[0] - 1 if bc == "fullway" else dims[0])
    amps = rng.normal(size=modes)
    if bc == "periodic":
        wave = rng.integers(1, 3, size=(modes, d)) * rng.choice([-1, 1], size=(modes, d))
        kvecs = TWO_PI * wave / (np.asarray(dims) * dx)
    elif d == 4:
        kvecs = np.full((modes, d), math.pi)
    else:
        kvecs = TWO_PI * rng.uniform(-1.5, 1.5, size=(modes, d))
    phases = rng.uniform(0.0, TWO_PI, size=modes)
    return {"u": u, "R": R, "dx": dx, "amps": amps, "kvecs": kvecs, "phases": phases,
            "shift": 0.5 if bc == "halfway" else 0.0}


def _axis(n, a, d, dx, shift, device):
    """Coordinates of axis a (x_1 is the last tensor axis), shaped to broadcast."""
    x = (torch.arange(n, dtype=torch.float64, device=device) + shift) * dx
    return x.view([n if b == d - 1 - a else 1 for b in range(d)])


def _initial(case, pr, device):
    """phi0 and its gradient (d, N_d, ..., N_1) of the field at t = 0."""
    dims = _dims(case)
    d = len(dims)
    xs = [_axis(dims[a], a, d, pr["dx"], pr["shift"], device) for a in range(d)]
    shape = list(reversed(dims))
    phi = torch.zeros(shape, dtype=torch.float64, device=device)
    grad = torch.zeros([d] + shape, dtype=torch.float64, device=device)
    for amp, kv, ph in zip(pr["amps"], pr["kvecs"], pr["phases"]):
        arg = ph + sum(float(kv[a]) * xs[a] for a in range(d))
        phi += amp * torch.cos(arg)
        s = amp * torch.sin(arg)
        for a in range(d):
            grad[a] -= float(kv[a]) * s
    return phi, grad


def _smooth(dims, seed, device="cuda", corr=0.1):
    """Periodic Gaussian random field of unit variance, correlation length corr."""
    g = torch.Generator(device=device).manual_seed(seed)
    shape = list(reversed(dims))
    w = torch.fft.fftn(torch.randn(shape, generator=g, dtype=torch.float64, device=device))
    k2 = 0.0
    for a, n in enumerate(shape):
        k = TWO_PI * torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device=device)
        k2 = k2 + (k * k).view([n if b == a else 1 for b in range(len(shape))])
    f = torch.fft.ifftn(w * torch.exp(-0.25 * k2 * corr * corr)).real
    f = f - f.mean()
    return (f / f.std()).contiguous()


def _specs(case, seed):
    """Instances of a sweep: sizes, tau ~ U(0.5, 2), u ~ U(-0.75, 0.75)^2; the mix
    of sizes is the case's own, the parameters are the seed's."""
    rng, pick = np.random.default_rng(seed), np.random.default_rng(case["count"])
    sizes = _sizes(case)
    out = []
    for _ in range(case["count"]):
        n = sizes[pick.integers(0, len(sizes))]
        out.append({"dims": (n, n), "tau": float(rng.uniform(0.5, 2.0)),
                    "u": rng.uniform(-0.75, 0.75, size=2).tolist(), "dx": 1.0 / n, "K": 1})
    return out


def _noise(specs, seed, device="cuda"):
    g = torch.Generator(device=device).manual_seed(seed)
    n = sum(math.prod(sp["dims"]) for sp in specs)
    return 1e-3 * torch.randn(n, generator=g, dtype=torch.float64, device=device)


def _points(case, seed):
    """Velocities of a map (a grid over [-0.75, 0.75]^d, moved by the seed) and rates s."""
    rng = np.random.default_rng(seed)
    ax = np.linspace(-0.75, 0.75, case["side"])
    pts = np.stack(np.meshgrid(*([ax] * case["d"]), indexing="ij"), -1).reshape(-1, case["d"])
    return pts + rng.uniform(-0.01, 0.01, size=case["d"]), np.full(len(pts), case["s"])


def prepare(case, seed):
    import paper_2410_13165_amd as lb
    kind = case["kind"]
    if kind == "map":
        pts, s = _points(case, seed)
        return {"kind": kind, "map": lb.stability_map, "m": case["m"],
                "pts": torch.from_numpy(pts).cuda(), "s": torch.from_numpy(s).cuda()}
    if kind == "sweep":
        specs = _specs(case, seed)
        return {"kind": kind, "batch": lb.Batch(2, specs, precision=case["precision"]),
                "phi0": _noise(specs, seed), "steps": case["steps"], "count": case["count"]}
    dims = tuple(_dims(case))
    d = len(dims)
    if kind == "evolve":
        pr = _problem(case, seed)
        phi0, grad0 = _initial(case, pr, "cuda")
        walls = case["bc"] != "periodic"
        field = {"kind": "cos_sum", "amps": pr["amps"], "kvecs": pr["kvecs"],
                 "phases": pr["phases"]} if walls else None
        lat = lb.Lattice(d, dims, case["tau"], dx=pr["dx"], u=pr["u"], R=pr["R"],
                         bc=[case["bc"]] * d, precision=case["precision"], field=field)
        return {"kind": kind, "lat": lat, "phi0": phi0, "grad0": grad0 if walls else None,
                "steps": case["steps"]}
    phi0, target = _smooth(dims, seed), _smooth(dims, seed + 1000003)
    dx = 1.0 / dims[0]
    if kind == "gradient":
        lat = lb.Lattice(d, dims, case["tau"], dx=dx, u=_U[:d], precision=case["precision"])
        return {"kind": kind, "lat": lat, "phi0": phi0, "target": target, "vol": dx ** d,
                "steps": case["steps"], "every": case["every"], "tau": case["want_tau"]}
    from paper_2410_13165_amd.autograd import Evolve
    kw = {"d": d, "dims": dims, "dx": dx, "u": _U[:d], "precision": case["precision"]}
    return {"kind": kind, "fn": Evolve, "kw": kw, "phi0": phi0.requires_grad_(True),
            "tau": torch.tensor(case["tau"], dtype=torch.float64, requires_grad=True),
            "target": target, "vol": dx ** d, "steps": case["steps"], "every": case["every"]}


def run(state):
    kind = state["kind"]
    if kind == "evolve":
        lat = state["lat"]
        lat.set_initial(state["phi0"], state["grad0"])
        lat.step(state["steps"])
        return lat.phi()
    if kind == "gradient":
        lat = state["lat"]
        lat.set_initial(state["phi0"])
        lat.tape_begin(state["every"])
        lat.step(state["steps"])
        phi = lat.phi()
        g = lat.tape_gradient((phi - state["target"]) * state["vol"], want_phi0=True,
                              want_tau=state["tau"])
        lat.tape_end()
        return {"phi": phi, **g}
    if kind == "autograd":
        state["phi0"].grad = state["tau"].grad = None
        phi = state["fn"].apply(state["phi0"], state["tau"], state["kw"], state["steps"],
                                state["every"])
        loss = 0.5 * (phi - state["target"]).pow(2).sum() * state["vol"]
        loss.backward()
        return {"phi": phi.detach(), "phi0": state["phi0"].grad, "tau": state["tau"].grad}
    if kind == "sweep":
        b = state["batch"]
        b.set_initial(state["phi0"])
        b.step(state["steps"])
        m = b.moments()
        return {"sum_phi": m[:, 0], "sum_phi2": m[:, 1], "entropy": m[:, 3], "max_phi": m[:, 4],
                "phi": torch.cat([b.instance(i).phi().view(-1) for i in range(state["count"])])}
    return state["map"](state["pts"], state["s"], m=state["m"])


def work(case):
    """Inputs read once, outputs written once; 5 operations per population, node
    and step (the sum, and the relaxation's two multiply-adds)."""
    kind = case["kind"]
    if kind == "map":
        d, q = case["d"], 2 * case["d"] ** 2 + 1
        n = case["side"] ** d
        # per matrix: a few sweeps over q roots and q poles, tens of operations each
        return {"bytes": n * (8.0 * (d + 1) + 20.0),
                "flops": 5.0 * 50.0 * q * q * n * case["m"] ** d}
    if kind == "sweep":
        nodes = case["count"] * float(np.mean(np.square(_sizes(case))))
        return {"bytes": 16.0 * nodes, "flops": 45.0 * nodes * case["steps"]}
    nodes = float(math.prod(_dims(case)))
    d = len(_dims(case))
    flops = 5.0 * (2 * d * d + 1) * nodes * case["steps"]
    if kind == "evolve":
        inputs = 8.0 * (1 if case["bc"] == "periodic" else 1 + d)
        return {"bytes": nodes * (inputs + 8.0), "flops": flops}
    # forward, transposed steps and the contraction for tau
    return {"bytes": nodes * 32.0, "flops": 3.0 * flops}


# -------------------------------------------------------- 64-bit references --

def _velocities(d):
    """Rest, +e_a, -e_a, then (1,1), (-1,1), (-1,-1), (1,-1) of each pair of axes."""
    e = np.eye(d, dtype=int)
    vs = [np.zeros(d, int)] + [e[a] for a in range(d)] + [-e[a] for a in range(d)]
    for i, j in itertools.combinations(range(d), 2):
        vs += [e[i] + e[j], -e[i] + e[j], -e[i] - e[j], e[i] - e[j]]
    return [tuple(int(x) for x in v) for v in vs]


def _weights(u):
    """Equilibrium weights from the moments 1, u, u^2 on the diagonal of the
    second, the third u_i m2 = u_i / 3 and one fourth-order moment, at its middle
    value (the paper's entropy-stable choice), for unit lattice speed."""
    u = np.asarray(u, float)
    d = len(u)
    s2 = float(u @ u)
    m4 = 0.0
    if d > 1:
        lo = [(-6.0 + 2.0 * d + 4.0 * s2) / (3.0 * d * (d - 1))]
        for i, j in itertools.combinations(range(d), 2):
            lo += [(abs(u[i] + u[j]) - 2.0 * u[i] * u[j]) / 3.0,
                   (abs(u[i] - u[j]) + 2.0 * u[i] * u[j]) / 3.0]
        hi = min((1.0 + 2.0 * v * v - abs((4 - d) * v)) / (3.0 * (d - 1)) for v in u)
        m4 = 0.5 * max(lo) + 0.5 * hi
    w = []
    for c in _velocities(d):
        ax = [a for a in range(d) if c[a]]
        if not ax:
            w.append(1.0 - d / 3.0 - 2.0 * s2 / 3.0 + 0.5 * d * (d - 1) * m4)
        elif len(ax) == 1:
            v = u[ax[0]]
            w.append((c[ax[0]] * (4 - d) * v + 1.0 + 2.0 * v * v - 3.0 * (d - 1) * m4) / 6.0)
        else:
            a, b = c[ax[0]] * u[ax[0]], c[ax[1]] * u[ax[1]]
            w.append((3.0 * m4 + 2.0 * a * b + a + b) / 12.0)
    return w


def _roll(f, c, sign=1):
    """f(x - sign c) on the periodic grid; tensor axis d - 1 - a holds x_{a+1}."""
    d = len(c)
    ax = [a for a in range(d) if c[a]]
    off = f.dim() - d
    return torch.roll(f, [sign * c[a] for a in ax], [off + d - 1 - a for a in ax]) if ax else f


class _Walls:
    """The Dirichlet data of the fourth-order wall schemes, mode by mode: a
    derivative of Re(A exp(i theta)) along c is a product with i kappa . c, one in
    time a product with -i kappa . u."""

    def __init__(self, case, pr, device):
        self.half, self.pr = case["bc"] == "halfway", pr
        dims = _dims(case)
        d = len(dims)
        shape = list(reversed(dims))
        idx = [torch.arange(dims[a], device=device).view([dims[a] if b == d - 1 - a else 1
                                                          for b in range(d)]) for a in range(d)]
        edge = torch.zeros(shape, dtype=torch.bool, device=device)
        for a in range(d):
            edge |= (idx[a] == 0) | (idx[a] == dims[a] - 1)
        nodes = edge.reshape(-1).nonzero().squeeze(1)
        i, rest = [], nodes
        for a in range(d):
            i.append(rest % dims[a])
            rest = rest // dims[a]
        self.vel, self.w = _velocities(d), _weights(pr["u"])
        self.opp = [self.vel.index(tuple(-v for v in c)) for c in self.vel]
        self.nodes, self.x = [], []
        for c in self.vel:
            out = torch.zeros_like(nodes, dtype=torch.bool)
            for a in range(d):
                if c[a]:
                    out |= i[a] == (0 if c[a] > 0 else dims[a] - 1)
            sel = out.nonzero().squeeze(1)
            self.nodes.append(nodes[sel])
            self.x.append([(i[a][sel].double() + pr["shift"]) * pr["dx"] for a in range(d)])

    def apply(self, new, k, step, post):
        """Replace the entering values of population k after step -> step + 1;
        post: this step's post-collision value of the opposite population."""
        pr, c = self.pr, self.vel[k]
        if self.nodes[k].numel() == 0:
            return
        dt, u, R = pr["dx"], pr["u"], pr["R"]
        t = (step if self.half else step + 1) * dt
        xs = [x - (0.5 * c[a] * pr["dx"] if self.half else 0.0) for a, x in enumerate(self.x[k])]
        wp, wm = self.w[k] + self.w[self.opp[k]], self.w[k] - self.w[self.opp[k]]
        val = torch.zeros_like(xs[0])
        for amp, kv, ph in zip(pr["amps"], pr["kvecs"], pr["phases"]):
            theta = ph + sum(float(kv[a]) * (xs[a] - u[a] * t) for a in range(len(u)))
            dc = dt * 1j * sum(float(kv[a]) * c[a] for a in range(len(u)))
            dts = -dt * 1j * sum(float(kv[a]) * u[a] for a in range(len(u)))
            if self.half:
                z = (wp * (1 + dts / 2 - dc ** 2 / 8 - dc ** 2 * dts / 16 - dts ** 3 / 24)
                     + wm * (-dc * dts / 4 - dc * dts ** 2 / 8))
            else:
                z = self.w[k] * (1 - (dts + dc) / 2 + (dts + dc) ** 3 / 24)
            val += amp * (z.real * torch.cos(theta) - z.imag * torch.sin(theta))
        if self.half:
            val += wp * R * (t + dt) - post.reshape(-1)[self.nodes[k]]
        else:
            val += self.w[k] * R * t
        new.view(-1)[self.nodes[k]] = val


def _evolve(f, w, vel, s, dt, R, steps, walls=None):
    """`steps` collide-and-stream steps of the populations f (a list, changed in place)."""
    opp = [vel.index(tuple(-v for v in c)) for c in vel]
    for n in range(steps):
        phi = sum(f[1:], f[0].clone())
        for k in range(len(vel)):
            f[k].mul_(1.0 - s).add_(phi * (s * w[k])).add_(dt * R * w[k])
        if walls is None:
            for k, c in enumerate(vel):
                f[k] = _roll(f[k], c)
            continue
        for k in range(len(vel)):
            if k > opp[k]:
                continue
            a, b = f[k], f[opp[k]]
            na = _roll(a, vel[k]) if opp[k] != k else a
            nb = _roll(b, vel[opp[k]])
            if opp[k] != k:
                walls.apply(na, k, n, b)
                walls.apply(nb, opp[k], n, a)
                f[opp[k]] = nb
            f[k] = na
    return f


def _start(phi, grad, u, w, vel, tau, dt):
    """omega_k [phi + tau dt (u - c_k) . grad phi]"""
    return [w[k] * (phi + tau * dt * sum((u[a] - c[a]) * grad[a] for a in range(len(u))))
            for k, c in enumerate(vel)]


def _difference(phi, a, dx):
    """Fourth-order central difference along axis a on the periodic grid."""
    ax = phi.dim() - 1 - a
    return (8.0 * (torch.roll(phi, -1, ax) - torch.roll(phi, 1, ax))
            - torch.roll(phi, -2, ax) + torch.roll(phi, 2, ax)) / (12.0 * dx)


def _exact_evolve(case, seed):
    pr = _problem(case, seed)
    vel, w = _velocities(len(_dims(case))), _weights(pr["u"])
    phi, grad = _initial(case, pr, "cuda")
    walls = None
    if case["bc"] == "periodic":
        grad = [_difference(phi, a, pr["dx"]) for a in range(len(_dims(case)))]
    else:
        walls = _Walls(case, pr, "cuda")
    f = _start(phi, grad, pr["u"], w, vel, case["tau"], pr["dx"])
    del phi, grad
    f = _evolve(f, w, vel, 1.0 / case["tau"], pr["dx"], pr["R"], case["steps"], walls)
    return sum(f[1:], f[0].clone())


def _exact_gradient(case, seed, with_tau):
    """phi^N, dL/dphi0 by the transposed steps, dL/dtau by the linearised ones."""
    dims = _dims(case)
    d = len(dims)
    u, dt, tau = _U[:d], 1.0 / dims[0], case["tau"]
    s = 1.0 / tau
    vel, w = _velocities(d), _weights(u)
    phi0, target = _smooth(dims, seed), _smooth(dims, seed + 1000003)
    grad = [_difference(phi0, a, dt) for a in range(d)]
    f = _start(phi0, grad, u, w, vel, tau, dt)
    df = [(f[k] - w[k] * phi0) / tau for k in range(len(vel))]
    for _ in range(case["steps"]):
        phi, dphi = sum(f[1:], f[0].clone()), sum(df[1:], df[0].clone())
        for k, c in enumerate(vel):
            df[k] = _roll((1.0 - s) * df[k] + s * w[k] * dphi - (w[k] * phi - f[k]) * s * s, c)
            f[k] = _roll((1.0 - s) * f[k] + s * w[k] * phi, c)
    phi = sum(f[1:], f[0].clone())
    seed_ = (phi - target) * dt ** d
    dtau = float((seed_ * sum(df[1:], df[0].clone())).sum())
    del f, df
    lam = [seed_.clone() for _ in vel]
    for _ in range(case["steps"]):
        nu = [_roll(lam[k], c, -1) for k, c in enumerate(vel)]
        m = sum(w[k] * nu[k] for k in range(len(vel)))
        lam = [(1.0 - s) * nu[k] + s * m for k in range(len(vel))]
    g = sum(w[k] * lam[k] for k in range(len(vel)))
    for a in range(d):
        h = tau * dt * sum(w[k] * (u[a] - c[a]) * lam[k] for k, c in enumerate(vel))
        g = g - _difference(h, a, dt)
    return {"phi": phi, "phi0": g, **({"tau": dtau} if with_tau else {})}


def _exact_sweep(case, seed):
    specs = _specs(case, seed)
    flat = _noise(specs, seed)
    vel = _velocities(2)
    fields, scalars = [None] * len(specs), np.zeros((len(specs), 4))
    starts = np.concatenate([[0], np.cumsum([math.prod(sp["dims"]) for sp in specs])])
    for n in sorted({sp["dims"][0] for sp in specs}):
        ids = [i for i, sp in enumerate(specs) if sp["dims"][0] == n]

        def column(values):
            return torch.tensor(values, dtype=torch.float64, device="cuda").view(-1, 1, 1)
        ws = np.array([_weights(specs[i]["u"]) for i in ids])
        w = [column(ws[:, k].tolist()) for k in range(len(vel))]
        s = column([1.0 / specs[i]["tau"] for i in ids])
        phi0 = torch.stack([flat[starts[i]:starts[i] + n * n].view(n, n) for i in ids])
        f = [w[k] * phi0 for k in range(len(vel))]
        for _ in range(case["steps"]):
            phi = sum(f[1:], f[0].clone())
            f = [_roll((1.0 - s) * f[k] + s * w[k] * phi, c) for k, c in enumerate(vel)]
        phi = sum(f[1:], f[0].clone())
        ent = sum((f[k] ** 2 / (2.0 * w[k])).sum((1, 2)) for k in range(len(vel)))
        cols = [phi.sum((1, 2)), (phi ** 2).sum((1, 2)), ent, phi.abs().amax((1, 2))]
        scalars[ids] = torch.stack(cols, 1).cpu().numpy()
        for j, i in enumerate(ids):
            fields[i] = phi[j]
    # the sum is conserved near 0: on an unstable instance it holds only rounding
    return {"sum_phi": None, "sum_phi2": scalars[:, 1], "entropy": scalars[:, 2],
            "max_phi": scalars[:, 3], "phi": torch.cat([f.reshape(-1) for f in fields])}


def _exact_map(case, seed):
    pts, s = _points(case, seed)
    d, m = case["d"], case["m"]
    vel = np.array(_velocities(d))
    w = np.array([_weights(p) for p in pts])
    out = {"rho": None, "min_omega": torch.from_numpy(w.min(1)), "unconverged": None}
    js = np.array(list(itertools.product(range(m), repeat=d)))
    js = js[[tuple(j) <= tuple((-j) % m) for j in js]]  # rho(-xi) = rho(xi)
    if len(js) * len(pts) * len(vel) ** 3 > 6e8:
        return out
    T = np.exp(-2j * np.pi / m * (js @ vel.T))
    rho = np.zeros(len(pts))
    for p in range(len(pts)):
        C = (1.0 - s[p]) * np.eye(len(vel)) + s[p] * np.outer(w[p], np.ones(len(vel)))
        rho[p] = np.abs(np.linalg.eigvals(T[:, :, None] * C)).max()
    out["rho"] = torch.from_numpy(rho)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "evolve":
        return _exact_evolve(case, seed)
    if kind in ("gradient", "autograd"):
        return _exact_gradient(case, seed, kind == "autograd" or case["want_tau"])
    if kind == "sweep":
        return _exact_sweep(case, seed)
    return _exact_map(case, seed)
