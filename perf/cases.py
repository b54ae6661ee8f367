"""The work a program has this library do, as cases that can be timed.

Every case goes through the public entry points of ``paper_1602_09079_amd.dg`` (``Solver`` and
``MLP``).  A case's ``kind`` says which call one pass makes:

* ``step``: SSP-RK3 steps with the device-side CFL time step, in place (``Solver.step_async``); the
  options are the driving source, the positivity limiter with the isothermal reset, and the learned
  closure (k = 1);
* ``rhs``: one evaluation of the spatial operator (``Solver.rhs``);
* ``diag``: what a run writes out between steps: conserved totals, velocity power spectrum, density
  PDF and rms Mach number;
* ``train``: one training iteration of the closure's network (``MLP.loss_grad`` and ``MLP.adam``).

``exact`` evaluates the same passes in FP64 with plain torch operations.
"""
import math

import numpy as np
import torch

from paper_1602_09079_amd import dg

GAMMA = 5.0 / 3.0
GAMMA_ISO = 1.01      # the isothermal runs (arXiv 1602.09079, Sec. 3.2)
CFL = 0.3
MACH = 0.3
DRIVE_A0 = 0.03       # driving amplitude of the benchmark
HIDDEN = (128, 128)   # hidden layers of the closure's network
LR = 1e-3
TRAIN_ROWS = 131072   # training samples held on the device
TRAIN_STEP = 100      # a training iteration some way into the run
NOISE = 0.1           # input noise of the training (standardised units)
PDF_BINS = 100


def listed():
    return [
        # the smallest run: an advected density wave, FP64, ten steps in one call; launches and latency
        _solver("wave_k1_16_fp64", 1, (16, 16, 16), "fp64", nsteps=10, wave=True),
        # driven subsonic turbulence at third order, the middle-sized run, in both storage types
        _solver("driven_k2_64_fp64", 2, (64, 64, 64), "fp64", force=True),
        _solver("driven_k2_64_fp32", 2, (64, 64, 64), "fp32", force=True),
        # the paper's own set-up (gamma = 1.01, isothermal reset and limiter), on a mesh with no round sizes
        _solver("paper_k2_ragged_fp32", 2, (90, 77, 51), "fp32", force=True, iso=True),
        # fourth order with reduced-precision contractions
        _solver("driven_k3_128_bf16", 3, (128, 128, 128), "bf16", force=True),
        # one operator evaluation for a caller's own time integrator: FP64, ragged mesh
        _solver("operator_k3_ragged_fp64", 3, (100, 62, 45), "fp64", kind="rhs"),
        # the production run: the largest mesh, FP32-grade tier
        _solver("driven_k3_256_bf16x3", 3, (256, 256, 256), "bf16x3", force=True),
        # fifth order
        _solver("driven_k4_64_fp32", 4, (64, 64, 64), "fp32", force=True),
        # the first-order finite-volume scheme that DG is compared with, on the largest mesh
        _solver("fv_k0_256_fp32", 0, (256, 256, 256), "fp32", force=True),
        # an under-resolved run with the learned closure switched on
        _solver("closure_k1_64_fp32", 1, (64, 64, 64), "fp32", force=True, closure=True),
        # training that closure: one iteration at its usual batch
        {"name": "train_4096", "kind": "train", "batch": 4096, "h1": HIDDEN[0], "h2": HIDDEN[1]},
        # the diagnostics of a run's output times, on the 4x finer sample grid
        _solver("diag_k2_64_fp32", 2, (64, 64, 64), "fp32", kind="diag"),
    ]


def _solver(name, k, n, prec, kind="step", nsteps=1, force=False, iso=False, closure=False, wave=False):
    c = {"name": name} if name else {}
    return {**c, "kind": kind, "k": k, "nx": n[0], "ny": n[1], "nz": n[2], "prec": prec, "nsteps": nsteps,
            "force": force, "iso": iso, "closure": closure, "wave": wave}


# the most cells drawn at each degree: no dearer than the production run
_MOST = {0: 256 ** 3, 1: 160 ** 3, 2: 128 ** 3, 3: 112 ** 3, 4: 64 ** 3}


def draw(rng):
    what = rng.choice(("step",) * 8 + ("closure", "closure", "rhs", "rhs", "train", "train", "diag"))
    if what == "train":
        return {"kind": "train", "batch": int(round(2 ** rng.uniform(7, 14))), "h1": rng.choice((64, 100, 128, 128)),
                "h2": rng.choice((64, 72, 128, 128))}
    k = 1 if what == "closure" else rng.choice((0, 1, 1, 2, 2, 2, 3, 3, 3, 4))
    prec = rng.choice(("fp32", "fp64") if k in (0, 4) else ("fp32", "fp32", "fp64", "bf16x3", "bf16"))
    if what == "closure":
        prec = "fp32"
    if what == "diag":
        m = rng.randrange(16, 73)
        return _solver(None, k, (m, m, m), rng.choice(("fp32", "fp64")), kind="diag")
    cells = math.exp(rng.uniform(math.log(16 ** 3), math.log(96 ** 3 if what == "closure" else _MOST[k])))
    side = cells ** (1 / 3)
    fx, fy = math.exp(rng.uniform(-0.4, 0.4)), math.exp(rng.uniform(-0.4, 0.4))
    n = [max(8, int(side * fx)), max(8, int(side * fy)), max(8, int(side / (fx * fy)))]
    if rng.random() < 0.3:
        n = [max(8, 8 * round(v / 8)) for v in n]
    force = rng.random() < 0.7
    return _solver(None, k, n, prec, kind="rhs" if what == "rhs" else "step",
                   nsteps=rng.choice((1, 1, 1, 5)) if cells < 40000 else 1, force=force,
                   iso=what == "step" and k > 0 and rng.random() < 0.25, closure=what == "closure")


# ------------------------------------------------------------------ inputs

def _rng(seed, salt=0):
    return np.random.default_rng([seed, salt])


def _fourier(seed):
    """Random Fourier modes: wave vectors [m][3], solenoidal velocity amplitudes [m][3] and scalar
    amplitudes [m], all complex, with a k^(-5/3) shell spectrum on 1 <= |n| <= 6."""
    r = _rng(seed)
    nv = []
    while len(nv) < 48:
        v = r.integers(-6, 7, 3)
        if 1 <= v @ v <= 36:
            nv.append(v)
    nv = np.array(nv, dtype=np.float64)
    kk = (nv * nv).sum(1)
    amp = kk ** (-11.0 / 12.0)
    a = (r.standard_normal((48, 3)) + 1j * r.standard_normal((48, 3))) * amp[:, None]
    a -= nv * ((a * nv).sum(1) / kk)[:, None]
    s = (r.standard_normal(48) + 1j * r.standard_normal(48)) * amp
    return nv, a / math.sqrt(0.5 * (abs(a) ** 2).sum()), s / math.sqrt(0.5 * (abs(s) ** 2).sum())


def _points(case, dtype, seed):
    """Point values [5][c][b][a][z][y][x] at the Gauss points, in ``dtype``: a density wave, or
    turbulence at rms Mach number 0.3 with 5 % density fluctuations and p = rho^gamma."""
    k, n = case["k"], (case["nx"], case["ny"], case["nz"])
    q = k + 1
    xi = np.polynomial.legendre.leggauss(q)[0]
    gamma = GAMMA_ISO if case["iso"] else GAMMA
    out = torch.empty((5, q, q, q, n[2], n[1], n[0]), dtype=dtype, device="cuda")
    axis = [[torch.tensor((np.arange(n[d]) + 0.5 * (1 + xi[j])) / n[d], dtype=torch.float64, device="cuda")
             for j in range(q)] for d in range(3)]
    if case["wave"]:
        shift = float(_rng(seed).random())
    else:
        nv, av, sc = _fourier(seed)
        amps = torch.tensor(np.concatenate([av.T * MACH * math.sqrt(gamma), 0.05 * sc[None]]), device="cuda")
        phase = [[torch.exp(2j * math.pi * torch.outer(p, torch.tensor(nv[:, d], device="cuda"))) for p in axis[d]]
                 for d in range(3)]
    for c in range(q):
        for b in range(q):
            for a in range(q):
                if case["wave"]:
                    ph = axis[2][c][:, None, None] + axis[1][b][:, None] + axis[0][a] + shift
                    rho = 1 + 0.1 * torch.sin(2 * math.pi * ph)
                    vel = [torch.ones_like(rho)] * 3
                    p = torch.ones_like(rho)
                else:
                    zy = (phase[2][c][:, None, :] * phase[1][b][None]).reshape(n[2] * n[1], -1)
                    px = torch.cat([phase[0][a].real, -phase[0][a].imag], 1).T
                    f = []
                    for m in range(4):
                        w = zy * amps[m]
                        f.append((torch.cat([w.real, w.imag], 1) @ px).reshape(n[2], n[1], n[0]))
                        del w
                    vel, rho = f[:3], 1 + f[3]
                    p = rho ** gamma
                out[0, c, b, a] = rho
                e = p / (gamma - 1)
                for d in range(3):
                    out[1 + d, c, b, a] = rho * vel[d]
                    e = e + 0.5 * rho * vel[d] * vel[d]
                out[4, c, b, a] = e
    return out


def _driving(seed):
    """Solenoidal driving amplitudes on 1 < |n| < 3: wave vectors [m][3] and ahat [m][3][2]."""
    nv = np.array([(x, y, z) for z in range(-2, 3) for y in range(-2, 3) for x in range(-2, 3)
                   if 1 < x * x + y * y + z * z < 9 and (x, y, z) > (0, 0, 0)], dtype=np.int32)
    th = _rng(seed, 1).standard_normal((len(nv), 3, 2))
    kk = (nv * nv).sum(1).astype(np.float64)
    prof = 1 - (np.sqrt(kk) - 2) ** 2
    ah = th - nv[:, :, None] * ((th * nv[:, :, None]).sum(1) / kk[:, None])[:, None, :]
    return nv, DRIVE_A0 * prof[:, None, None] * ah


def _params(shape, r):
    """Xavier-uniform weights and small biases, packed W1 b1 W2 b2 W3 b3."""
    parts = []
    for i, o in zip(shape[:-1], shape[1:]):
        lim = math.sqrt(6.0 / (i + o))
        parts += [r.uniform(-lim, lim, (o, i)).ravel(), 0.05 * r.standard_normal(o)]
    return np.concatenate(parts).astype(np.float32)


def _closure(canon, seed):
    """A closure for the state canon[5][4][z][y][x]: parameters, feature mean and deviation, output
    scale and bound.  A feature's statistics are the same for every neighbour (periodic mesh)."""
    w = canon.double().reshape(20, -1)
    mean, std = w.mean(1).cpu().numpy(), w.std(1, correction=0).cpu().numpy()
    f32 = lambda a: a.astype(np.float32)
    return (_params((140, *HIDDEN, 20), _rng(seed, 2)), f32(np.tile(mean, 7)), f32(np.tile(std, 7)), f32(0.5 * std),
            np.full(20, 16, np.float32))


def prepare(case, seed):
    if case["kind"] == "train":
        return _train_state(case, seed)
    f64 = case["prec"] == "fp64"
    s = dg.Solver(case["k"], (case["nx"], case["ny"], case["nz"]), gamma=GAMMA_ISO if case["iso"] else GAMMA, cfl=CFL,
                  precision=case["prec"], forcing=case["force"], limit=case["iso"], isothermal=case["iso"],
                  closure=case["closure"])
    if case["force"]:
        s.set_forcing(*_driving(seed))
    if case["iso"]:
        s.set_isothermal(1.0, 1.0)
    y = s.project(_points(case, torch.float64 if f64 else torch.float32, seed))
    if case["closure"]:
        s.set_closure(*_closure(s.export_state(y), seed))
    state = {"case": case, "solver": s, "y": y}
    if case["kind"] == "rhs":
        state["r"] = s.empty_state()
    elif case["kind"] == "diag":
        nb = dg.lib().dg_spectrum_workspace_bytes(s._ctx, 4)
        state["work"] = torch.empty(nb, dtype=torch.uint8, device="cuda")
    else:
        s.workspace()
    return state


def _train_state(case, seed):
    shape = (140, case["h1"], case["h2"], 20)
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = torch.tensor(_params(shape, _rng(seed, 3)), device="cuda")
    rand = lambda *n: torch.randn(*n, generator=g, device="cuda")
    return {"case": case, "net": dg.MLP(shape, case["batch"]), "params": p, "x": rand(TRAIN_ROWS, 140),
            "t": rand(TRAIN_ROWS, 20), "m": 1e-4 * rand(p.numel()), "v": 1e-6 * (0.5 + rand(p.numel()) ** 2),
            "grad": torch.empty_like(p), "loss": torch.empty((), dtype=torch.float64, device="cuda"),
            "perm": torch.randperm(TRAIN_ROWS, generator=g, device="cuda").int(), "it": TRAIN_STEP, "seed": seed}


def run(state):
    case = state["case"]
    if case["kind"] == "train":
        st, b = state, case["batch"]
        at = (st["it"] - TRAIN_STEP) % (TRAIN_ROWS // b) * b
        st["it"] += 1
        st["net"].loss_grad(st["params"], st["x"], st["t"], rows=st["perm"][at:at + b], grad=st["grad"],
                            loss=st["loss"], noise=NOISE, seed=st["seed"] * 1000003 + st["it"])
        st["net"].adam(st["params"], st["grad"], st["m"], st["v"], st["it"], lr=LR)
        return [st["grad"], st["params"], st["m"], st["v"]]
    s, y = state["solver"], state["y"]
    if case["kind"] == "rhs":
        return s.rhs(y, out=state["r"])
    if case["kind"] == "diag":
        return {"totals": s.totals(y), "spectrum": s.velocity_spectrum(y, 4, work=state["work"]),
                "pdf": s.density_pdf(y, 4, -0.2, 0.2, PDF_BINS), "mach": s.rms_mach(y, 4)}
    s.step_async(y, case["nsteps"])
    return y


def work(case):
    if case["kind"] == "train":
        b, net = case["batch"], 140 * case["h1"] + case["h1"] * case["h2"] + case["h2"] * 20
        # rows in; the parameters, gradient and both moments out, the parameters and moments in
        return {"bytes": 4.0 * (160 * b + 7 * net), "flops": 2.0 * b * (3 * net - 140 * case["h1"])}
    k, cells = case["k"], case["nx"] * case["ny"] * case["nz"]
    n, q, p = (k + 1) * (k + 2) * (k + 3) // 6, (k + 1) ** 3, (k + 1) ** 2
    elem = 8 if case["prec"] == "fp64" else 4
    state = 5.0 * n * cells * elem
    if case["kind"] == "diag":
        m = 64.0 * cells  # sample points; one real transform per velocity component
        return {"bytes": state, "flops": m * (2 * 5 * n + 3 * 2.5 * math.log2(m))}
    # contractions of one operator evaluation (an FMA counts 2): point values, volume integral,
    # driving source, face traces and lift; then the point and face fluxes
    f = 2 * 5 * n * q * 4 + 2 * 6 * 5 * n * p * 2 + 40 * q + 60 * 3 * p + (8 * n * q if case["force"] else 0)
    if case["closure"]:
        f += 2 * (140 * HIDDEN[0] + HIDDEN[0] * HIDDEN[1] + HIDDEN[1] * 20)
    return {"bytes": 2 * state, "flops": float(f) * cells * (1 if case["kind"] == "rhs" else 3 * case["nsteps"])}


# ------------------------------------------------------------------ the same in 64 bits

def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    ref = _Exact(case, seed)
    if case["kind"] == "rhs":
        return ref.out(ref.rhs(ref.y))
    if case["kind"] == "diag":
        return ref.diagnostics()
    for _ in range(case["nsteps"]):
        ref.step()
    return ref.out(ref.y)


def _legendre(u, x):
    """The scaled Legendre polynomial sqrt(2u+1) P_u and its derivative at x."""
    c = np.zeros(u + 1)
    c[u] = math.sqrt(2 * u + 1)
    return np.polynomial.legendre.legval(x, c), np.polynomial.legendre.legval(x, np.polynomial.legendre.legder(c))


class _Exact:
    """The modal DG scheme in FP64 on canonical states [5][l][z][y][x] (arXiv 1602.09079, Sec. 2)."""

    def __init__(self, case, seed):
        self.case, self.k, self.n = case, case["k"], (case["nx"], case["ny"], case["nz"])
        self.gamma = GAMMA_ISO if case["iso"] else GAMMA
        k = self.k
        self.modes = [(u, v, d - u - v) for d in range(k + 1) for u in range(d, -1, -1) for v in range(d - u, -1, -1)]
        self.xi, self.om = np.polynomial.legendre.leggauss(k + 1)
        q = k + 1
        dev = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda")
        pts = [(a, b, c) for c in range(q) for b in range(q) for a in range(q)]
        self.pts = pts
        x = np.array([[self.xi[i] for i in p] for p in pts])
        self.w3 = np.array([np.prod([self.om[i] for i in p]) for p in pts]) / 8
        val, grad = self.basis(x)
        self.V, self.G = dev(val), [dev((g * self.w3[:, None]).T) for g in grad]
        self.PW = dev((val * self.w3[:, None]).T)
        self.face, self.lift = [], []
        w2 = np.array([self.om[i] * self.om[j] for j in range(q) for i in range(q)]) / 4
        for ax in range(3):
            for side in (-1.0, 1.0):
                f = np.array([np.insert([self.xi[i], self.xi[j]], ax, side) for j in range(q) for i in range(q)])
                v = self.basis(f)[0]
                self.face.append(dev(v))
                self.lift.append(dev((v * w2[:, None]).T))
        qp = _points(case, torch.float64 if case["prec"] == "fp64" else torch.float32, seed)
        nz, ny, nx = self.n[2], self.n[1], self.n[0]
        self.y = torch.empty((5, len(self.modes), nz, ny, nx), dtype=torch.float64, device="cuda")
        for i in range(5):
            for z in range(0, nz, 32):
                g = qp[i, :, :, :, z:z + 32].double().reshape(len(pts), -1)
                self.y[i, :, z:z + 32] = (self.PW @ g).reshape(len(self.modes), -1, ny, nx)
        del qp
        self.drive = _driving(seed) if case["force"] else None
        self.net = None
        if case["closure"]:
            self.net = [torch.tensor(a, device="cuda").double() for a in _closure(self.y.float(), seed)]

    def basis(self, x):
        cols, grads = [], [[], [], []]
        for m in self.modes:
            f = [_legendre(m[d], x[:, d]) for d in range(3)]
            cols.append(f[0][0] * f[1][0] * f[2][0])
            for a in range(3):
                grads[a].append(np.prod([f[d][1] if d == a else f[d][0] for d in range(3)], axis=0))
        return np.stack(cols, 1), [np.stack(g, 1) for g in grads]

    @staticmethod
    def out(y):
        """The library's order [z][y][i][l][x]."""
        return y.permute(2, 3, 0, 1, 4)

    def apply(self, table, w):
        """table[p][l] on w[5][l][...cells]."""
        return torch.matmul(table, w.reshape(5, w.shape[1], -1)).reshape(5, table.shape[0], *w.shape[2:])

    def flux(self, q, ax):
        p = (self.gamma - 1) * (q[4] - 0.5 * (q[1] ** 2 + q[2] ** 2 + q[3] ** 2) / q[0])
        u = q[1 + ax] / q[0]
        f = q * u
        f[1 + ax] += p
        f[4] += p * u
        return f, p, u

    def hllc(self, ql, qr, ax):
        fl, pl, ul = self.flux(ql, ax)
        fr, pr, ur = self.flux(qr, ax)
        cl, cr = torch.sqrt(self.gamma * pl / ql[0]), torch.sqrt(self.gamma * pr / qr[0])
        sl, sr = torch.minimum(ul - cl, ur - cr), torch.maximum(ul + cl, ur + cr)
        ml, mr = ql[0] * (sl - ul), qr[0] * (sr - ur)
        ss = (pr - pl + ml * ul - mr * ur) / (ml - mr)

        def star(q, f, p, u, s):
            r = q[0] * (s - u) / (s - ss)
            us = r * (q / q[0])
            us[1 + ax] = r * ss
            us[4] = r * (q[4] / q[0] + (ss - u) * (ss + p / (q[0] * (s - u))))
            return f + s * (us - q)

        f = torch.where(ss >= 0, star(ql, fl, pl, ul, sl), star(qr, fr, pr, ur, sr))
        return torch.where(sl >= 0, fl, torch.where(sr > 0, f, fr))

    def accel(self, z0, z1):
        """The driving acceleration [3][points][z][y][x] of the planes z0..z1-1."""
        nv, ah = self.drive
        amp = torch.tensor(ah[..., 0] + 1j * ah[..., 1], device="cuda")
        e = []
        for d, (lo, hi) in enumerate(((0, self.n[0]), (0, self.n[1]), (z0, z1))):
            x = (np.arange(lo, hi)[None] + 0.5 * (1 + self.xi[:, None])) / self.n[d]
            e.append(torch.tensor(np.exp(2j * np.pi * x[..., None] * nv[:, d]), device="cuda"))
        out = torch.empty((3, len(self.pts), z1 - z0, self.n[1], self.n[0]), dtype=torch.float64, device="cuda")
        for j, (a, b, c) in enumerate(self.pts):
            zy = (e[2][c][:, None] * e[1][b][None]).reshape(-1, len(nv))
            for i in range(3):
                w = zy * amp[:, i]
                o = w.real @ e[0][a].real.T - w.imag @ e[0][a].imag.T
                out[i, j] = o.reshape(z1 - z0, self.n[1], self.n[0])
        return out

    def rhs(self, y):
        """R(y), a few planes at a time."""
        nx, ny, nz = self.n
        r = torch.empty_like(y)
        dz = max(1, int(6e6 / (nx * ny * len(self.pts))))
        for z0 in range(0, nz, dz):
            z1 = min(nz, z0 + dz)
            idx = torch.arange(z0 - 1, z1 + 1, device="cuda") % nz
            ext = y[:, :, idx]
            w = ext[:, :, 1:-1]
            acc = r[:, :, z0:z1]
            q = self.apply(self.V, w)
            acc.zero_()
            for ax in range(3):
                acc -= 2 * self.n[ax] * self.apply(self.G[ax], self.flux(q, ax)[0])
            if self.drive is not None:
                a = self.accel(z0, z1)
                src = torch.cat([torch.zeros_like(q[:1]), q[:1] * a, (q[1:4] * a).sum(0, keepdim=True)])
                acc -= self.apply(self.PW, src)
                del a, src
            del q
            for ax, dim in ((0, 4), (1, 3), (2, 2)):
                if ax < 2:
                    lo, hi = self.apply(self.face[2 * ax + 1], w), self.apply(self.face[2 * ax], w)
                    fp = self.hllc(lo, torch.roll(hi, -1, dim), ax)
                    fm = torch.roll(fp, 1, dim)
                else:
                    lo = self.apply(self.face[5], ext[:, :, :-1])
                    f = self.hllc(lo, self.apply(self.face[4], ext[:, :, 1:]), ax)
                    fm, fp = f[:, :, :-1], f[:, :, 1:]
                acc += self.n[ax] * (self.apply(self.lift[2 * ax + 1], fp) - self.apply(self.lift[2 * ax], fm))
        if self.net is not None:
            r -= self.correction(y)
        return r

    def correction(self, y):
        p, mean, std, scale, bound = self.net
        w = y.reshape(20, *y.shape[2:])
        f = torch.cat([w] + [torch.roll(w, s, d) for d in (3, 2, 1) for s in (1, -1)]).reshape(140, -1)
        o = _network(p, (140, *HIDDEN, 20), ((f - mean[:, None]) / std[:, None]).T)[-1]
        bad = ~((o.abs() <= bound) & o.isfinite()).all(1, keepdim=True)
        c = torch.where(bad, torch.zeros_like(o), o * scale).T.reshape(y.shape)
        c[:, 0] -= c[:, 0].mean((1, 2, 3), keepdim=True)
        return c

    def dt(self):
        q = self.y[:, 0]
        _, p, _ = self.flux(q, 0)
        c = torch.sqrt(self.gamma * p / q[0])
        rate = sum((torch.abs(q[1 + a] / q[0]) + c) * self.n[a] for a in range(3)).max().item()
        f = 1.0 / (2 * self.k + 1)
        if self.case["iso"]:  # the limiter's bound: half the first Gauss-Lobatto weight
            f = min(f, 0.5 * {1: 1.0, 2: 1 / 3, 3: 1 / 3, 4: 1 / 6}[self.k])
        return CFL * f / rate

    def step(self):
        """One SSP-RK3 step.  The limiter is not evaluated: these states stay far from its bounds,
        where it changes nothing."""
        h, y0 = self.dt(), self.y
        y1 = self.rhs(y0).mul_(-h).add_(y0)
        y2 = self.rhs(y1).mul_(-h).add_(y1).mul_(0.25).add_(y0, alpha=0.75)
        del y1
        self.y = self.rhs(y2).mul_(-h).add_(y2).mul_(2.0 / 3.0).add_(y0, alpha=1.0 / 3.0)
        del y0, y2
        if self.case["iso"]:
            g = self.gamma
            q = self.apply(self.V, self.y)
            assert q[0].min() > 0.1 and self.flux(q, 0)[1].min() > 0.1
            e = 0.5 * (q[1] ** 2 + q[2] ** 2 + q[3] ** 2) / q[0] + q[0] ** g / (g - 1)
            self.y[4] = torch.matmul(self.PW, e.reshape(len(self.pts), -1)).reshape(self.y[4].shape)

    def diagnostics(self):
        s, (nx, ny, nz) = 4, self.n
        x = -1 + (2 * np.arange(s) + 1.0) / s
        pts = np.array([[x[a], x[b], x[c]] for c in range(s) for b in range(s) for a in range(s)])
        q = self.apply(torch.tensor(self.basis(pts)[0], device="cuda"), self.y)
        q = q.reshape(5, s, s, s, nz, ny, nx).permute(0, 4, 1, 5, 2, 6, 3).reshape(5, s * nz, s * ny, s * nx)
        v = q[1:4] / q[0]
        _, p, _ = self.flux(q, 0)
        mach = math.sqrt(((v ** 2).sum(0) * q[0] / (self.gamma * p)).mean().item())
        m = s * nx
        power = sum(torch.fft.fftn(c).abs() ** 2 for c in v) / float(m) ** 6
        f = torch.fft.fftfreq(m, 1.0 / m, dtype=torch.float64, device="cuda")
        shell = torch.floor(torch.sqrt(f[:, None, None] ** 2 + f[:, None] ** 2 + f ** 2) + 0.5).long()
        spec = torch.bincount(shell.reshape(-1), power.reshape(-1), minlength=m)[:m]
        vol = 1.0 / (nx * ny * nz)
        # the counts hang on single points' rounding, and are whole numbers in any case
        return {"totals": self.y[:, 0].sum((1, 2, 3)) * vol, "spectrum": spec, "pdf": None, "mach": mach}


def _network(p, shape, x):
    """Activations of the tanh network with packed parameters p on rows x."""
    acts, at = [x], 0
    for j, (i, o) in enumerate(zip(shape[:-1], shape[1:])):
        w, b = p[at:at + i * o].reshape(o, i), p[at + i * o:at + i * o + o]
        at += i * o + o
        z = acts[-1] @ w.T + b
        acts.append(torch.tanh(z) if j < 2 else z)
    return acts


def _normals(seed, n):
    """The input noise: SplitMix64 of a counter (Steele, Lea and Flood, 2014), Box-Muller."""
    s64 = lambda v: v - (1 << 64) if v >= 1 << 63 else v
    z = torch.arange(1, n + 1, device="cuda") * s64(0x9E3779B97F4A7C15) + s64(seed % (1 << 64))
    shr = lambda a, b: (a >> b) & ((1 << (64 - b)) - 1)
    z = (z ^ shr(z, 30)) * s64(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * s64(0x94D049BB133111EB)
    z = z ^ shr(z, 31)
    u1, u2 = (shr(z, 40) + 1).double() / 2 ** 24, (z & 0xffffff).double() / 2 ** 24
    return torch.sqrt(-2 * torch.log(u1)) * torch.cos(2 * math.pi * u2)


def _exact_train(case, seed):
    st, b = _train_state(case, seed), case["batch"]
    shape, it = (140, case["h1"], case["h2"], 20), TRAIN_STEP + 1
    rows = st["perm"][:b].long()
    x, t, p = st["x"][rows].double(), st["t"][rows].double(), st["params"].double().requires_grad_(True)
    x = x + NOISE * _normals(seed * 1000003 + it, 140 * b).reshape(140, b).T
    ((_network(p, shape, x)[-1] - t) ** 2).mean().backward()
    g, p = p.grad, p.detach()
    m = 0.9 * st["m"].double() + 0.1 * g
    v = 0.999 * st["v"].double() + 0.001 * g * g
    p = p - LR * (m / (1 - 0.9 ** it)) / (torch.sqrt(v / (1 - 0.999 ** it)) + 1e-8)
    return [g, p, m, v]
