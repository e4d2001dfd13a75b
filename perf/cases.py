"""Timing cases of the SPG reconstruction: what a refinement program has the library do, by call.

A refinement goes around this loop: backproject the particle images into (w, b); solve the
reweighted l1 + TV problem for each half map or class volume (set the data, a few rounds of
iterations with a reweight between them, fetch the map, check it); compare the half maps by
their Fourier shell correlation.  Tuning lambda and mu differentiates an unrolled solve.
The kinds below are those calls:

  run         set_map + run + get_map on a problem whose data and penalty weights are set
  solve       the whole step: set_data, rounds of run with reweights, get_map (, final_check)
  batch       several volumes advanced together in one graph
  diff        an unrolled solve and its gradient in (lambda, mu, b) through autograd
  backproject particle images to (w, b)
  fsc         the shell correlation of two maps

`listed` holds one case for each size that matters, `draw` draws more of the same ranges,
`prepare` / `run` / `work` / `exact` make, run, price and check a case.
"""
import math

import numpy as np
import torch

from paper_1905_13408_amd import spg
from paper_1905_13408_amd.autograd import UnrolledSPG

DEVICE = "cuda"
LAM, MU, EPS, EPS1, EPS2 = 0.01, 0.05, 1e-3, 0.01, 0.01  # the workloads' solver constants


def _solver_case(name, kind, shape, storage, iters, rounds=1, gamma=0.0, weights=False, check=False, accel=True,
                 monitor=0):
    nz, ny, nx = shape
    c = {"kind": kind, "nz": nz, "ny": ny, "nx": nx, "storage": storage, "iters": iters, "rounds": rounds,
         "gamma": gamma, "weights": weights, "check": check, "accel": accel, "monitor": monitor}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the small plain workload: 50 iterations of a 32^3 map, where launches and latency count
        _solver_case("run-32", "run", (32, 32, 32), "compensated", 50),
        # a cropped, non-cubic box with mixed-radix axes, plain fp32 iterate, explicit weights
        _solver_case("run-box", "run", (64, 192, 160), "fp32", 20, weights=True),
        # a class volume: three short reweighting rounds and the final check
        _solver_case("solve-128", "solve", (128, 128, 128), "compensated", 20, rounds=3, check=True),
        # a mixed-radix box with the implicit-descent term towards the previous map
        _solver_case("solve-160-prior", "solve", (160, 160, 160), "compensated", 20, rounds=2, gamma=0.05),
        # half-precision weight storage
        _solver_case("solve-192-bf16", "solve", (192, 192, 192), "bf16", 20, rounds=2),
        # the reweighting workload's box
        _solver_case("solve-256", "solve", (256, 256, 256), "compensated", 20, rounds=3, check=True),
        # the precision workload's box: the largest call
        _solver_case("solve-512", "solve", (512, 512, 512), "compensated", 12, rounds=2, check=True),
        # two half maps and six class volumes of uneven boxes
        {"name": "batch-8", "kind": "batch", "sizes": "128,160,192,256,256,192,160,128", "iters": 50},
        # differentiation workload: forward and reverse through 50 iterations
        {"name": "diff-128", "kind": "diff", "n": 128, "iters": 50, "every": 10},
        # a mini-batch of small images, as the tests and coarse first passes use
        {"name": "backproject-32", "kind": "backproject", "nz": 32, "ny": 32, "nx": 32, "images": 40, "m": 32,
         "ctf": True, "weighted": True},
        # particle images of the box size into their volume
        {"name": "backproject-128", "kind": "backproject", "nz": 128, "ny": 128, "nx": 128, "images": 200, "m": 128,
         "ctf": True, "weighted": True},
        # half maps against each other
        {"name": "fsc-256", "kind": "fsc", "nz": 256, "ny": 256, "nx": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng, lo, hi):
    """A box of lo..hi voxels, spread over the logarithm of its size: a cube half the time."""
    axes = [8, 16, 32, 64, 128, 160, 192, 256, 512]
    target = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.5:
        cubes = [n for n in axes if lo <= n ** 3 <= hi]
        n = min(cubes, key=lambda k: abs(math.log(k ** 3 / target)))
        return (n, n, n)
    while True:
        s = tuple(rng.choice(axes) for _ in range(3))
        if lo <= s[0] * s[1] * s[2] <= hi and abs(math.log(s[0] * s[1] * s[2] / target)) < 0.6:
            return s


def draw(rng):
    kind = rng.choices(["run", "solve", "batch", "diff", "backproject", "fsc"], [30, 30, 8, 8, 16, 8])[0]
    if kind in ("run", "solve"):
        shape = _draw_shape(rng, 1 << 13, 1 << 25)
        storage = rng.choices(["compensated", "fp32", "bf16"], [6, 2, 2])[0]
        gamma = rng.choice([0.0, 0.0, 0.0, round(rng.uniform(0.01, 0.3), 3)])
        accel = rng.random() < 0.85
        if kind == "run":
            return _solver_case("", kind, shape, storage, _log_int(rng, 5, 40), 1, gamma, rng.random() < 0.6,
                                False, accel)
        return _solver_case("", kind, shape, storage, _log_int(rng, 5, 20), rng.randint(1, 3), gamma, False,
                            storage == "compensated" and rng.random() < 0.5, accel,
                            rng.choice([0, 0, 5]) if storage == "compensated" else 0)
    if kind == "batch":
        sizes = sorted(rng.choice([32, 64, 128, 160, 192]) for _ in range(rng.randint(2, 6)))
        return {"kind": kind, "sizes": ",".join(map(str, sizes)), "iters": _log_int(rng, 10, 60)}
    if kind == "diff":
        iters = _log_int(rng, 8, 50)
        return {"kind": kind, "n": rng.choice([32, 64, 128]), "iters": iters, "every": rng.randint(3, min(12, iters))}
    if kind == "backproject":
        n = rng.choice([32, 64, 128, 160, 192])
        m = max(8, n - rng.choice([0, 0, 1, 7, n // 4]))
        most = max(2, min(400, int(4e6 / (m * m))))
        return {"kind": kind, "nz": n, "ny": n, "nx": n, "images": _log_int(rng, 1, most), "m": m,
                "ctf": rng.random() < 0.8, "weighted": rng.random() < 0.7}
    nz, ny, nx = _draw_shape(rng, 1 << 15, 1 << 24)
    return {"kind": kind, "nz": nz, "ny": ny, "nx": nx}


# ------------------------------------------------------------------ inputs

def _generator(seed, *salt):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(np.random.SeedSequence([int(seed) & 0x7FFFFFFF, *salt]).generate_state(1)[0]))
    return g


def _freq(n):
    return torch.fft.fftfreq(n, device=DEVICE, dtype=torch.float64) * n


def _blobs(shape, seed):
    """A density: Gaussian blobs (width 1.2 voxels) on random-walk chains of step 1.5 in a ball."""
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 17, *shape])
    n = int(np.clip(0.0003 * np.prod(shape), 8, 30000))
    chains = max(1, n // 250)
    radius = 0.39 * np.array(shape)
    start = rng.uniform(-0.5, 0.5, (chains, 1, 3)) * radius
    step = rng.standard_normal((chains, -(-n // chains), 3))
    step *= 1.5 / np.linalg.norm(step, axis=2, keepdims=True)
    p = (start + np.cumsum(step, axis=1)).reshape(-1, 3)
    p *= np.minimum(1.0, 1.0 / np.maximum(1e-9, np.linalg.norm(p / radius, axis=1, keepdims=True)))
    at = np.mod(np.rint(p + np.array(shape) / 2).astype(np.int64), np.array(shape))
    idx, inv = np.unique((at[:, 0] * shape[1] + at[:, 1]) * shape[2] + at[:, 2], return_inverse=True)
    amp = np.bincount(inv.reshape(-1), weights=rng.uniform(0.5, 1.0, len(at)))
    x = torch.zeros(int(np.prod(shape)), device=DEVICE)
    x[torch.from_numpy(idx).to(DEVICE)] = torch.from_numpy(amp.astype(np.float32)).to(DEVICE)
    F = torch.fft.rfftn(x.reshape(shape))
    for a, m in enumerate(shape):
        k = _freq(m)[: m // 2 + 1] if a == 2 else _freq(m)
        k = k.abs() / m
        F *= torch.exp(-0.5 * (2 * math.pi * 1.2 * k) ** 2).float().reshape([-1 if i == a else 1 for i in range(3)])
    return torch.fft.irfftn(F, s=shape) * (1.2 * math.sqrt(2 * math.pi)) ** 3


def _weights(shape, g):
    """Fourier weights in the role of N(n): a Gaussian falloff with a floor, uneven coverage."""
    w = torch.ones((1, 1, 1), device=DEVICE, dtype=torch.float64)
    for a, n in enumerate(shape):
        w = w * torch.exp(-_freq(n) ** 2 / (2 * (0.25 * n) ** 2)).reshape([-1 if i == a else 1 for i in range(3)])
    return (w.float() + 1e-3) * (0.9 + 0.2 * torch.rand(shape, device=DEVICE, generator=g))


def _volume(shape, seed, snr=0.5):
    """(x_true, w, b): b = A x_true plus circular complex noise at the given SNR."""
    g = _generator(seed, 3, *shape)
    x = _blobs(shape, seed)
    w = _weights(shape, g)
    sigma = float(torch.sqrt(torch.sum(x.double() ** 2) / (x.numel() * snr)))
    noise = torch.randn((*shape, 2), device=DEVICE, generator=g)
    b = torch.fft.fftn(x, norm="ortho") + torch.view_as_complex(noise) * (sigma / math.sqrt(2))
    return x, w.contiguous(), b.contiguous()


def _solver_inputs(case, seed):
    shape = (case["nz"], case["ny"], case["nx"])
    x, w, b = _volume(shape, seed)
    g = _generator(seed, 5, *shape)
    d = {"shape": shape, "w": w, "b": b}
    if case["gamma"]:
        d["prior"] = x + 0.1 * x.abs().max() * torch.randn(shape, device=DEVICE, generator=g)
    if case["weights"]:  # weights of a former round: small on the density, large off it
        d["u"] = 1.0 / (x.abs() + 0.5 + 0.5 * torch.rand(shape, device=DEVICE, generator=g))
        d["v"] = 1.0 / (x.abs() + 0.5 + 0.5 * torch.rand(shape, device=DEVICE, generator=g))
    return d


def _images(case, seed):
    """Particle images in Fourier space with their CTFs, posterior weights and rotations."""
    n, m = case["images"], case["m"]
    g = _generator(seed, 7, n, m)
    k2 = (_freq(m)[:, None] ** 2 + _freq(m)[None, :] ** 2) / (m * m / 4)
    fall = torch.exp(-2.0 * k2).float()
    im = torch.randn((n, m, m, 2), device=DEVICE, generator=g) * fall[None, :, :, None]
    d = {"images": torch.view_as_complex(im), "ctf": None, "weights": None}
    if case["ctf"]:  # oscillation by each image's defocus under an envelope, its zeros masked by a floor
        defocus = 8.0 + 8.0 * torch.rand((n, 1, 1), device=DEVICE, generator=g)
        c = -torch.sin(defocus * k2.float()[None] * math.pi + 0.1) * torch.exp(-0.5 * k2.float())[None]
        d["ctf"] = torch.where(c < 0, -1.0, 1.0) * torch.clamp(c.abs(), min=0.05)
    if case["weighted"]:
        d["weights"] = 0.2 + 0.8 * torch.rand(n, device=DEVICE, generator=g)
    q = np.random.default_rng([int(seed) & 0x7FFFFFFF, 19, n, m]).standard_normal((n, 4))
    a, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    rot = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * a), 2 * (x * z + y * a),
                    2 * (x * y + z * a), 1 - 2 * (x * x + z * z), 2 * (y * z - x * a),
                    2 * (x * z - y * a), 2 * (y * z + x * a), 1 - 2 * (x * x + y * y)], 1).reshape(n, 3, 3)
    d["rots"] = torch.from_numpy(rot).to(DEVICE)
    return d


def _sizes(case):
    return [int(n) for n in case["sizes"].split(",")]


def _diff_inputs(case, seed):
    shape = (case["n"],) * 3
    x, w, b = _volume(shape, seed)
    return {"shape": shape, "x_true": x, "w": w, "b": b.requires_grad_(True),
            "lam": torch.tensor(LAM, requires_grad=True), "mu": torch.tensor(MU, requires_grad=True)}


def _half_maps(case, seed):
    shape = (case["nz"], case["ny"], case["nx"])
    x = _blobs(shape, seed)
    g = _generator(seed, 11, *shape)
    noise = float(x.std()) * 1.5
    return {"a": x + noise * torch.randn(shape, device=DEVICE, generator=g),
            "b": x + noise * torch.randn(shape, device=DEVICE, generator=g)}


def _batch_inputs(case, seed):
    """Per member: (shape, lambda, mu, w, b)."""
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 23])
    out = []
    for i, n in enumerate(_sizes(case)):
        lam, mu = LAM * rng.uniform(0.5, 2.0), MU * rng.uniform(0.5, 2.0)
        _, w, b = _volume((n, n, n), seed + 1000 * (i + 1), rng.uniform(0.3, 1.0))
        out.append(((n, n, n), lam, mu, w, b))
    return out


# ------------------------------------------------------------------ the cases

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("run", "solve"):
        st = _solver_inputs(case, seed)
        s = spg.SPGSolver(st["shape"], LAM, MU, EPS, accel=case["accel"], storage=case["storage"],
                          monitor_every=case["monitor"])
        if kind == "run":
            s.set_data(st["w"], st["b"])
            if case["weights"]:
                s.set_penalty_weights(st["u"], st["v"])
            if case["gamma"]:
                s.set_prior(case["gamma"], st["prior"])
        st["solver"] = s
    elif kind == "batch":
        st = {"solvers": []}
        for shape, lam, mu, w, b in _batch_inputs(case, seed):
            s = spg.SPGSolver(shape, lam, mu, EPS)
            s.set_data(w, b)
            st["solvers"].append(s)
        st["batch"] = spg.SPGBatch(st["solvers"])
    elif kind == "diff":
        st = _diff_inputs(case, seed)
        st["solver"] = spg.SPGSolver(st["shape"], LAM, MU, EPS)
    elif kind == "backproject":
        st = _images(case, seed)
    else:
        st = _half_maps(case, seed)
    st["case"] = case
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "run":
        s = st["solver"]
        s.set_map(None)
        s.run(case["iters"])
        return {"map": s.get_map()}
    if kind == "solve":
        s = st["solver"]
        s.set_data(st["w"], st["b"])
        s.set_penalty_weights(None, None)
        if case["gamma"]:
            s.set_prior(case["gamma"], st["prior"])
        s.set_map(None)
        out = {}
        for r in range(case["rounds"]):
            if r > 0:
                s.reweight(EPS1, EPS2)
            stats = s.run(case["iters"])
            if case["monitor"] and case["iters"] >= case["monitor"]:
                out["objective_%d" % r] = stats.obj_smoothed
        out["map"] = s.get_map()
        if case["check"]:
            out["F_eps"], out["F_0"], out["kkt"] = s.final_check()
        return out
    if kind == "batch":
        for s in st["solvers"]:
            s.set_map(None)
        st["batch"].run(case["iters"])
        return [s.get_map() for s in st["solvers"]]
    if kind == "diff":
        x = UnrolledSPG.apply(st["lam"], st["mu"], st["b"], st["solver"], st["w"], case["iters"], case["every"])
        loss = ((x - st["x_true"]) ** 2).sum()
        lam, mu, b = torch.autograd.grad(loss, (st["lam"], st["mu"], st["b"]))
        return {"map": x.detach(), "lam": lam, "mu": mu, "b": b}
    if kind == "backproject":
        w, b = spg.backproject((case["nz"], case["ny"], case["nx"]), st["images"], st["rots"], st["ctf"],
                               st["weights"])
        return {"w": w, "b": b}
    return {"fsc": spg.fsc(st["a"], st["b"])}


def _iteration_work(n, weight_bytes, explicit, momentum):
    """(bytes, flops) of one iteration of n voxels: x_k, x_{k-1} and the folded data in, x_{k+1}
    out (fp32), u and v where given; two real 3D transforms and the stencil with its prox."""
    b = 4 * n * (2 + (1 if momentum else 0)) + 2 * n + 4 * n + (2 * weight_bytes * n if explicit else 0)
    return b, 2 * 2.5 * n * math.log2(n) + 45.0 * n


def work(case):
    kind = case["kind"]
    if kind in ("run", "solve"):
        n = case["nz"] * case["ny"] * case["nx"]
        wb = 2 if case["storage"] == "bf16" else 4
        total = [4.0 * n, 0.0]  # the map that is fetched
        for r in range(case["rounds"]):
            b, f = _iteration_work(n, wb, case["weights"] or r > 0, case["accel"])
            total[0] += case["iters"] * (b + (4 * n if case["gamma"] else 0))
            total[1] += case["iters"] * f
            if r > 0:  # reweight: the map in, u and v out
                total[0] += 4 * n + 2 * wb * n
                total[1] += 20.0 * n
        if kind == "solve":  # w and b in, folded weights and data out
            total[0] += 12 * n + 6 * n + (8 * n if case["gamma"] else 0)
            total[1] += 20.0 * n
        if case["check"]:
            b, f = _iteration_work(n, wb, case["rounds"] > 1, False)
            total[0] += b
            total[1] += f
        return {"bytes": total[0], "flops": total[1]}
    if kind == "batch":
        per = [_iteration_work(n ** 3, 4, False, True) for n in _sizes(case)]
        return {"bytes": case["iters"] * sum(p[0] for p in per) + sum(4.0 * n ** 3 for n in _sizes(case)),
                "flops": case["iters"] * sum(p[1] for p in per)}
    if kind == "diff":
        # forward; then per step back: the iterates, the adjoints (two in, two out), the folded
        # weights; two more real transforms and the second derivative of the stencil
        n = case["n"] ** 3
        b, f = _iteration_work(n, 4, False, True)
        return {"bytes": case["iters"] * (b + 4 * n * 6 + 2 * n) + 12 * n + 6 * n + 20 * n,
                "flops": case["iters"] * (f + 2 * 2.5 * n * math.log2(n) + 120.0 * n)}
    n = case["nz"] * case["ny"] * case["nx"]
    if kind == "backproject":
        pix = case["images"] * case["m"] ** 2
        return {"bytes": pix * (8 + (4 if case["ctf"] else 0)) + 12.0 * n, "flops": pix * 27 * 16.0 + 4.0 * n}
    return {"bytes": 8.0 * n, "flops": 2 * 2.5 * n * math.log2(n) + 12.0 * n}


# ------------------------------------------------------------------ the same in 64 bits

def _d(x):
    return [x - torch.roll(x, 1, a) for a in range(3)]


def _dt(p):
    return sum(p[a] - torch.roll(p[a], -1, a) for a in range(3))


def _neg(a):
    return torch.roll(torch.flip(a, (0, 1, 2)), (1, 1, 1), (0, 1, 2))


def _dnorm2(shape):
    return sum(max(4 * math.sin(math.pi * k / n) ** 2 for k in range(n)) for n in shape)


class _Problem:
    """One problem of eq 31 with plain torch in float64 (complex128)."""

    def __init__(self, shape, w, b, lam, mu, u=None, v=None, gamma=0.0, prior=None, accel=True):
        self.shape, self.lam, self.mu, self.gamma, self.accel = shape, lam, mu, gamma, accel
        self.w, self.b = w.double(), b.to(torch.complex128)
        self.u = 1.0 if u is None else u.double()
        self.v = 1.0 if v is None else v.double()
        self.prior = 0.0 if prior is None else prior.double()
        self.wmax = float((0.5 * (self.w + _neg(self.w))).max())

    def vmax(self):
        return float(self.v.max()) if torch.is_tensor(self.v) else self.v

    def lr(self):
        return 1.0 / (self.wmax + self.mu * self.vmax() * _dnorm2(self.shape) / EPS + 2 * self.gamma)

    def grad_data(self, y):
        return torch.fft.ifftn(self.w * (torch.fft.fftn(y, norm="ortho") - self.b), norm="ortho").real

    def grad_tv(self, y):
        d = _d(y)
        n2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
        low = n2 < EPS * EPS
        s = self.v * torch.where(low, torch.full_like(n2, 1.0 / EPS), torch.rsqrt(torch.where(low, torch.ones_like(n2), n2)))
        return _dt([s * q for q in d])

    def step(self, y, lr):
        g = self.grad_data(y) + self.mu * self.grad_tv(y)
        if self.gamma:
            g = g + 2 * self.gamma * (y - self.prior)
        z = y - lr * g
        return torch.sign(z) * torch.relu(z.abs() - lr * self.lam * self.u)

    def objective(self, x, smooth):
        r = torch.fft.fftn(x, norm="ortho") - self.b
        f = 0.5 * (self.w * (r.real ** 2 + r.imag ** 2)).sum() + self.lam * (self.u * x.abs()).sum()
        n = torch.sqrt(sum(q * q for q in _d(x)))
        phi = torch.where(n < EPS, n * n / (2 * EPS), n - 0.5 * EPS) if smooth else n
        f = f + self.mu * (self.v * phi).sum()
        if self.gamma:
            f = f + self.gamma * ((x - self.prior) ** 2).sum()
        return float(f)

    def kkt(self, x):
        q, n = x - self.step(x, self.lr()), float(torch.linalg.vector_norm(x))
        return float(torch.linalg.vector_norm(q)) / (n if n > 0 else 1.0)

    def iterate(self, x, iters, lr=None, watch=0):
        """x after `iters` iterations with the momentum restarted (, F_eps at the last watched y)."""
        lr = self.lr() if lr is None else lr
        old, t, m, seen = x, 1.0, 0.0, None
        for j in range(1, iters + 1):
            y = x + m * (x - old) if m else x
            if watch and j % watch == 0:
                seen = self.objective(y, True)
            x, old = self.step(y, lr), x
            if self.accel:
                tn = 0.5 * (1.0 + math.sqrt(1.0 + 4.0 * t * t))
                m, t = (t - 1.0) / tn, tn
        return x, seen


def _exact_solve(case, seed):
    d = _solver_inputs(case, seed)
    p = _Problem(d["shape"], d["w"], d["b"], LAM, MU, d.get("u"), d.get("v"), case["gamma"], d.get("prior"),
                 case["accel"])
    x = torch.zeros(d["shape"], device=DEVICE, dtype=torch.float64)
    out = {}
    for r in range(case["rounds"]):
        if r > 0:
            n = torch.sqrt(sum(q * q for q in _d(x)))
            p.u, p.v = 1.0 / (x.abs() + EPS1), 1.0 / (n + EPS2)
        x, seen = p.iterate(x, case["iters"], watch=case["monitor"])
        if seen is not None:
            out["objective_%d" % r] = seen
    out["map"] = x
    if case["check"]:
        out["F_eps"], out["F_0"], out["kkt"] = p.objective(x, True), p.objective(x, False), p.kkt(x)
    return out


def _exact_batch(case, seed):
    out = []
    for shape, lam, mu, w, b in _batch_inputs(case, seed):
        p = _Problem(shape, w, b, lam, mu)
        out.append(p.iterate(torch.zeros(shape, device=DEVICE, dtype=torch.float64), case["iters"])[0])
    return out


def _exact_diff(case, seed):
    d = _diff_inputs(case, seed)
    shape = d["shape"]
    lam = torch.tensor(float(d["lam"].detach()), dtype=torch.float64, device=DEVICE, requires_grad=True)
    mu = torch.tensor(float(d["mu"].detach()), dtype=torch.float64, device=DEVICE, requires_grad=True)
    p = _Problem(shape, d["w"], d["b"].detach(), lam, mu)
    p.b = p.b.requires_grad_(True)
    x, _ = p.iterate(torch.zeros(shape, device=DEVICE, dtype=torch.float64), case["iters"],
                     lr=1.0 / (p.wmax + mu * _dnorm2(shape) / EPS))
    loss = ((x - d["x_true"].double()) ** 2).sum()
    gl, gm, gb = torch.autograd.grad(loss, (lam, mu, p.b))
    return {"map": x.detach(), "lam": gl, "mu": gm, "b": gb}


def _exact_backproject(case, seed):
    d = _images(case, seed)
    shape, m = (case["nz"], case["ny"], case["nx"]), case["m"]
    n = shape[0] * shape[1] * shape[2]
    num = torch.zeros((n, 2), device=DEVICE, dtype=torch.float64)
    den = torch.zeros(n, device=DEVICE, dtype=torch.float64)
    v, u = torch.meshgrid(_freq(m), _freq(m), indexing="ij")
    for i0 in range(0, case["images"], 16):
        R = d["rots"][i0:i0 + 16].double()
        c = [R[:, a, 0, None, None] * u + R[:, a, 1, None, None] * v for a in range(3)]
        base = [torch.floor(q + 0.5) for q in c]
        X = torch.view_as_real(d["images"][i0:i0 + 16].to(torch.complex128))
        ctf = torch.ones_like(c[0]) if d["ctf"] is None else d["ctf"][i0:i0 + 16].double()
        pw = torch.ones_like(ctf) if d["weights"] is None else d["weights"][i0:i0 + 16].double()[:, None, None]
        for k in range(27):
            g = [base[a] + ((k // 3 ** a) % 3 - 1) for a in range(3)]
            K = pw * torch.exp(-((c[0] - g[0]) ** 2 + (c[1] - g[1]) ** 2 + (c[2] - g[2]) ** 2) / 2.0) * ctf
            ix, iy, iz = (torch.remainder(g[a], shape[2 - a]).long() for a in range(3))
            at = ((iz * shape[1] + iy) * shape[2] + ix).reshape(-1)
            num.index_add_(0, at, (K[..., None] * X).reshape(-1, 2))
            den.index_add_(0, at, (K * ctf).reshape(-1))
    b = torch.where(den[:, None] > 0, num / torch.where(den > 0, den, torch.ones_like(den))[:, None], torch.zeros_like(num))
    return {"w": den.reshape(shape), "b": torch.view_as_complex(b).reshape(shape)}


def _exact_fsc(case, seed):
    d = _half_maps(case, seed)
    shape = (case["nz"], case["ny"], case["nx"])
    n = min(shape) // 2 + 1
    F, G = torch.fft.fftn(d["a"].double()), torch.fft.fftn(d["b"].double())
    r2 = sum(((_freq(m) * min(shape) / m) ** 2).reshape([-1 if i == a else 1 for i in range(3)])
             for a, m in enumerate(shape))
    s = torch.floor(torch.sqrt(r2) + 0.5).long().reshape(-1).cpu()
    sums = [torch.bincount(s, weights=q.reshape(-1).cpu(), minlength=n)[:n]
            for q in ((F * G.conj()).real, F.abs() ** 2, G.abs() ** 2)]
    den = torch.sqrt(sums[1] * sums[2])
    return {"fsc": torch.where(den > 0, sums[0] / torch.where(den > 0, den, torch.ones_like(den)), torch.zeros_like(den)).numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("run", "solve"):
        return _exact_solve(case, seed)
    return {"batch": _exact_batch, "diff": _exact_diff, "backproject": _exact_backproject,
            "fsc": _exact_fsc}[kind](case, seed)
