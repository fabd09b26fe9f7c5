"""The work that users of this framework have it do, as measurable cases.

A case is one call sequence of a user's program on the public entry points
(``Simulation``, ``Batch``, ``ModEq``, ``final_density``), at the sizes of the
framework's own workloads or at odd and ragged sizes of the same kind.
``listed`` names the cases, ``draw`` makes more of the same ranges,
``prepare`` makes what the program has in hand before the call (handles,
buffers, captured graphs, initial fields), ``run`` is one pass, ``work`` what
the pass cannot do without, and ``exact`` the same outputs in 64 bits from
plain torch, written from the method's definitions.

Statistics, spectra and heights of FP32 runs are returned in single
precision: their last FP64 bits carry only the rounding of the FP32 state.
"""

import math

import numpy as np
import torch

from paper_1012_3632_amd import Batch, Params, Simulation, field_spectrum
from paper_1012_3632_amd.autograd import final_density
from paper_1012_3632_amd.modeq import ModEq, ModEqParams

CS2 = 1.0 / 3.0
IDEAL = dict(rho0=1.0, kT=1e-5, rate_bulk=1.2, rate_shear=1.6, rate_ghost=1.0)
LANDAU = dict(rho0=1.0, kT=1e-6, rate_bulk=1.0, rate_shear=1.0, rate_ghost=1.0, force_model=1,
              a=-0.01, b=0.1, rho_c=1.0, kappa=0.05)
EQUILIBRATION = dict(rho0=1.0, kT=1e-7, rate_bulk=1.0, rate_shear=1.0, rate_ghost=1.0,
                     force_model=1, a=-0.01755625, b=0.14045, rho_c=0.75, kappa=0.08, eta=1)
CAPILLARY = dict(rho0=0.75, kT=1e-7, rate_bulk=1.0, rate_shear=1.0, rate_ghost=1.0,
                 force_model=1, a=-0.0125, b=0.1, rho_c=0.75, kappa=0.08, eta=1)
RHO_L, RHO_V, WIDTH = 1.0, 0.5, math.sqrt(8.0 * 0.08 / 0.1) / 0.5
MODEQ = dict(rho0=1.0, kT=1e-7, cs2_0=0.265 ** 2, kappa=0.08, rate_bulk=1.0, rate_shear=1.0,
             rate_ghost=1.0)
HALF_WINDOW = 25


# ------------------------------------------------------------------ the cases

def _step(lattice, precision, nx, ny, nz, fluid, steps, stats, **kw):
    return dict(kind="step", lattice=lattice, precision=precision, nx=nx, ny=ny, nz=nz,
                fluid=fluid, steps=steps, stats=stats, **kw)


def listed():
    return [
        # the smallest: the FDT and conservation run on 32^2, FP64, every step
        # sampled, its mode variances read at the end
        dict(_step("D2Q9", "fp64", 32, 32, 1, "ideal", 100, 1, moments=True, kT=1e-4),
             name="ideal2d_32_fp64"),
        # one snapshot of the equilibration test: 250 captured steps and the
        # mode spectra of the state
        dict(kind="equilibration", precision="fp32", nx=128, ny=128, steps=250,
             name="equilibration_128"),
        # one snapshot of the capillary test: 474 captured steps, the heights
        # of both interfaces and their spectrum
        dict(kind="capillary", precision="fp32", nx=1024, ny=400, steps=474,
             name="capillary_1024x400"),
        # one gradient of the 400-step differentiable run (forward, backward)
        dict(kind="adjoint", lattice="D2Q9", precision="fp32", nx=256, ny=256, nz=1,
             fluid="landau", steps=400, every=20, name="adjoint2d_256"),
        # the modified-equilibrium model at a large lattice, steps alone
        dict(kind="modeq", precision="fp32", nx=1024, ny=1024, steps=32, snapshot=False,
             name="modeq_1024"),
        # and one of its snapshots on an odd box in FP64: steps, moment
        # fields, their spectra
        dict(kind="modeq", precision="fp64", nx=200, ny=150, steps=50, snapshot=True,
             name="modeq_200x150_fp64"),
        # the main path: the 128^3 ideal gas, FP32, statistics every step
        dict(_step("D3Q19", "fp32", 128, 128, 128, "ideal", 20, 1, moments=True),
             name="ideal3d_128_fp32"),
        # the same in FP64 on a ragged box, statistics every tenth step
        dict(_step("D3Q19", "fp64", 120, 100, 90, "ideal", 20, 10), name="ideal3d_120x100x90_fp64"),
        # an odd box in FP32 without statistics, on the default launch shape
        dict(_step("D3Q19", "fp32", 101, 77, 53, "ideal", 20, 0, tune=False),
             name="ideal3d_101x77x53"),
        # the largest: the 256^3 Landau fluid, statistics every step
        dict(_step("D3Q19", "fp32", 256, 256, 256, "landau", 20, 1), name="landau3d_256_fp32"),
        # a batch of cubic replicas of uneven size, one captured graph
        dict(kind="batch", precision="fp32", replicas=24, smallest=32, largest=96,
             size_seed=2024, steps=20, name="batch_24"),
        # a snapshot analysis in 3-D: all mode spectra of one state
        dict(kind="spectrum", precision="fp32", nx=128, ny=96, nz=80, name="spectrum3d_128x96x80"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step2d", "step3d", "step3d", "step3d", "equilibration", "capillary",
                       "adjoint", "modeq", "modeq", "batch", "spectrum"])
    precision = rng.choice(["fp32", "fp32", "fp64"])
    fluid = rng.choice(["ideal", "landau", "equilibration"])
    if kind == "step2d":
        nx, ny = _log_int(rng, 16, 1024), _log_int(rng, 16, 512)
        return _step("D2Q9", precision, nx, ny, 1, fluid, rng.randint(20, 200),
                     rng.choice([0, 1, 10]), tune=rng.random() < 0.5)
    if kind == "step3d":
        n = [_log_int(rng, 16, 176) for _ in range(3)]
        return _step("D3Q19", precision, *n, fluid, rng.randint(4, 24), rng.choice([0, 1, 1, 10]),
                     tune=rng.random() < 0.7)
    if kind == "equilibration":
        return dict(kind=kind, precision=precision, nx=_log_int(rng, 32, 400),
                    ny=_log_int(rng, 32, 400), steps=2 * rng.randint(25, 125))
    if kind == "capillary":
        return dict(kind=kind, precision=precision, nx=_log_int(rng, 64, 1024),
                    ny=rng.randint(160, 400), steps=2 * rng.randint(25, 120))
    if kind == "adjoint":
        if rng.random() < 0.6:
            lat, n = "D2Q9", [_log_int(rng, 32, 300), _log_int(rng, 32, 300), 1]
        else:
            lat, n = "D3Q19", [_log_int(rng, 12, 48) for _ in range(3)]
        return dict(kind=kind, lattice=lat, precision=precision, nx=n[0], ny=n[1], nz=n[2],
                    fluid=fluid, steps=rng.randint(20, 100), every=rng.choice([5, 10, 20]))
    if kind == "modeq":
        n = [2 ** rng.randint(5, 10) if rng.random() < 0.6 else _log_int(rng, 32, 400)
             for _ in range(2)]
        return dict(kind=kind, precision=precision, nx=n[0], ny=n[1], steps=rng.randint(8, 64),
                    snapshot=rng.random() < 0.4)
    if kind == "batch":
        return dict(kind=kind, precision=precision, replicas=rng.randint(4, 32),
                    smallest=_log_int(rng, 16, 32), largest=_log_int(rng, 40, 80),
                    size_seed=rng.randint(0, 1 << 30), steps=2 * rng.randint(2, 10))
    return dict(kind="spectrum", precision=precision,
                **{k: _log_int(rng, 16, 160) for k in ("nx", "ny", "nz")})


# ------------------------------------------------------------------ inputs

def _fluid(case):
    return dict({"ideal": IDEAL, "landau": LANDAU, "equilibration": EQUILIBRATION}[case["fluid"]],
                **({"kT": case["kT"]} if "kT" in case else {}))


def _params(case, seed, fluid, lattice="D2Q9"):
    return dict(fluid, lattice=case.get("lattice", lattice), precision=case["precision"],
                nx=case["nx"], ny=case["ny"], nz=case.get("nz", 1), seed=seed)


def _drho(case, seed):
    """The initial density of a Landau fluid, 1 % noise (float64, nz, ny, nx);
    an ideal gas starts uniform."""
    if case["fluid"] == "ideal":
        return None
    rng = np.random.default_rng(seed)
    return 0.01 * rng.standard_normal((case.get("nz", 1), case["ny"], case["nx"]))


def _stripe_at(case):
    return 0.25 * case["ny"], 0.75 * case["ny"]


def _stripe(case, seed):
    """A liquid stripe across the middle half, each column's edges moved by a
    seeded smooth height of a fraction of a site."""
    y1, y2 = _stripe_at(case)
    rng = np.random.default_rng(seed)
    x = 2.0 * np.pi * np.arange(case["nx"]) / case["nx"]
    h = [sum(0.2 * rng.standard_normal() * np.sin(k * x + rng.uniform(0, 2 * np.pi))
             for k in range(1, 4)) for _ in range(2)]
    y = np.arange(case["ny"], dtype=np.float64)[:, None]
    prof = RHO_V + 0.5 * (RHO_L - RHO_V) * (np.tanh(2 * (y - y1 - h[0]) / WIDTH)
                                            - np.tanh(2 * (y - y2 - h[1]) / WIDTH))
    return (prof - CAPILLARY["rho0"])[None]


def _edges(case):
    rng = np.random.default_rng(case["size_seed"])
    return [int(e) for e in rng.integers(case["smallest"], case["largest"] + 1, case["replicas"])]


def _populations(case, seed, q):
    """A thermal-like state: independent populations of the fluid's size."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.tensor(_lattice(q)[1], device="cuda", dtype=torch.float64).sqrt().view(-1, 1, 1, 1)
    z = torch.randn((q, case["nz"], case["ny"], case["nx"]), generator=g, device="cuda",
                    dtype=torch.float64)
    return (math.sqrt(IDEAL["kT"] / CS2) * w * z).to(_dtype(case))


def _dtype(case):
    return torch.float32 if case["precision"] == "fp32" else torch.float64


def _adjoint_inputs(case, seed):
    """Initial populations, and the target, noisy data of another fluid: the
    density that a run from them at shear rate 1.5 and twice the temperature
    ends in, with 1 % noise."""
    q, shape = (9 if case["lattice"] == "D2Q9" else 19), (case["nz"], case["ny"], case["nx"])
    rng = np.random.default_rng(seed)
    w = torch.tensor(_lattice(q)[1], dtype=torch.float64).view(-1, 1, 1, 1)
    f0 = (w * torch.as_tensor(0.01 * rng.standard_normal(shape))).to("cuda", _dtype(case))
    p = _params(case, seed, _fluid(case))
    F = _Fluid(dict(p, rate_shear=1.5, kT=2.0 * p["kT"]))
    with torch.no_grad():
        f = f0.double()
        for n in range(case["steps"]):
            f = F.step(f, n)
        target = F.p["rho0"] + F.pulled(f)[0]
    target += torch.as_tensor(0.01 * rng.standard_normal(shape), device="cuda")
    return f0, target.to(_dtype(case))


_streams = []


def _stream():
    """The one stream on which a program replays its captured graphs."""
    if not _streams:
        _streams.append(torch.cuda.Stream())
    return _streams[0]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        sim = Simulation(Params(**_params(case, seed, _fluid(case))), drho_init=_drho(case, seed))
        # a long run tunes its handle once
        if case.get("tune", True):
            sim.autotune()
        return dict(case=case, sim=sim)
    if kind in ("equilibration", "capillary"):
        equil = kind == "equilibration"
        sim = Simulation(Params(**_params(case, seed, EQUILIBRATION if equil else CAPILLARY)),
                         drho_init=None if equil else _stripe(case, seed))
        if not equil:
            sim.autotune()
        stream = _stream()
        with torch.cuda.stream(stream):
            sim.graph_capture(case["steps"], stats_stride=0, stream=stream)
            s = dict(case=case, sim=sim, stream=stream, dtype=_dtype(case))
            if equil:
                s["spec"] = sim.spectrum_buffer()
            else:
                y1, y2 = _stripe_at(case)
                s["ifs"] = [(y1, 1, HALF_WINDOW), (y2, -1, HALF_WINDOW)]
                s["spec"] = torch.zeros((2, case["nx"]), dtype=torch.float64, device="cuda")
                s["work"] = torch.empty(16 * 2 * case["nx"], dtype=torch.uint8, device="cuda")
        stream.synchronize()
        return s
    if kind == "adjoint":
        f0, target = _adjoint_inputs(case, seed)
        fluid = _fluid(case)
        params = Params(**_params(case, seed, fluid))
        theta = [torch.tensor(fluid[k], dtype=_dtype(case), requires_grad=True)
                 for k in ("rate_shear", "kT")]
        return dict(case=case, f0=f0.requires_grad_(True), target=target, params=params,
                    theta=theta)
    if kind == "modeq":
        sim = ModEq(ModEqParams(nx=case["nx"], ny=case["ny"], precision=case["precision"],
                                seed=seed, **MODEQ))
        s = dict(case=case, sim=sim, dtype=_dtype(case))
        if case["snapshot"]:
            s["spec"] = torch.zeros((9, 1, case["ny"], case["nx"]), dtype=torch.float64,
                                    device="cuda")
            s["m"] = torch.empty_like(s["spec"])
            s["work"] = torch.empty(16 * s["spec"].numel(), dtype=torch.uint8, device="cuda")
        return s
    if kind == "batch":
        e = _edges(case)
        b = Batch(Params(lattice="D3Q19", precision=case["precision"], **IDEAL),
                  [(n, n, n) for n in e], seeds=[seed + r for r in range(len(e))])
        b.autotune()
        stream = _stream()
        b.graph_capture(case["steps"], stats_stride=1, stream=stream)
        return dict(case=case, batch=b, stream=stream)
    sim = Simulation(Params(**_params(case, seed, IDEAL, lattice="D3Q19")))
    sim.load_state(_populations(case, seed, 19))
    return dict(case=case, sim=sim, spec=sim.spectrum_buffer())


# ------------------------------------------------------------------ one pass

def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "step":
        sim = state["sim"]
        sim.step(case["steps"], stats_stride=case["stats"])
        out = dict(f=sim.state())
        if case.get("moments"):
            s, s2, n = sim.moments()
            out["sum"], out["sumsq"] = (v.astype(np.float32) for v in (s, s2))
        return out
    if kind == "equilibration":
        sim, stream = state["sim"], state["stream"]
        with torch.cuda.stream(stream):
            sim.graph_launch(stream)
            sim.accumulate_spectrum(state["spec"], stream=stream)
            return dict(f=sim.state(), spec=state["spec"].to(state["dtype"]))
    if kind == "capillary":
        sim, stream = state["sim"], state["stream"]
        with torch.cuda.stream(stream):
            sim.graph_launch(stream)
            h = sim.interface_heights(state["ifs"], RHO_L, RHO_V, WIDTH, stream=stream)
            field_spectrum(h, state["spec"], work=state["work"], stream=stream)
            return dict(f=sim.state(), h=h.to(state["dtype"]),
                        spec=state["spec"].to(state["dtype"]))
    if kind == "adjoint":
        f0, (rate, kT) = state["f0"], state["theta"]
        rho = final_density(f0, rate, kT, state["params"], case["steps"], case["every"])
        rho = rho.to(f0.dtype)
        loss = ((rho - state["target"]) ** 2).mean()
        g = torch.autograd.grad(loss, (f0, rate, kT))
        return dict(rho=rho.detach(), g_f0=g[0], g_rate=g[1], g_kT=g[2])
    if kind == "modeq":
        sim = state["sim"]
        sim.step(case["steps"])
        out = dict(f=sim.f)
        if case["snapshot"]:
            sim.moments(out=state["m"])
            field_spectrum(state["m"], state["spec"], work=state["work"])
            out["spec"] = state["spec"].to(state["dtype"])
        return out
    if kind == "batch":
        b = state["batch"]
        b.graph_launch(state["stream"])
        return [b.replica_state(r) for r in range(b.nrep)]
    return dict(spec=state["sim"].accumulate_spectrum(state["spec"]))


# ------------------------------------------------------------------ what a pass needs

def _fft_flops(dims, fields):
    v = math.prod(dims)
    return 2.5 * fields * v * math.log2(max(v, 2))


def work(case):
    """Bytes: every step reads and writes the populations once (the noise and
    the force come from what it reads); a snapshot reads the state and adds to
    its spectra; a reverse step reads the state and the adjoint and writes the
    adjoint (the checkpointed run also recomputes its states).  Flops: about
    6 Q + 12 per noise normal for a collision, 2.5 n log2 n for a real DFT."""
    kind = case["kind"]
    if kind == "batch":
        sites, q, s = sum(n ** 3 for n in _edges(case)), 19, 4 if case["precision"] == "fp32" else 8
        steps = case["steps"]
        return dict(bytes=2.0 * q * s * sites * steps, flops=500.0 * sites * steps)
    q = 19 if case.get("nz", 1) > 1 or case.get("lattice") == "D3Q19" else 9
    s = 4 if case["precision"] == "fp32" else 8
    v = case["nx"] * case["ny"] * case.get("nz", 1)
    steps = case.get("steps", 0)
    bytes_, flops = 2.0 * q * s * v * steps, (500.0 if q == 19 else 220.0) * v * steps
    dims = (case["nx"], case["ny"], case.get("nz", 1))
    if kind == "equilibration":
        bytes_ += q * s * v + 16.0 * (q + 1) * v
        flops += _fft_flops(dims, q)
    elif kind == "capillary":
        bytes_ += q * s * v + 40.0 * case["nx"]
        flops += 2 * case["nx"] * (51 * 40 * 4) + _fft_flops((case["nx"],), 2)
    elif kind == "adjoint":
        bytes_ += (2.0 + 3.0) * q * s * v * steps
        flops *= 4
    elif kind == "modeq":
        flops += 2 * steps * _fft_flops(dims, 2)
        if case["snapshot"]:
            bytes_ += q * s * v + 16.0 * q * v
            flops += _fft_flops(dims, q)
    elif kind == "spectrum":
        bytes_, flops = q * s * v + 16.0 * (q + 3) * v, _fft_flops(dims, q)
    return dict(bytes=bytes_, flops=flops)


# ------------------------------------------------------------------ 64-bit values

def _lattice(q):
    """(velocities, weights, basis rows, class of every row) of D2Q9 / D3Q19
    from the defining polynomials; classes c(onserved), b(ulk), s(hear), g(host)."""
    if q == 9:
        c = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0),
             (-1, -1, 0), (1, -1, 0)]
        w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
        row = lambda x, y, z, n: [  # noqa: E731
            1, x, y, 3 * n - 2, x * x - y * y, x * y, (3 * n - 4) * x, (3 * n - 4) * y,
            9 * n * n - 15 * n + 2]
        cls = "cccbssggg"
    else:
        c = [(0, 0, 0)] + [tuple(s if k == a else 0 for k in range(3)) for a in range(3)
                           for s in (1, -1)]
        c += [tuple(s if k == a else (t if k == b else 0) for k in range(3))
              for a, b in ((0, 1), (0, 2), (1, 2)) for s in (1, -1) for t in (1, -1)]
        w = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
        row = lambda x, y, z, n: [  # noqa: E731
            1, x, y, z, n - 1, 3 * x * x - n, y * y - z * z, x * y, y * z, z * x,
            (3 * n - 5) * x, (3 * n - 5) * y, (3 * n - 5) * z,
            (y * y - z * z) * x, (z * z - x * x) * y, (x * x - y * y) * z,
            3 * n * n - 6 * n + 1, (2 * n - 3) * (3 * x * x - n), (2 * n - 3) * (y * y - z * z)]
        cls = "ccccbsssss" + "g" * 9
    T = np.array([row(x, y, z, x * x + y * y + z * z) for x, y, z in c], dtype=np.float64).T
    return c, w, T, cls


def _philox(site, step, block, replica, seed):
    """Four 32-bit words (int64 tensors) of Philox4x32-10 at counter
    (site, step, block, replica), key = seed."""
    m32 = 0xFFFFFFFF
    x = [site, torch.full_like(site, step & m32), torch.full_like(site, block),
         torch.full_like(site, replica)]
    k0, k1 = seed & m32, (seed >> 32) & m32

    def mul(m, v):
        hi = ((m >> 16) * v + (((m & 0xFFFF) * v) >> 16)) >> 16
        return hi, (m * v) & m32

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, x[0])
        h1, l1 = mul(0xCD9E8D57, x[2])
        x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return x


def _normals(site, step, count, seed, replica=0):
    """``count`` Box-Muller normals per site: pair p takes its radius from
    word p and its angle from half of word P + p / 2."""
    pairs = (count + 1) // 2
    words = []
    for b in range((pairs + (pairs + 1) // 2 + 3) // 4):
        words += _philox(site, step, b, replica, seed)
    out = []
    for p in range(pairs):
        a = words[pairs + p // 2]
        h = (a >> 16) if p % 2 == 0 else (a & 0xFFFF)
        r = torch.sqrt(-2.0 * torch.log((words[p].double() + 1.0) * 2.0 ** -32))
        t = 2.0 * math.pi * ((h.double() + 1.0) * 2.0 ** -16)
        out += [r * torch.cos(t), r * torch.sin(t)]
    return out[:count]


def _at(phi, c):
    """phi(x + c) on the periodic box (dims z, y, x)."""
    return torch.roll(phi, shifts=(-c[2], -c[1], -c[0]), dims=(-3, -2, -1))


class _Fluid:
    """The fluctuating step in 64 bits on shifted populations (q, nz, ny, nx)."""

    def __init__(self, p, replica=0):
        self.p, self.replica, self.q = p, replica, 9 if p["lattice"] == "D2Q9" else 19
        self.d = 2 if self.q == 9 else 3
        self.c, self.w, T, self.cls = _lattice(self.q)
        self.N = (T ** 2 * np.array(self.w)).sum(1)
        dev = dict(dtype=torch.float64, device="cuda")
        self.T = torch.tensor(T, **dev)
        self.Tinv = torch.tensor(np.array(self.w)[:, None] * T.T / self.N, **dev)
        self.site = torch.arange(p["nx"] * p["ny"] * p["nz"], device="cuda",
                                 dtype=torch.int64).view(p["nz"], p["ny"], p["nx"])

    def initial(self, drho):
        r = torch.zeros(self.site.shape, dtype=torch.float64, device="cuda")
        if drho is not None:
            r = torch.as_tensor(drho, device="cuda").reshape(self.site.shape)
        return torch.tensor(self.w, dtype=torch.float64, device="cuda").view(-1, 1, 1, 1) * r

    def _rows(self, M, f):
        return torch.mm(M, f.reshape(self.q, -1)).view(self.q, *self.site.shape)

    def pulled(self, f):
        return self._rows(self.T, torch.stack([_at(f[i], [-v for v in self.c[i]])
                                               for i in range(self.q)]))

    def force(self, rho):
        p = self.p
        nb = [(w, c) for w, c in zip(self.w[1:], self.c[1:])]
        lap = sum(w * (_at(rho, c) - rho) for w, c in nb) * (2.0 / CS2)
        e = rho - p["rho_c"]
        mu = 2 * p["a"] * e + 4 * p["b"] * e ** 3 - p["kappa"] * lap

        def grad(phi):
            return [sum(w * c[k] * _at(phi, c) for w, c in nb if c[k]) / CS2 for k in range(self.d)]
        F = [-rho * g for g in grad(mu)]
        if p.get("eta", 0):
            F = [x + CS2 * g for x, g in zip(F, grad(rho))]
        return F

    def collide(self, m, n, rate_shear=None, kT=None):
        p, d = self.p, self.d
        rate_shear = p["rate_shear"] if rate_shear is None else rate_shear
        kT = p["kT"] if kT is None else kT
        rho = p["rho0"] + m[0]
        F = self.force(rho) if p.get("force_model") else [0.0] * d
        u = [(m[1 + k] + 0.5 * F[k]) / rho for k in range(d)]
        z = _normals(self.site, n, self.q - d - 1, p["seed"], self.replica)
        # equilibrium and forcing moments of a row Gamma_ab c_a c_b + gamma:
        # Gamma : rho u u and Gamma : (u F + F u)
        if d == 2:
            gam = [[(3, 0, 0), (3, 1, 1)], [(1, 0, 0), (-1, 1, 1)], [(1, 0, 1)]]
        else:
            gam = [[(1, 0, 0), (1, 1, 1), (1, 2, 2)], [(2, 0, 0), (-1, 1, 1), (-1, 2, 2)],
                   [(1, 1, 1), (-1, 2, 2)], [(1, 0, 1)], [(1, 1, 2)], [(1, 2, 0)]]
        out = [m[0]] + [m[1 + k] + F[k] for k in range(d)]
        for a in range(d + 1, self.q):
            lam = {"b": p["rate_bulk"], "s": rate_shear, "g": p["rate_ghost"]}[self.cls[a]]
            v = m[a] * (1.0 - lam)
            if a - d - 1 < len(gam):
                g = gam[a - d - 1]
                v = v + lam * rho * sum(k * u[i] * u[j] for k, i, j in g)
                if p.get("force_model"):
                    v = v + (1.0 - 0.5 * lam) * sum(k * (u[i] * F[j] + F[i] * u[j])
                                                    for k, i, j in g)
            amp = (rho * (float(self.N[a]) / CS2 * lam * (2.0 - lam))) ** 0.5 * kT ** 0.5
            out.append(v + amp * z[a - d - 1])
        return self._rows(self.Tinv, torch.stack(out))

    def step(self, f, n, *theta):
        return self.collide(self.pulled(f), n, *theta)

    def mode_rows(self, f):
        m = self.pulled(f)
        if self.p.get("force_model"):
            F = self.force(self.p["rho0"] + m[0])
            m = torch.cat([m[:1], torch.stack([m[1 + k] + 0.5 * F[k] for k in range(self.d)]),
                           m[1 + self.d:]])
        return m


def _spectra(m, pairs):
    """|m_a(k)|^2 of every field, then Re(m_1+a conj m_1+b) for the pairs."""
    M = [torch.fft.fftn(x) for x in m]
    out = [x.abs() ** 2 for x in M]
    out += [(M[1 + a] * M[1 + b].conj()).real for a, b in pairs]
    return torch.stack(out)


def _exact_adjoint(case, seed):
    from torch.utils.checkpoint import checkpoint
    fluid = _fluid(case)
    F = _Fluid(_params(case, seed, fluid))
    f0, target = _adjoint_inputs(case, seed)
    f0 = f0.double().requires_grad_(True)
    # the parameters as the program holds them
    th = [torch.tensor(float(torch.tensor(fluid[k], dtype=_dtype(case))), dtype=torch.float64,
                       device="cuda", requires_grad=True) for k in ("rate_shear", "kT")]

    def segment(f, rate, kT, k0, k1):
        for n in range(k0, k1):
            f = F.step(f, n, rate, kT)
        return f
    f = f0
    for k0 in range(0, case["steps"], 10):
        f = checkpoint(segment, f, *th, k0, min(k0 + 10, case["steps"]), use_reentrant=False)
    rho = F.p["rho0"] + F.pulled(f)[0]
    g = torch.autograd.grad(((rho - target.double()) ** 2).mean(), [f0] + th)
    return dict(rho=rho.detach(), g_f0=g[0], g_rate=g[1], g_kT=g[2])


def _exact_modeq(case, seed):
    p, nx, ny = MODEQ, case["nx"], case["ny"]
    c, w, T, cls = _lattice(9)
    dev = dict(dtype=torch.float64, device="cuda")
    N = (T ** 2 * np.array(w)).sum(1)
    Tt = torch.tensor(T, **dev)
    Ti = torch.tensor(np.array(w)[:, None] * T.T / N, **dev)
    site = torch.arange(nx * ny, device="cuda", dtype=torch.int64).view(1, ny, nx)
    cx = torch.cos(2 * math.pi * torch.arange(nx, **dev) / nx)[None, :]
    cy = torch.cos(2 * math.pi * torch.arange(ny, **dev) / ny)[:, None]
    c2 = p["cs2_0"] + p["kappa"] * p["rho0"] * ((4 / 3) * (2 - cx - cy) + (2 / 3) * (1 - cx * cy))
    le, ls, lg = p["rate_bulk"], p["rate_shear"], p["rate_ghost"]
    pre = 12 * p["rho0"] * p["kT"]
    l11 = (pre * le * (2 - le) * (2 - 3 * c2)).sqrt()
    l21 = pre * (3 * c2 - 1) * (le + lg - le * lg) / l11
    l22 = (pre * lg * (2 - lg) * (5 - 3 * c2) - l21 ** 2).sqrt()
    amp = [math.sqrt(p["rho0"] * p["kT"] * N[a] * lam * (2 - lam) / CS2)
           for a, lam in ((4, ls), (5, ls), (6, lg), (7, lg))]

    def pulled(f):
        g = torch.stack([_at(f[i], [-v for v in c[i]]) for i in range(9)])
        return torch.mm(Tt, g.reshape(9, -1)).view(9, 1, ny, nx)
    f = torch.zeros((9, 1, ny, nx), **dev)
    for n in range(case["steps"]):
        m = pulled(f)
        lap = sum(wi * (_at(m[0], ci) - m[0]) for wi, ci in zip(w[1:], c[1:])) * (2 / CS2)
        D = 6 * (p["cs2_0"] - CS2) * m[0] - 6 * p["kappa"] * p["rho0"] * lap
        z = _normals(site, n, 6, seed)
        ze, zp = torch.fft.fft2(z[0][0]), torch.fft.fft2(z[5][0])
        xe = torch.fft.ifft2(l11 * ze).real
        xp = torch.fft.ifft2(l21 * ze + l22 * zp).real
        lam = (0, 0, 0, le, ls, ls, lg, lg, lg)
        eq = {3: D, 8: -D}
        xi = {3: xe[None], 8: xp[None], **{4 + k: amp[k] * z[1 + k] for k in range(4)}}
        m = torch.stack([m[a] - lam[a] * (m[a] - eq.get(a, 0.0)) + xi.get(a, 0.0)
                         for a in range(9)])
        f = torch.mm(Ti, m.reshape(9, -1)).view(9, 1, ny, nx)
    out = dict(f=f.view(9, ny, nx))
    if case["snapshot"]:
        out["spec"] = _spectra(pulled(f), [])
    return out


def _exact_heights(rho, y_refs, n):
    """Gauss-Newton fit of the mean-field profile to every column (rho: y, x)."""
    out = []
    for y, sign in y_refs:
        y0 = int(math.floor(y + 0.5))
        k = torch.arange(-HALF_WINDOW, HALF_WINDOW + 1, device="cuda")
        r = rho[(y0 + k) % n]
        yk = (y0 + k).double()[:, None]
        h = torch.full((rho.shape[1],), float(y0), dtype=torch.float64, device="cuda")
        s = sign * 0.5 * (RHO_L - RHO_V)
        for _ in range(40):
            t = torch.tanh(2 / WIDTH * (yk - h))
            mp = s * (1 - t * t) * 2 / WIDTH
            step = ((r - 0.5 * (RHO_L + RHO_V) - s * t) * mp).sum(0) / (mp * mp).sum(0)
            h = (h - step).clamp(y0 - HALF_WINDOW, y0 + HALF_WINDOW)
        out.append(h)
    return torch.stack(out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "adjoint":
        return _exact_adjoint(case, seed)
    with torch.no_grad():
        if kind == "modeq":
            return _exact_modeq(case, seed)
        if kind == "batch":
            out = []
            for r, e in enumerate(_edges(case)):
                F = _Fluid(dict(IDEAL, lattice="D3Q19", nx=e, ny=e, nz=e, seed=seed + r), r)
                f = F.initial(None)
                for n in range(case["steps"]):
                    f = F.step(f, n)
                out.append(f)
            return out
        if kind == "spectrum":
            F = _Fluid(_params(case, seed, IDEAL, lattice="D3Q19"))
            m = F.mode_rows(_populations(case, seed, 19).double())
            return dict(spec=_spectra(m, [(0, 1), (1, 2), (2, 0)]))
        fluid = {"step": None, "equilibration": EQUILIBRATION, "capillary": CAPILLARY}[kind]
        p = _params(case, seed, fluid or _fluid(case))
        F = _Fluid(p)
        drho = (_drho(case, seed) if kind == "step" else
                _stripe(case, seed) if kind == "capillary" else None)
        f = F.initial(drho)
        stats = torch.zeros((2, F.q), dtype=torch.float64, device="cuda")
        for n in range(case["steps"]):
            m = F.pulled(f)
            if case.get("moments") and case["stats"] and (n + 1) % case["stats"] == 0:
                stats[0] += m.sum((1, 2, 3))
                stats[1] += (m * m).sum((1, 2, 3))
            f = F.collide(m, n)
        out = dict(f=f)
        if kind == "equilibration":
            out["spec"] = _spectra(F.mode_rows(f), [(0, 1)])
        elif kind == "capillary":
            y1, y2 = _stripe_at(case)
            h = _exact_heights(p["rho0"] + F.pulled(f)[0, 0], [(y1, 1), (y2, -1)], case["ny"])
            out["h"] = h
            out["spec"] = torch.stack([torch.fft.fft(x).abs() ** 2 for x in h])
        elif case.get("moments"):
            out["sum"], out["sumsq"] = stats[0].cpu().numpy(), stats[1].cpu().numpy()
        return out
