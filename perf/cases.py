"""Performance cases: what a user of this framework has it do, over the range of its use.

listed() names the standing cases, draw(rng) gives further ones of the same ranges, prepare()
builds what a program holds before the call (a handle, its inputs on the GPU), run() is one pass
through the public entry points, work() the bytes and operations a pass cannot do without, and
exact() the outputs in 64 bits from torch alone.

Every pass of a stepping case loads a state, advances it by a few steps and reads it back, so a
pass can be repeated on the same handle.  Inputs are smooth, domain-like unit fields with some
cell-to-cell noise (a film at work, neither uniform nor white).
"""
import math
import random

import numpy as np
import torch
import torch.utils.checkpoint

import paper_1501_07293_amd as mm
import synthetic

DEV = "cuda:0"
MU0 = 4.0e-7 * math.pi
RK4, EULER = "rk4", "euler"


def _sim_case(name, nx, ny, nz, **kw):
    c = dict(name=name, kind="step", nx=nx, ny=ny, nz=nz, dtype="f32", method=RK4, steps=8, dt=5e-14, cell=4e-9,
             alpha=0.1, ku=500.0, field=True, per_x=False, per_y=False, graph=False)
    c.update(kw)
    return c


def listed():
    return [
        # the small strip: a few microseconds of device work per step, launches and latency count
        _sim_case("strip_32x8x1_f32", 32, 8, 1, cell=5e-9, alpha=0.5, dt=1e-13, steps=32, graph=True),
        # the standard-problem-4 film of the paper's appendix under a time-dependent protocol
        # (saturate, ramp down, relax, reverse), explicit Euler, FP64, trace of <m>
        dict(name="protocol_166x42x1_f64", kind="schedule", nx=166, ny=42, nz=1, dtype="f64", steps=160, dt=5e-15,
             cell=3e-9, alpha=0.5, ku=0.0, every=20, graph=True),
        # gradient of a rollout with respect to a per-cell anisotropy map and the initial state
        # (forward with checkpoints, then the reverse sweep)
        dict(name="gradient_128x128x1_f32", kind="adjoint", nx=128, ny=128, nz=1, dtype="f32", steps=40, ckpt=20,
             dt=1e-13, cell=5e-9, alpha=0.1),
        # a mid-size film under a step field
        _sim_case("film_256x64x4_f32", 256, 64, 4, alpha=0.02, steps=32, graph=True),
        # the large film, in single and in double precision
        _sim_case("film_512x512x16_f32", 512, 512, 16, cell=3e-9, ku=0.0, field=False, steps=4),
        _sim_case("film_512x512x16_f64", 512, 512, 16, cell=3e-9, ku=0.0, field=False, steps=2, dtype="f64"),
        # a film whose sides are whatever the sample's outline gives: no powers of two, an odd
        # width, default padding
        _sim_case("film_301x190x6_f32", 301, 190, 6, steps=8),
        # a rectangle periodic in x and y, as for an extended film
        _sim_case("periodic_360x300x10_f32", 360, 300, 10, per_x=True, per_y=True, steps=8),
        # cube sweep (the shape of the paper's own benchmark): explicit Euler
        _sim_case("cube_128_f32", 128, 128, 128, method=EULER, cell=34e-9 / 128, alpha=1.0, dt=1e-14, ku=6.283e4,
                  field=False, steps=8, graph=True),
        # read-out of a state in double precision: effective field, energies, largest torque
        dict(name="readout_100x80x50_f64", kind="readout", nx=100, ny=80, nz=50, dtype="f64", cell=4e-9, ku=500.0),
        # many uneven small grids in one handle: default padding, and power-of-two padding
        dict(name="batch_512_f32", kind="batch", n=512, lo=32, hi=128, dtype="f32", steps=2, dt=1e-13, pow2=False,
             shapes=0, graph=True),
        dict(name="batch_512_pow2_f32", kind="batch", n=512, lo=32, hi=128, dtype="f32", steps=4, dt=1e-13,
             pow2=True, shapes=0, graph=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _smooth7(n):
    for p in (2, 3, 5, 7):
        while n % p == 0:
            n //= p
    return n == 1


def _period(rng, lo, hi):
    while True:
        n = _log_int(rng, lo, hi)
        if _smooth7(n):
            return n


def draw(rng: random.Random):
    kind = rng.choice(["film", "film", "film", "cube", "periodic", "schedule", "adjoint", "readout", "batch", "batch"])
    dtype = "f64" if rng.random() < 0.3 else "f32"
    if kind == "film":
        nx, ny, nz = _log_int(rng, 20, 512), _log_int(rng, 8, 512), rng.choice([1, 1, 2, 3, 4, 6, 10, 16])
        c = _sim_case("", nx, ny, nz, dtype=dtype, method=rng.choice([RK4, RK4, EULER]), graph=rng.random() < 0.5)
        c["steps"] = 16 if nx * ny * nz < 1 << 18 else (4 if nx * ny * nz < 1 << 21 else 1)
    elif kind == "cube":
        n = _log_int(rng, 8, 160)
        c = _sim_case("", n, n, n, dtype=dtype, method=EULER, cell=34e-9 / n, alpha=1.0, dt=1e-14, ku=6.283e4,
                      field=False, graph=True)
        c["steps"] = 16 if n <= 64 else 4
    elif kind == "periodic":
        nx, ny, nz = _period(rng, 32, 512), _period(rng, 32, 512), rng.choice([1, 2, 4, 8, 12])
        c = _sim_case("", nx, ny, nz, dtype=dtype, per_x=True, per_y=rng.random() < 0.7)
        c["steps"] = 8 if nx * ny * nz < 1 << 19 else 2
    elif kind == "schedule":
        c = dict(kind="schedule", nx=_log_int(rng, 32, 300), ny=_log_int(rng, 12, 150), nz=1, dtype="f64", steps=160,
                 dt=5e-15, cell=3e-9, alpha=0.5, ku=0.0, every=20, graph=True)
    elif kind == "adjoint":
        c = dict(kind="adjoint", nx=_log_int(rng, 24, 160), ny=_log_int(rng, 24, 160), nz=rng.choice([1, 1, 2]),
                 dtype=dtype, steps=20, ckpt=rng.choice([7, 10, 20]), dt=1e-13, cell=5e-9, alpha=0.1)
    elif kind == "readout":
        c = dict(kind="readout", nx=_log_int(rng, 16, 160), ny=_log_int(rng, 16, 160), nz=_log_int(rng, 1, 100),
                 dtype="f64", cell=4e-9, ku=500.0)
    else:
        c = dict(kind="batch", n=_log_int(rng, 8, 384), lo=rng.choice([16, 32]), hi=rng.choice([64, 96, 128]),
                 dtype=dtype, steps=2, dt=1e-13, pow2=rng.random() < 0.5, shapes=rng.randrange(1, 1000),
                 graph=rng.random() < 0.5)
    c.pop("name", None)
    return c


# ---------------------------------------------------------------- inputs
def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _state(nx, ny, nz, seed, device):
    """Smooth unit field with noise, (3, nz, ny, nx) float64."""
    g = np.random.default_rng(seed)
    ax = [torch.arange(n, dtype=torch.float64, device=device) / n for n in (nz, ny, nx)]
    z, y, x = ax[0][:, None, None], ax[1][None, :, None], ax[2][None, None, :]
    out = torch.empty((3, nz, ny, nx), dtype=torch.float64, device=device)
    for a in range(3):
        f = torch.full((nz, ny, nx), float(g.normal() * (2.0 if a == 0 else 0.5)), dtype=torch.float64, device=device)
        for _ in range(4):
            kx, ky, kz, ph, am = g.uniform(0, 3), g.uniform(0, 3), g.uniform(0, 1), g.uniform(0, 2 * math.pi), g.normal()
            f = f + float(am) * torch.cos(2 * math.pi * (float(kx) * x + float(ky) * y + float(kz) * z) + float(ph))
        # noise in +-0.15: an integer hash of the cell number
        n = torch.arange(nz * ny * nx, dtype=torch.int64, device=device).reshape(nz, ny, nx)
        h = (n * 2654435761 + (int(seed) % 65536) * 40503 + a * 97531) & 0xFFFFFFFF
        h = ((h ^ (h >> 15)) * 1140671485 + 12820163) & 0xFFFFFFFF
        h = ((h ^ (h >> 13)) * 1103515245 + 12345) & 0xFFFFFFFF
        out[a] = f + 0.3 * (h.double() / 4294967296.0 - 0.5)
    return out / torch.sqrt((out * out).sum(0, keepdim=True))


def _given(case, seed, device):
    """The initial state in the case's precision."""
    return _state(case["nx"], case["ny"], case["nz"], seed, device).to(_dtype(case))


def _hext(case, seed):
    if not case.get("field"):
        return (0.0, 0.0, 0.0)
    g = np.random.default_rng(seed + 1)
    return tuple(float(v) for v in synthetic.mT_to_Apm(np.array([-20.0, 3.0, 0.0]) * g.uniform(0.8, 1.2)))


def _ku_map(case, seed, device):
    g = np.random.default_rng(seed + 2)
    ku = 500.0 + 50.0 * g.standard_normal((case["nz"], case["ny"], case["nx"]))
    return torch.from_numpy(ku).to(device=device, dtype=_dtype(case))


def _cotangent(case, seed, device):
    g = np.random.default_rng(seed + 3)
    w = g.standard_normal((3, case["nz"], case["ny"], case["nx"]))
    return torch.from_numpy(w).to(device=device, dtype=_dtype(case))


def _pieces(case):
    """The appendix protocol (saturate, ramp to zero, relax, reverse) over case["steps"] steps."""
    q = case["steps"] // 8
    sat, zero, rev = (1.0e5, 1.0e5, 1.0e5), (0.0, 0.0, 0.0), (-19.576e3, 3.422e3, 0.0)
    return [(q, sat, sat, 0.5), (q, sat, zero, 0.5), (2 * q, zero, zero, 0.5),
            (case["steps"] - 4 * q, rev, rev, 0.02)]


def _grids(case):
    """Grids and applied fields of a batch case: nx, ny uniform in [lo, hi], nz 1 or 2."""
    s = synthetic.batch_samples(case["n"], seed=case["shapes"], lo=case["lo"], hi=case["hi"])
    return [(q.nx, q.ny, q.nz) for q in s], np.array([q.hext for q in s])


def _batch_states(case, seed, device):
    grids, _ = _grids(case)
    return [_state(*g, seed=seed + 7 * i, device=device).to(_dtype(case)) for i, g in enumerate(grids)]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        grids, hext = _grids(case)
        b = mm.BatchSim(grids, 5e-9, Ku=500.0, alpha=0.5, hext=hext, precision=case["dtype"], graph=case["graph"],
                        pow2_pad=case["pow2"], device=DEV)
        flat = torch.cat([m.reshape(-1) for m in _batch_states(case, seed, DEV)])
        return dict(case=case, sim=b, m0=flat)
    kw = dict(Ku=case["ku"]) if "ku" in case else {}
    sim = mm.Sim(case["nx"], case["ny"], case["nz"], case["cell"], alpha=case.get("alpha", 0.5),
                 precision=case["dtype"], graph=case.get("graph", False),
                 periodic=(case.get("per_x", False), case.get("per_y", False), False), device=DEV, **kw)
    st = dict(case=case, sim=sim, m0=_given(case, seed, DEV))
    if kind == "adjoint":
        st["ku"] = _ku_map(case, seed, DEV)
        st["w"] = _cotangent(case, seed, DEV)
    else:
        sim.set_hext(_hext(case, seed))
    return st


def run(state):
    case, sim = state["case"], state["sim"]
    kind = case["kind"]
    if kind == "step":
        sim.set_m(state["m0"])
        (sim.step if case["method"] == RK4 else sim.step_euler)(case["steps"], case["dt"])
        return sim.get_m()
    if kind == "schedule":
        sim.set_m(state["m0"])
        trace = sim.run_schedule(_pieces(case), case["dt"], case["every"], method="euler")
        return {"trace": trace, "m": sim.get_m()}
    if kind == "adjoint":
        ku = state["ku"].clone().requires_grad_(True)
        m0 = state["m0"].clone().requires_grad_(True)
        m = mm.rollout(sim, ku, m0, case["steps"], case["dt"], ckpt_every=case["ckpt"])
        m.backward(state["w"])
        return {"m": m.detach(), "dku": ku.grad, "dm0": m0.grad}
    if kind == "readout":
        sim.set_m(state["m0"])
        return {"field": sim.field("eff"), "energy": sim.energy(), "torque": sim.max_torque()}
    sim.set_m(state["m0"])
    sim.step(case["steps"], case["dt"])
    return sim.get_m_flat()


# ---------------------------------------------------------------- least work
def _grid_flops(nx, ny, nz, evals, per):
    """Operations of `evals` field evaluations: three real-to-complex transforms each way over the
    least padded size (x lines of the grid's own rows, y lines of its own planes, every z line),
    the tensor product, and the local terms with the stage update."""
    px, py, pz = (nx if per[0] else 2 * nx), (ny if per[1] else 2 * ny), (1 if nz == 1 else 2 * nz)
    hx = px // 2 + 1
    lines = 2.5 * px * math.log2(px) * ny * nz + 5 * py * math.log2(py) * nz * hx
    if pz > 1:
        lines += 5 * pz * math.log2(pz) * py * hx
    return evals * (6 * lines + 30 * hx * py * pz + 80 * nx * ny * nz)


def _octant_bytes(nx, ny, nz, esz, per):
    """The kernel spectrum of a grid (real, one octant, 4 or 6 components)."""
    return (6 if nz > 1 else 4) * ((nx // 2 if per[0] else nx) + 1) * ((ny // 2 if per[1] else ny) + 1) * \
        (nz + 1 if nz > 1 else 1) * esz


def work(case):
    """The state in and out once per step (it need not leave the chip between a step's stages) and
    the kernel spectrum once per pass."""
    esz = 4 if case["dtype"] == "f32" else 8
    kind = case["kind"]
    grids = _grids(case)[0] if kind == "batch" else [(case["nx"], case["ny"], case["nz"])]
    per = (case.get("per_x", False), case.get("per_y", False))
    steps = case.get("steps", 1)
    nbytes = flops = 0.0
    for nx, ny, nz in grids:
        n = nx * ny * nz
        # a gradient runs each step three times: forward, recomputed, reversed
        per_step = 1 if kind == "schedule" or case.get("method") == EULER else 4
        evals = {"readout": 1, "adjoint": 3 * steps * per_step}.get(kind, steps * per_step)
        passes = {"readout": 1, "adjoint": 3 * steps}.get(kind, steps)
        flops += _grid_flops(nx, ny, nz, evals, per)
        nbytes += 6 * n * esz * passes + _octant_bytes(nx, ny, nz, esz, per)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- 64-bit reference (torch only)
def _corner_sum(comp, X, Y, Z):
    """Point tensor (atan / log corner sums) at offsets X, Y, Z in cells, broadcast FP64."""
    s = 0.0
    for i in (0, 1):
        for j in (0, 1):
            for k in (0, 1):
                x, y, z = X + (i - 0.5), Y + (j - 0.5), Z + (k - 0.5)
                r = torch.sqrt(x * x + y * y + z * z)
                if comp == 0:
                    t = torch.atan(y * z / (x * r))
                elif comp == 3:
                    t = torch.atan(x * z / (y * r))
                elif comp == 5:
                    t = torch.atan(x * y / (z * r))
                else:
                    a, b, c = {1: (x, y, z), 2: (x, z, y), 4: (y, z, x)}[comp]
                    one = torch.ones_like(r)
                    c = c * one
                    t = torch.where(c >= 0, torch.log(torch.clamp(c + r, min=1e-300)), torch.log((a * a + b * b) / (r - c) * one))
                s = s - t if (i + j + k) & 1 else s + t
    s = s / (4 * math.pi)
    return s if comp in (0, 3, 5) else -s


class _Exact:
    """Field and steps in 64 bits: torch.fft on a padded grid, plain torch elsewhere.  States are
    (G, 3, nz, ny, nx); G > 1 are grids of uneven sizes in one box, `inside` (G, 1, nz, ny, nx)
    marking the cells of each (the demag tensor depends on the offset of two cells alone)."""

    def __init__(self, nx, ny, nz, cell, ku, alpha, hext, per=(False, False), device="cpu", inside=None,
                 Ms=8.0e5, A=1.3e-11, gamma=2.211e5):
        self.n, self.per, self.Ms, self.alpha, self.gamma = (nz, ny, nx), (False, per[1], per[0]), Ms, alpha, gamma
        self.cex, self.kfac = 2 * A / (MU0 * Ms * Ms * cell * cell), 2 / (MU0 * Ms * Ms)
        self.A, self.cell, self.ku, self.inside = A, cell, ku, inside
        self.set_field(torch.tensor(hext, dtype=torch.float64, device=device))
        # open axes take a power of two of at least 2 n points (the library has kernels for it at hand)
        self.p = tuple(n if p else (1 if n == 1 else 1 << (2 * n - 1).bit_length()) for n, p in zip(self.n, self.per))
        # wrapped offsets per axis; along a period the nearest image, and at exactly half an even
        # period the two equally near ones, one half each
        options = []
        for P, p in zip(self.p, self.per):
            r = torch.arange(P, dtype=torch.float64, device=device)
            d = torch.where(2 * r > P, r - P, r)
            options.append([d, torch.where(2 * r == P, -d, d)] if p and P % 2 == 0 else [d])
        self.k = []
        for c in range(6):
            t, terms = 0.0, 0
            for z in options[0]:
                for y in options[1]:
                    for x in options[2]:
                        t = t + _corner_sum(c, x[None, None, :], y[None, :, None], z[:, None, None])
                        terms += 1
            t = (t / terms).expand(self.p).clone()
            for ax, (P, p) in enumerate(zip(self.p, self.per)):
                if not p and P > 1:  # the padding's middle offset meets no pair of cells
                    t.narrow(ax, P // 2, 1).zero_()
            self.k.append(torch.fft.rfftn(t).real.clone())

    def set_field(self, h):
        self.h = h.reshape(-1, 3, 1, 1, 1) / self.Ms

    def demag(self, m):
        f = [torch.fft.rfftn(m[:, d], s=self.p, dim=(1, 2, 3)) for d in range(3)]
        k = self.k
        rows = ((0, 1, 2), (1, 3, 4), (2, 4, 5))
        nz, ny, nx = self.n
        return torch.stack([torch.fft.irfftn(sum(k[r[d]] * f[d] for d in range(3)), s=self.p, dim=(1, 2, 3))[:, :nz, :ny, :nx]
                            for r in rows], 1)

    def lap(self, m):
        out = torch.zeros_like(m)
        for ax in (2, 3, 4):
            n = m.shape[ax]
            if n > 1:
                d = m.narrow(ax, 1, n - 1) - m.narrow(ax, 0, n - 1)
                if self.inside is not None:
                    d = d * (self.inside.narrow(ax, 1, n - 1) * self.inside.narrow(ax, 0, n - 1))
                z = torch.zeros_like(m.narrow(ax, 0, 1))
                out = out + torch.cat([d, z], ax) - torch.cat([z, d], ax)
                if self.per[ax - 2]:
                    w = m.narrow(ax, 0, 1) - m.narrow(ax, n - 1, 1)
                    zz = torch.zeros_like(m.narrow(ax, 0, n - 1))
                    out = out + torch.cat([zz, w], ax) - torch.cat([w, zz], ax)
        return out

    def field(self, m):
        """Reduced effective field."""
        zero = torch.zeros_like(m[:, 0])
        return self.cex * self.lap(m) + torch.stack([self.kfac * self.ku * m[:, 0], zero, zero], 1) + self.h + self.demag(m)

    def rate(self, m, dt):
        t = torch.linalg.cross(m, self.field(m), dim=1)
        g = self.gamma * self.Ms * dt / (1 + self.alpha ** 2)
        return -g * (t + self.alpha * torch.linalg.cross(m, t, dim=1))

    def unit(self, v):
        r = torch.sqrt((v * v).sum(1, keepdim=True))
        return v / (r if self.inside is None else torch.where(self.inside > 0, r, torch.ones_like(r)))

    def rk4(self, m, dt):
        a = self.rate(m, dt)
        b = self.rate(m + 0.5 * a, dt)
        c = self.rate(m + 0.5 * b, dt)
        d = self.rate(m + c, dt)
        return self.unit(m + (a + 2 * b + 2 * c + d) / 6)

    def euler(self, m, dt):
        return self.unit(m + self.rate(m, dt))


def _exact_batch(case, seed, dev):
    """The grids of a batch by thickness, 64 at a time in one box that holds the largest."""
    grids, hext = _grids(case)
    states = _batch_states(case, seed, dev)
    out = [None] * len(grids)
    for nz in sorted({g[2] for g in grids}):
        ids = [i for i, g in enumerate(grids) if g[2] == nz]
        e = _Exact(case["hi"], case["hi"], nz, 5e-9, 500.0, 0.5, (0.0, 0.0, 0.0), device=dev)
        for at in range(0, len(ids), 64):
            part = ids[at:at + 64]
            m = torch.zeros((len(part), 3, nz, case["hi"], case["hi"]), dtype=torch.float64, device=dev)
            e.inside = torch.zeros_like(m[:, :1])
            for q, i in enumerate(part):
                nx, ny, _ = grids[i]
                m[q, :, :, :ny, :nx] = states[i].double()
                e.inside[q, :, :, :ny, :nx] = 1.0
            e.set_field(torch.from_numpy(hext[part]).to(dev))
            m = e.unit(m)
            for _ in range(case["steps"]):
                m = e.rk4(m, case["dt"]) * e.inside
            for q, i in enumerate(part):
                nx, ny, _ = grids[i]
                out[i] = m[q, :, :, :ny, :nx].reshape(-1)
    return torch.cat(out)


def exact(case, seed):
    dev = DEV if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "batch":
        return _exact_batch(case, seed, dev)
    per = (case.get("per_x", False), case.get("per_y", False))
    m = _given(case, seed, dev).double()
    hext = _hext(case, seed) if kind != "adjoint" else (0.0, 0.0, 0.0)
    ku = _ku_map(case, seed, dev).double() if kind == "adjoint" else case.get("ku", 0.0)
    e = _Exact(case["nx"], case["ny"], case["nz"], case["cell"], ku, case.get("alpha", 0.5), hext, per, dev)
    if kind == "adjoint":
        ku.requires_grad_(True)
        m.requires_grad_(True)
        v = e.unit(m[None])
        for _ in range(case["steps"]):
            v = torch.utils.checkpoint.checkpoint(e.rk4, v, case["dt"], use_reentrant=False)
        v[0].backward(_cotangent(case, seed, dev).double())
        return {"m": v.detach()[0], "dku": ku.grad, "dm0": m.grad}
    m = e.unit(m[None])
    if kind == "step":
        for _ in range(case["steps"]):
            m = e.rk4(m, case["dt"]) if case["method"] == RK4 else e.euler(m, case["dt"])
        return m[0]
    if kind == "schedule":
        rows, done = [], 0
        for steps, h0, h1, alpha in _pieces(case):
            e.alpha = alpha
            h0, h1 = np.array(h0), np.array(h1)
            for n in range(steps):
                e.set_field(torch.from_numpy(h0 + (h1 - h0) * (n / steps)).to(dev))
                m = e.euler(m, case["dt"])
                done += 1
                if done % case["every"] == 0:
                    t = torch.tensor([done * case["dt"]], dtype=torch.float64, device=dev)
                    rows.append(torch.cat([t, m.mean((2, 3, 4))[0]]))
        return {"trace": torch.stack(rows), "m": m[0]}
    h, hd = e.field(m), e.demag(m)
    vol, js = case["cell"] ** 3, MU0 * e.Ms * e.Ms
    pairs = sum(((m.narrow(ax, 1, m.shape[ax] - 1) - m.narrow(ax, 0, m.shape[ax] - 1)) ** 2).sum() for ax in (2, 3, 4) if m.shape[ax] > 1)
    parts = [float(e.A * case["cell"] * pairs), float(case["ku"] * vol * (m[:, 1] ** 2 + m[:, 2] ** 2).sum()),
             float(-0.5 * js * vol * (m * hd).sum()), float(-js * vol * (m * e.h).sum())]
    torque = float(torch.sqrt((torch.linalg.cross(m, h, dim=1) ** 2).sum(1)).max()) * e.Ms
    return {"field": h[0] * e.Ms, "energy": np.array(parts + [sum(parts)]), "torque": torque}
